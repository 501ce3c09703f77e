"""Products of fp32 operands on the bf16 matrix pipes (pb_split.h) against the oracle."""
import re

import pytest

import pb_workloads as W
from tests.test_gpu_conv3 import _follow

pytestmark = pytest.mark.gpu


# maps of 8x8 to 16x16 behind the stem: pixel counts that are and are not multiples of 4 and of the tiles' columns, stride 2
# on even maps, 64 and 128 channels (tiles of 64 and 128 rows)
@pytest.mark.parametrize("base", [64, 128])
@pytest.mark.parametrize("hw,layers", [(32, (2,)), (36, (2,)), (52, (1, 1)), (64, (1, 1)), (40, (1, 1))])
def test_dense_1x1_tiles_follow_the_oracle(base, hw, layers):
    from paper_2003_11666_amd.binding import plan_summary
    net = W._net("dense1", W.preact_resnet_bottleneck(layers, base, 16, n_classes=5), 3, hw, hw, 5, 1e-3, 0.9, 8, 3, 8)
    tuning = dict(tile_budget_us=24.0)
    plan = plan_summary(net, tuning=tuning)
    assert {m for m in re.findall(r"gm(\d) .* dense", plan)} == {"1", "2", "3"}, plan
    # (a ReLU or a pooling window decided the other way by the last bit shows in the gradients of 200 000 activations)
    _follow(net, tuning, tol=2e-3)


def _basic(widths, hw):
    return W._net("split3", W.preact_resnet_basic(widths, 1, 4, in_c=3, n_classes=5), 3, hw, hw, 5, 1e-3, 0.9, 8, 3, 8)


# 3x3 layers: one to six blocks of 32 channels dealt out to one, two or four waves, every wave tile, maps of 16 pixels and more
# whose rows and pixel counts fit no tile, both strides; 48 channels next to them stay on the fp32 pipes
@pytest.mark.parametrize("budget", [1.0, 18.0, 26.0, 400.0])
@pytest.mark.parametrize("widths,hw", [((32, 96), 9), ((64, 64), 12), ((96, 192), 8), ((128, 128), 17), ((48, 96), 10), ((64, 128, 256), 32)])
def test_split_3x3_tiles_follow_the_oracle(widths, hw, budget):
    from paper_2003_11666_amd.binding import plan_summary
    net, tuning = _basic(widths, hw), dict(tile_budget_us=budget)
    plan = plan_summary(net, tuning=tuning)
    assert {m for m in re.findall(r"gm(\d) .* split", plan)} == {"1", "2"}, plan
    _follow(net, tuning)


def test_every_wave_tile_of_the_split_form_is_planned_above():
    from paper_2003_11666_amd.binding import plan_summary
    seen = set()
    for widths, hw in [((32, 96), 9), ((64, 64), 12), ((96, 192), 8), ((128, 128), 17), ((48, 96), 10), ((64, 128, 256), 32)]:
        for budget in (1.0, 18.0, 26.0, 400.0):
            seen |= set(re.findall(r"gm(\d) .* (mi\d ni\d) .* split", plan_summary(_basic(widths, hw), tuning=dict(tile_budget_us=budget))))
    assert {s for _, s in seen} == {"mi2 ni4", "mi2 ni2", "mi2 ni1", "mi1 ni2", "mi1 ni1"}, seen


# layers whose weights lie in the order of their tiles' lanes: read back before the first gradient they are the initial ones
@pytest.mark.parametrize("ticks", [0, 1, 2])
def test_weights_in_lane_order_read_back_in_their_own(ticks):
    import numpy as np
    from oracle import pb_oracle as O
    from paper_2003_11666_amd import PBEngine
    net = _basic((64, 96), 12)
    xs, ys = W.sample_pool(net)
    eng = PBEngine(net, tuning=dict(tile_budget_us=26.0))
    for t in range(ticks):
        eng.tick(xs[t], ys[t])
    want = O.PBOracle(net).read_weights().astype(np.float32)
    assert np.array_equal(eng.read_weights(), want) and not eng.read_velocity().any()
    eng.close()


def test_a_read_back_leaves_the_training_as_it_was():
    """Read-backs in canonical order go by way of the gradients' block, from ticks before a stage's first gradient on."""
    import numpy as np
    from paper_2003_11666_amd import PBEngine
    net = _basic((64, 96), 12)
    (xs, ys), S = W.sample_pool(net), len(net["stages"])
    one, other = (PBEngine(net, tuning=dict(tile_budget_us=26.0)) for _ in range(2))
    for t in range(2 * S + 4):
        for e in (one, other):
            e.tick(xs[t % len(ys)], ys[t % len(ys)])
        one.read_weights(), one.read_velocity()
    for k in ("read_weights", "read_velocity", "loss_history"):
        assert np.array_equal(getattr(one, k)(), getattr(other, k)()), k
    one.close(), other.close()
