"""Direct tiles (pb_conv.h) against the oracle.  3x3 layers: every wave tile, chunks and splits of the reduction, maps whose
rows and pixel counts fit no tile, stride 2 on even and odd maps, in all three passes, with the update inside the
weight-gradient tiles (odd and even numbers of ticks) and without (stashing, updates every two samples).  1x1 layers on
small maps: 1 to 49 pixels, stride 2."""
import re

import numpy as np
import pytest

import pb_workloads as W
from tests.parity_util import assert_tensors_follow, reference

pytestmark = pytest.mark.gpu


def _net(widths, hw, groups=4):
    return W._net("conv3", W.preact_resnet_basic(widths, 1, groups, in_c=3, n_classes=5), 3, hw, hw, 5, 1e-3, 0.9, 8, 3, 8)


@pytest.mark.parametrize("budget", [1.0, 14.0, 24.0, 400.0])
@pytest.mark.parametrize("widths,hw", [((16, 32), 7), ((32, 64), 13), ((64, 128), 14), ((64, 64, 128), 32), ((48, 80), 20), ((128, 256), 8),
                                       ((16, 256), 4)])
def test_direct_tiles_follow_the_oracle(widths, hw, budget):
    from paper_2003_11666_amd.binding import plan_summary
    net, tuning = _net(widths, hw), dict(tile_budget_us=budget)
    plan = plan_summary(net, tuning=tuning)
    assert {m for m in re.findall(r"gm(\d) .* direct", plan)} == {"1", "2", "3"}, plan
    _follow(net, tuning)


def _follow(net, tuning, tol=1e-4, **kw):
    from paper_2003_11666_amd import PBEngine
    (xs, ys), S = W.sample_pool(net), len(net["stages"])
    eng, ref = PBEngine(net, tuning=tuning, **kw), reference(net, (2 * S + 4, 2 * S + 5), **kw)
    for n, want in ref.items():
        for t in range(eng.ticks, n):
            eng.tick(xs[t % len(ys)], ys[t % len(ys)])
        for k in ("read_weights", "read_velocity", "loss_history"):
            assert np.linalg.norm(getattr(eng, k)() - want[k]) < tol * np.linalg.norm(want[k]), k
        assert_tensors_follow(eng, want)
    eng.close()


# maps of fewer than 16 pixels stay on the fp32 pipes at a multiple of 32 channels too, their predicted weights in those tiles' order
@pytest.mark.parametrize("widths,hw", [((64, 128), 6), ((96, 160), 5), ((32, 64, 96), 9)])
def test_lane_order_on_maps_of_a_few_pixels(widths, hw):
    from paper_2003_11666_amd.binding import plan_summary
    net, tuning = _net(widths, hw), dict(tile_budget_us=24.0)
    steps = [l for l in plan_summary(net, tuning=tuning).splitlines() if "direct" in l and "k3" in l]
    for gm in ("gm1", "gm3"):
        assert any(f"| {gm} " in l and l.endswith("predicted in lanes/4") for l in steps), steps
    _follow(net, tuning)


@pytest.mark.parametrize("kw", [dict(lwp_form="w"), dict(bwd_weights=1), dict(update_size=2), dict(mitigation=0)])
def test_direct_tiles_with_other_updates(kw):
    _follow(_net((32, 64), 8), dict(tile_budget_us=14.0), **kw)


@pytest.mark.parametrize("budget", [1.0, 400.0])
@pytest.mark.parametrize("hw,layers", [(8, (1, 1)), (16, (1, 2)), (32, (1, 1, 1)), (56, (1, 1)), (24, (1, 1))])
def test_small_1x1_tiles_follow_the_oracle(hw, layers, budget):
    from paper_2003_11666_amd.binding import plan_summary
    net = W._net("small1", W.preact_resnet_bottleneck(layers, 64, 16, n_classes=5), 3, hw, hw, 5, 1e-3, 0.9, 8, 3, 8)
    plan = plan_summary(net, tuning=dict(tile_budget_us=budget))
    assert {m for m in re.findall(r"gm(\d) .* small", plan)} == {"1", "2"}, plan
    # (a ReLU or a pooling window decided the other way by the last bit shows in the gradients of 200 000 activations)
    _follow(net, dict(tile_budget_us=budget), tol=2e-3)
