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


SPLIT = [((32, 96), 9), ((64, 64), 12), ((96, 192), 8), ((128, 128), 17), ((48, 96), 10), ((64, 128, 256), 32), ((128, 256), 29)]
BUDGETS = [1.0, 18.0, 22.0, 26.0, 400.0]
ORDERS = [dict(), dict(bwd_weights=1)]   # weights in the order of the tiles' lanes where the layer allows it, and in their own


# 3x3 layers: one to six blocks of 32 channels dealt out to one, two or four waves, every wave tile, maps of 16 pixels and more
# whose rows and pixel counts fit no tile, both strides; 48 channels next to them stay on the fp32 pipes
@pytest.mark.parametrize("kw", ORDERS, ids=["lanes", "own"])
@pytest.mark.parametrize("budget", BUDGETS)
@pytest.mark.parametrize("widths,hw", SPLIT)
def test_split_3x3_tiles_follow_the_oracle(widths, hw, budget, kw):
    from paper_2003_11666_amd.binding import plan_summary
    net, tuning = _basic(widths, hw), dict(tile_budget_us=budget)
    plan = plan_summary(net, tuning=tuning, **kw)
    assert {m for m in re.findall(r"gm(\d) .* split", plan)} == {"1", "2"}, plan
    _follow(net, tuning, **kw)


def test_every_wave_tile_of_the_split_form_is_planned_above():
    """Per pass (backward data of stride 2 is one of its own), wave tile and order of the weights."""
    from paper_2003_11666_amd.binding import plan_summary
    seen = set()
    for widths, hw in SPLIT:
        for budget in BUDGETS:
            for kw in ORDERS:
                for l in plan_summary(_basic(widths, hw), tuning=dict(tile_budget_us=budget), **kw).splitlines():
                    m = re.search(r"k3 s(\d) \| gm([12]) .* (mi\d ni\d) .* split(.*)$", l)
                    if m:
                        seen.add(("gm" + m[2] + (" s2" if m[2] == "2" and m[1] == "2" else ""), m[3], "lanes" in m[4]))
    tiles = ["mi2 ni2", "mi2 ni1", "mi1 ni2", "mi1 ni1"]
    want = {(p, t, lanes) for p in ("gm1", "gm2") for t in tiles for lanes in (False, True)} | {(p, "mi2 ni4", True) for p in ("gm1", "gm2")}
    assert seen == want | {("gm2 s2", t, lanes) for t in tiles[2:] for lanes in (False, True)}, seen


def _bottleneck(layers, base, hw):
    return W._net("split1", W.preact_resnet_bottleneck(layers, base, 16, n_classes=5), 3, hw, hw, 5, 1e-3, 0.9, 8, 3, 8)


def _vgg(widths, pools, hw):
    return W._net("splitv", W.vgg(widths, pools, 8, n_classes=5, in_hw=hw), 3, hw, hw, 5, 1e-3, 0.9, 8, 3, 8)


@pytest.mark.parametrize("net", [_basic((64, 96), 12), _basic((32, 96), 9), _basic((64, 128), 32), _bottleneck((2,), 64, 32),
                                 _bottleneck((1, 1), 64, 40), _bottleneck((1,), 128, 36), _vgg((64, 128, 256, 256), (0, 1), 24)],
                         ids=lambda n: f"{n['name']}-{n['in_h']}-{W.count_params(n)}")
def test_gradients_are_as_near_float64_as_those_of_fp32_products(net):
    """Weights held fixed and no momentum: the velocity is the gradient of each stage's latest sample.  Its distance from float64
    (2-norm, per weight tensor) is up to 5.1e-7 in these networks, and up to 6.5e-7 with every product on the fp32 pipes; pieces
    that lose their last 8 bits (x = h + m) leave 5e-6 to 7e-6 in every sum they take part in, forward or backward."""
    import numpy as np
    from oracle import pb_oracle as O
    from paper_2003_11666_amd import PBEngine
    from paper_2003_11666_amd.binding import plan_summary
    from tests.parity_util import tensor_slices
    (xs, ys), S = W.sample_pool(net), len(net["stages"])
    weights = [q for q in tensor_slices(net) if q[1] in ("w", "wp")]
    forms = dict(lanes=dict(tuning=dict(tile_budget_us=26.0)), own=dict(tuning=dict(tile_budget_us=26.0), bwd_weights=1),
                 fp32=dict(tuning=dict(tile_budget_us=26.0, dense_1x1=-1)))
    for f, kw in forms.items():
        assert bool(re.search(r"gm[123] .*(direct| dense mi)", plan_summary(net, **kw))) == (f != "fp32"), f
    engines = {f: PBEngine(net, lr=0.0, momentum=0.0, **kw) for f, kw in forms.items()}
    ref, errs = O.PBOracle(net, lr=0.0, momentum=0.0), {f: [] for f in forms}
    for t in range(2 * S + 4):
        for e in [ref, *engines.values()]:
            e.tick(xs[t % len(ys)], ys[t % len(ys)])
        if t < 2 * S:
            continue
        want = ref.read_velocity()
        for f, e in engines.items():
            got = e.read_velocity().astype(np.float64)
            errs[f].append([np.linalg.norm(got[lo:hi] - want[lo:hi]) / np.linalg.norm(want[lo:hi]) for _, _, lo, hi in weights])
    for f, e in engines.items():
        e.close()
    rms = {f: np.sqrt(np.mean(np.square(v))) for f, v in errs.items()}
    print(f"error of the gradients against float64, split {rms['lanes']:.2e} (weights in their own order {rms['own']:.2e}), fp32 {rms['fp32']:.2e}")
    for f in ("lanes", "own"):
        assert np.max(errs[f]) < 1.5e-6, (f, np.max(errs[f]))
        assert rms[f] <= rms["fp32"], rms


def test_values_that_are_not_finite_stay_so():
    """An infinite input of a layer on the bf16 pipes: whatever the oracle's tick makes infinite or NaN is not finite here."""
    import numpy as np
    from oracle import pb_oracle as O
    from paper_2003_11666_amd import PBEngine
    from paper_2003_11666_amd.binding import plan_summary
    net = W._net("inf", [[W.conv(3, 32, 3, 1, 1)], [W.conv(32, 32, 3, 1, 1)], [W.conv(32, 64, 1, 1, 0)], [W.conv(64, 64, 1, 1, 0)],
                         [W.gn(4, 64), W.relu(), W.gap(), W.linear(64, 5, bias=1), W.ce()]], 3, 12, 12, 5, 1e-3, 0.9, 8, 3, 8)
    tuning, (xs, ys), S = dict(tile_budget_us=26.0), W.sample_pool(net), len(net["stages"])
    plan = plan_summary(net, tuning=tuning)
    assert "gm1" in plan and " split" in plan and " dense mi" in plan, plan
    eng, ref = PBEngine(net, tuning=tuning), O.PBOracle(net)
    for t in range(3 * S):
        x = xs[t % len(ys)].copy()
        if t == S:
            x[1, 5, 6] = np.inf
        for e in (eng, ref):
            e.tick(x, ys[t % len(ys)])
        for k in ("read_weights", "read_velocity", "loss_history"):
            got, want = np.isfinite(getattr(eng, k)()), np.isfinite(np.asarray(getattr(ref, k)()))
            assert np.array_equal(got, want), (t, k, got.sum(), want.sum())
    eng.close()


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
