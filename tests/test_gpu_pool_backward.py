"""Gradients routed back through a max-pool (GroupNorm backward of the stages in front of one) against the oracle: 2x2
windows and overlapping 3x3 windows with padding, maps with odd sides, small maps, a map whose windows' maxima do not fit
in LDS beside it, networks tiled for latency and for throughput."""
import numpy as np
import pytest

import pb_workloads as W
from tests.parity_util import assert_tensors_follow, reference

pytestmark = pytest.mark.gpu


def _stem(hw):       # 7x7 stride-2 stem, 3x3 stride-2 pool with padding 1
    return W._net("stem", W.preact_resnet_bottleneck((1,), 16, 8, n_classes=5), 3, hw, hw, 5, 1e-3, 0.9, 8, 3, 8)


def _vgg(hw):        # 2x2 pools behind two of the layers
    return W._net("pools", W.vgg((8, 16, 16), (0, 2), 4, n_classes=5, in_hw=hw), 3, hw, hw, 5, 1e-3, 0.9, 8, 3, 8)


@pytest.mark.parametrize("tuning", [None, dict(tile_budget_us=14.0)])
@pytest.mark.parametrize("net", [_stem(33), _stem(46), _stem(65), _stem(244), _vgg(9), _vgg(12), _vgg(21), _vgg(32)],
                         ids=lambda n: f"{n['name']}{n['in_h']}")
def test_pool_backward_follows_the_oracle(net, tuning):
    from paper_2003_11666_amd import PBEngine
    (xs, ys), S = W.sample_pool(net), len(net["stages"])
    kw = dict(tuning=tuning) if tuning else {}
    ref, eng = reference(net, (2 * S + 5,))[2 * S + 5], PBEngine(net, **kw)
    for t in range(2 * S + 5):
        eng.tick(xs[t % len(ys)], ys[t % len(ys)])
    for k in ("read_weights", "read_velocity", "loss_history"):
        # 32-bit sums; a window or ReLU decided the other way by the last bit shows in the velocity (2e-3 on the large maps)
        assert np.linalg.norm(getattr(eng, k)() - ref[k]) < (2e-3 if net["in_h"] > 100 else 2e-4) * np.linalg.norm(ref[k]), k
    assert_tensors_follow(eng, ref)
    eng.close()


@pytest.mark.parametrize("widths,pools,hw", [((8, 24, 256), (0, 1), 14), ((32, 40, 512), (0, 1), 14), ((64, 128, 72, 256), (1, 2), 16),
                                             ((16, 16, 1024), (1,), 8), ((32, 40, 512, 20), (0, 1, 2), 15)], ids=str)
def test_pooled_gradients_of_small_maps(widths, pools, hw):
    """A wavefront takes four channels of up to 64 pixels: channels that do not fill the wavefronts, maps of 1 to 64 pixels,
    pooled gradients left in up to four parts by the next stage."""
    net = W._net("pools", W.vgg(widths, pools, 4, n_classes=5, in_hw=hw), 3, hw, hw, 5, 1e-3, 0.9, 8, 3, 8)
    test_pool_backward_follows_the_oracle(net, dict(tile_budget_us=6.0))
