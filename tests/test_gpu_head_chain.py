"""Last stages behind a global average pool that do not run as one workgroup: statistics with the pool (K_GAP_STATS: channels of
one to 16 and of more elements, groups in LDS and beyond it, of no multiple of 4), the dense layer, the loss and both backward
passes in one workgroup (K_HEAD_FC: one to 256 rows of threads, up to its limit), the channels' sums taken by it, by the dense
backward step of networks tiled for throughput, and by the one-step GroupNorm backward."""
import re

import pytest

import pb_workloads as W
from tests.test_gpu_conv3 import _follow

pytestmark = pytest.mark.gpu
THR = dict(tile_budget_us=14.0)


def _net(c, g, k, hw, relu=True, dtype="fp32", bias=1):
    act = [W.relu()] if relu else []
    st = [[W.conv(3, c, 1, 1, 0)], [W.gn(g, c), W.relu(), W.conv(c, c, 1, 1, 0)], [W.gn(g, c), *act, W.gap(), W.linear(c, k, bias=bias), W.ce()]]
    return W._net("headchain", st, 3, hw, hw, k, 1e-3, 0.9, 8, 3, 8, act_dtype=dtype)


def _kinds(net, tuning, **kw):
    from paper_2003_11666_amd.binding import plan_summary
    return re.findall(rf"stage +{len(net['stages']) - 1} phase (\d+) (\w+)", plan_summary(net, tuning=tuning, **kw))


@pytest.mark.parametrize("tuning", [{}, THR], ids=["latency", "throughput"])
@pytest.mark.parametrize("c,g,k,hw", [(4, 1, 17, 4), (12, 3, 63, 6), (36, 2, 100, 9), (40, 2, 5, 7), (64, 4, 512, 2), (256, 8, 128, 3),
                                      (1024, 32, 32, 1), (1024, 32, 32, 2), (520, 4, 63, 2), (20, 1, 33, 33), (36, 2, 20, 33)])
def test_dense_head_in_one_workgroup(c, g, k, hw, tuning):
    net = _net(c, g, k, hw)
    kinds = _kinds(net, tuning)
    head = "fc_fwd" if tuning and c >= 256 else "head_fc"
    assert ("0", "gap_stats") in kinds and ("1", head) in kinds and not [x for x in kinds if x[1] in ("gap_fwd", "gnb_reduce")], kinds
    _follow(net, tuning, tol=2e-4)


@pytest.mark.parametrize("kw", [dict(bwd_weights=1), dict(update_size=3), dict(mitigation=0), dict(lwp_form="w")], ids=str)
@pytest.mark.parametrize("hw", [5, 6])       # two-step and one-step GroupNorm backward
def test_dense_head_with_other_updates(hw, kw):
    _follow(_net(24, 2, 30, hw), {}, **kw)


@pytest.mark.parametrize("delays", ["larger", "zero", "mixed"])
@pytest.mark.parametrize("c,k,hw", [(24, 30, 5), (24, 30, 6), (256, 129, 5)])
def test_head_chain_with_other_delays(c, k, hw, delays):
    from tests import test_gpu_delays
    test_gpu_delays.test_delays_in_networks_tiled_for_throughput(_net(c, 2, k, hw), delays, {})


def test_without_a_relu_and_without_a_bias():
    _follow(_net(24, 2, 30, 5, relu=False), {})
    _follow(_net(24, 2, 30, 5, bias=0), {})


# beyond the one workgroup's weights
@pytest.mark.parametrize("c,g,k,hw", [(256, 8, 129, 5), (256, 8, 129, 4), (260, 4, 300, 3), (1028, 4, 33, 3)])
@pytest.mark.parametrize("kw", [{}, dict(bwd_weights=1), dict(update_size=2)], ids=str)
def test_large_dense_heads(c, g, k, hw, kw):
    net = _net(c, g, k, hw)
    kinds = _kinds(net, THR, **kw)
    assert ("0", "gap_stats") in kinds and ("1", "fc_fwd") in kinds and not [x for x in kinds if x[1] in ("gap_fwd", "gnb_reduce")], kinds
    _follow(net, THR, tol=2e-4, **kw)
    _follow(net, {}, tol=2e-4, **kw)         # (tiled for latency: the pool in the statistics, matrix-core tiles for the layer)


def test_head_chain_with_bf16_activations():
    from tests.parity_util import reference
    import numpy as np
    from paper_2003_11666_amd import PBEngine
    for c, k in ((24, 30), (256, 129)):
        net = _net(c, 2, k, 5, dtype="bf16")
        (xs, ys), n = W.sample_pool(net), 12
        ref, eng = reference(net, (n,))[n], PBEngine(net, tuning=THR)
        for t in range(n):
            eng.tick(xs[t % len(ys)], ys[t % len(ys)])
        # a rounding decided the other way is half a unit in 2^8 of one activation
        assert np.linalg.norm(eng.read_weights() - ref["read_weights"]) < 1e-4 * np.linalg.norm(ref["read_weights"])
        assert np.linalg.norm(eng.loss_history() - ref["loss_history"]) < 1e-3 * np.linalg.norm(ref["loss_history"])
        eng.close()
