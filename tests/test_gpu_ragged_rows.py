"""GEMM tiles on maps whose rows are no multiple of 4 floats, and on weight rows and gradient segments that are none: every
remainder, 1x1 to 7x7 kernels of stride 1 and 2, reductions in one and several chunks, both tilings, all three passes."""
import pytest

import pb_workloads as W
from tests.test_gpu_conv3 import _follow

pytestmark = pytest.mark.gpu


def _net(stages, h, w):
    return W._net("ragged", stages, 3, h, w, 5, 1e-3, 0.9, 8, 3, 8)


def _plain(c1, c2, k, s, h, w, mid=2):
    st = [[W.conv(3, c1, k, 1, k // 2)], [W.gn(1, c1), W.relu(), W.conv(c1, c2, k, s, k // 2)]]
    st += [[W.gn(1, c2), W.relu(), W.conv(c2, c2, 3, 1, 1)] for _ in range(mid)]
    return _net(st + [[W.gn(1, c2), W.relu(), W.gap(), W.linear(c2, 5, bias=1), W.ce()]], h, w)


@pytest.mark.parametrize("tuning", [{}, dict(tile_budget_us=14.0, dense_1x1=-1)], ids=["latency", "throughput"])
@pytest.mark.parametrize("net", [_plain(5, 7, 3, 1, 5, 5), _plain(6, 10, 3, 2, 7, 9), _plain(7, 9, 1, 1, 6, 7), _plain(12, 20, 3, 1, 13, 14), _plain(9, 18, 5, 2, 11, 6),
                                 _plain(33, 35, 3, 1, 9, 11), _plain(64, 65, 3, 1, 17, 15), _plain(10, 30, 1, 2, 10, 10), _plain(3, 130, 3, 1, 3, 3),
                                 _plain(16, 24, 3, 1, 41, 43, mid=1), _plain(4, 4, 3, 1, 1, 1)],
                         ids=lambda n: f"{n['stages'][1][2]['cin']}-{n['stages'][1][2]['cout']}-k{n['stages'][1][2]['k']}s{n['stages'][1][2]['stride']}-{n['in_h']}x{n['in_w']}")
def test_ragged_rows_follow_the_oracle(net, tuning):
    _follow(net, tuning, tol=5e-4)


@pytest.mark.parametrize("hw", [41, 42, 43])
def test_ragged_stems_and_pools_follow_the_oracle(hw):
    net = W._net("raggedstem", W.preact_resnet_bottleneck((1, 1), 16, 4, n_classes=5), 3, hw, hw, 5, 1e-3, 0.9, 8, 3, 8)
    # (a ReLU or a pooling window decided the other way by the last bit shows in the gradients of 200 000 activations)
    for tuning in ({}, dict(tile_budget_us=14.0)):
        _follow(net, tuning, tol=2e-3)


@pytest.mark.parametrize("tuning", [{}, dict(tile_budget_us=14.0)], ids=["latency", "throughput"])
@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("hw,c", [(5, 5), (6, 9), (7, 16), (8, 6), (12, 20), (33, 18)])
def test_projections_beside_a_layer_behind_a_relu_follow_the_oracle(hw, c, stride, tuning):
    st = [[W.conv(3, c, 3, 1, 1)], [W.relu(), W.conv(c, 2 * c + 1, 3, stride, 1)],
          [W.relu(), W.conv(2 * c + 1, 2 * c + 1, 3, 1, 1), W.add(1, c, 2 * c + 1, stride, 1)],
          [W.gn(1, 2 * c + 1), W.relu(), W.gap(), W.linear(2 * c + 1, 5, bias=1), W.ce()]]
    _follow(_net(st, hw, hw), tuning, tol=5e-4)


@pytest.mark.parametrize("tuning", [{}, dict(tile_budget_us=14.0)], ids=["latency", "throughput"])
@pytest.mark.parametrize("net", [_plain(192, 200, 3, 1, 1, 1), _plain(130, 192, 3, 2, 2, 1), _plain(192, 96, 3, 1, 5, 1), _plain(70, 200, 5, 1, 1, 1)],
                         ids=["1x1", "stride", "5x1", "k5"])
def test_rows_of_one_pixel_in_several_chunks_follow_the_oracle(net, tuning):
    _follow(net, tuning, tol=5e-4)
