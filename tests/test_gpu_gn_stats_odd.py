"""GroupNorm statistics of groups that no workgroup holds in whole vectors: every remainder of 4, one and several batches of
requests, groups that fit LDS and groups that do not, beyond 32768 elements too."""
import pytest

import pb_workloads as W
from tests.test_gpu_conv3 import _follow

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tuning", [{}, dict(tile_budget_us=14.0)], ids=["latency", "throughput"])
@pytest.mark.parametrize("hw,width,groups", [(5, 6, 2), (5, 5, 1), (7, 10, 2), (29, 30, 2), (31, 36, 2), (33, 36, 2), (32, 64, 1), (41, 20, 1)])
def test_statistics_follow_the_oracle(hw, width, groups, tuning):
    net = W._net("oddstats", W.preact_resnet_basic((width,), 1, groups, in_c=3, n_classes=5), 3, hw, hw, 5, 1e-3, 0.9, 8, 3, 8)
    # (a ReLU decided the other way by the last bit shows in the gradients of up to 200 000 activations)
    _follow(net, tuning, tol=2e-3)
