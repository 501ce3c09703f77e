"""The two-step GroupNorm backward where its passes are more than the chip has places for: elementwise workgroups of two and four
rounds (the last one of a group shorter), channel sums with a wavefront per channel on maps of 1024 to 4096 pixels, channel
counts that leave wavefronts without one; skip gradients and none."""
import re

import pytest

import pb_workloads as W
from tests.test_gpu_conv3 import _follow

pytestmark = pytest.mark.gpu


def _chain(c, g, n, hw):
    st = [[W.conv(3, c, 1, 1, 0)]] + [[W.gn(g, c), W.relu(), W.conv(c, c, 1, 1, 0)] for _ in range(n)]
    st[3].append(W.add(2, c, c, 1, 0))
    return W._net("rounds", st + [[W.gn(g, c), W.relu(), W.gap(), W.linear(c, 5, bias=1), W.ce()]], 3, hw, hw, 5, 1e-3, 0.9, 8, 3, 8)


@pytest.mark.parametrize("c,g,n,hw,reduce,apply", [(130, 2, 8, 34, 33, 38), (129, 3, 8, 64, 33, 129), (64, 2, 7, 126, 64, 126), (32, 2, 26, 128, 32, 32)])
def test_many_rounds_follow_the_oracle(c, g, n, hw, reduce, apply):
    from paper_2003_11666_amd.binding import plan_summary
    net, tuning = _chain(c, g, n, hw), dict(tile_budget_us=14.0)
    plan = plan_summary(net, tuning=tuning)
    tiles = {k: {int(x) for x in re.findall(rf"{k} +tiles +(\d+) ", plan)} for k in ("gnb_reduce", "gnb_apply")}
    assert reduce in tiles["gnb_reduce"] and apply in tiles["gnb_apply"], tiles
    # (a ReLU decided the other way by the last bit shows in the gradients of millions of activations)
    _follow(net, tuning, tol=5e-3)
