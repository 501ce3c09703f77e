"""GroupNorm backward of a group that one workgroup walks twice: maps of no multiple of 4 pixels from one pixel to several
1024-element rounds per channel, channels that leave quarter-wavefronts without one, groups up to the largest, maps of a multiple
of 4 pixels beyond a workgroup's registers, more channels than a workgroup has threads; skip gradients, and a head's pooled ones."""
import re

import pytest

import pb_workloads as W
from tests.test_gpu_conv3 import _follow

pytestmark = pytest.mark.gpu


def _chain(c, g, h, w, n=4, skip=True):
    st = [[W.conv(3, c, 1, 1, 0)]] + [[W.gn(g, c), W.relu(), W.conv(c, c, 1, 1, 0)] for _ in range(n)]
    if skip:
        st[3].append(W.add(2, c, c, 1, 0))
    return W._net("walk", st + [[W.gn(g, c), W.relu(), W.gap(), W.linear(c, 5, bias=1), W.ce()]], 3, h, w, 5, 1e-3, 0.9, 8, 3, 8)


# channels, groups, map, tile budget (< 0: small networks' plans), options of the run
CASES = [(20, 2, 1, 1, -1.0, {}), (18, 2, 3, 5, -1.0, {}), (12, 3, 15, 17, -1.0, dict(bwd_weights=1)), (9, 3, 17, 17, -1.0, {}),
         (20, 1, 16, 16, -1.0, {}), (300, 1, 3, 3, -1.0, dict(update_size=2, lwp_form="w")), (2, 1, 50, 51, -1.0, {}),
         (20, 4, 35, 35, 36.0, {}), (64, 4, 5, 5, 36.0, dict(update_size=2)), (24, 4, 21, 13, 36.0, dict(bwd_weights=1)),
         (32, 4, 63, 65, 40.0, {}),
         (1028, 4, 3, 3, -1.0, {}), (54, 18, 19, 17, -1.0, {})]


@pytest.mark.parametrize("c,g,h,w,budget,kw", CASES, ids=lambda v: "-".join(map(str, v.values())) if isinstance(v, dict) else str(v))
def test_walked_groups_follow_the_oracle(c, g, h, w, budget, kw):
    from paper_2003_11666_amd.binding import plan_summary
    net, tuning = _chain(c, g, h, w), dict(tile_budget_us=budget)
    plan = plan_summary(net, tuning=tuning, **kw)
    # (a step of the register form has a map of a multiple of 4 pixels and at most 4096 elements in a group)
    assert (h * w) % 4 or c // g * h * w > 4096
    assert re.search(rf"gn_bwd +tiles +{g} .* C{c}x{h}x{w} ", plan), plan
    # 32-bit sums of up to 32760 terms; a ReLU decided the other way by the last bit shows in the velocity, of the order of one over
    # the root of the activations, and among 10^4 of them a few stand within rounding of zero (24 channels of 21x13 pixels: one
    # moves it by 2.1e-4 at tick 6, by 8.4e-4 a tick on, with the two-step form by the same)
    _follow(net, tuning, tol=5e-3 if c * h * w > 5000 else 2e-4, **kw)
