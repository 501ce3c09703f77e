"""The elementwise step of the two-step GroupNorm backward in 16-byte vectors: maps whose channels end inside a vector (1, 2 and 3
elements over), in networks tiled for throughput and in small ones, of one and of several rounds per workgroup; skip gradients."""
import re

import pytest

from tests.test_gpu_conv3 import _follow
from tests.test_gpu_gn_walk import _chain

pytestmark = pytest.mark.gpu

# channels, groups, map, normed stages, tile budget (< 0: small networks' plans), workgroups of a step, options of the run
CASES = [(28, 2, 35, 35, 4, 16.0, 10, {}), (6, 1, 30, 31, 4, -1.0, 6, {}), (10, 2, 33, 35, 4, -1.0, 12, dict(bwd_weights=1)),
         (24, 4, 40, 36, 4, -1.0, 36, {}), (9, 3, 53, 37, 4, -1.0, 18, dict(update_size=2)), (8, 1, 129, 131, 16, -1.0, 34, {}),
         (6, 1, 86, 87, 4, 20.0, 11, {})]


@pytest.mark.parametrize("c,g,h,w,n,budget,tiles,kw", CASES, ids=lambda v: "-".join(map(str, v.values())) if isinstance(v, dict) else str(v))
def test_vectors_over_ends_of_channels_follow_the_oracle(c, g, h, w, n, budget, tiles, kw):
    from paper_2003_11666_amd.binding import plan_summary
    net, tuning = _chain(c, g, h, w, n), dict(tile_budget_us=budget)
    plan = plan_summary(net, tuning=tuning, **kw)
    assert re.search(rf"gnb_apply +tiles +{tiles} .* C{c}x{h}x{w} ", plan), plan
    # (a ReLU decided the other way by the last bit shows in the gradients of 10^4 and more activations a layer)
    _follow(net, tuning, tol=5e-3, **kw)
