"""Channel sums of the two-step GroupNorm backward on maps of 260 to 1020 pixels, where a wavefront takes a channel:
the smallest and largest map of the range, channel counts that leave wavefronts without one, maps just outside it."""
import numpy as np
import pytest

import pb_workloads as W
from tests.parity_util import assert_tensors_follow, reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nt", [0, 1])       # (1: the other kernel instantiation asked for, where the plan allows it)
@pytest.mark.parametrize("hw,width,groups", [(18, 32, 2), (22, 44, 2), (28, 30, 3), (32, 24, 4), (30, 36, 2), (17, 32, 2), (34, 16, 2)])
def test_channel_sums_follow_the_oracle(hw, width, groups, nt):
    from paper_2003_11666_amd import PBEngine
    net = W._net("channels", W.preact_resnet_basic((width,), 1, groups, in_c=3, n_classes=5), 3, hw, hw, 5, 1e-3, 0.9, 8, 3, 8)
    (xs, ys), S = W.sample_pool(net), len(net["stages"])
    ref, eng = reference(net, (2 * S + 5,))[2 * S + 5], PBEngine(net, tuning=dict(tile_budget_us=14.0, nt_stores=nt))
    for t in range(2 * S + 5):
        eng.tick(xs[t % len(ys)], ys[t % len(ys)])
    for k in ("read_weights", "read_velocity", "loss_history"):
        # 32-bit sums of up to 1156 terms; a ReLU decided the other way by the last bit shows in the velocity
        assert np.linalg.norm(getattr(eng, k)() - ref[k]) < 2e-4 * np.linalg.norm(ref[k]), k
    assert_tensors_follow(eng, ref)
    eng.close()
