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
