"""GroupNorm scale and shift updated inside the GroupNorm backward step, at update sizes above one and with weight stashing,
against the oracle: groups of few channels (old values requested ahead of the sums) and of more than 64 (behind them),
through the first updates and the ticks before the first gradient."""
import pytest

import pb_workloads as W
from tests.test_gpu_conv3 import _follow

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [dict(update_size=3), dict(bwd_weights=1), dict(update_size=2, bwd_weights=1), dict(update_size=2, lwp_form="w"), dict()], ids=str)
@pytest.mark.parametrize("widths,hw,groups", [((16, 32), 8, 4), ((96,), 6, 1)])
def test_scale_and_shift_follow_the_oracle(widths, hw, groups, kw):
    from paper_2003_11666_amd.binding import plan_summary
    net = W._net("gn", W.preact_resnet_basic(widths, 1, groups, in_c=3, n_classes=5), 3, hw, hw, 5, 1e-3, 0.9, 8, 3, 8)
    phases = {l.split("phase")[1].split()[0] for l in plan_summary(net, **kw).splitlines() if " phase " in l}
    assert phases == {"0", "1"}, phases
    _follow(net, None, **kw)
