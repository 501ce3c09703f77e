"""The dense layer in front of the loss in networks tiled for throughput: the gradient of the logits worked out by the
backward-data workgroups, weights updated where their gradient arises, against the oracle.  Weight counts that are and are not
multiples of a workgroup's 4096, fewer and more classes than a round of loads (512), GroupNorm in front and none."""
import re

import pytest

import pb_workloads as W
from tests.test_gpu_conv3 import _follow

pytestmark = pytest.mark.gpu


def _basic(classes, c=256, hw=4):
    return W._net("dense_head", W.preact_resnet_basic((c,), 1, 4, in_c=3, n_classes=classes), 3, hw, hw, classes, 1e-3, 0.9, 8, 3, 8)


def _phases(net, **kw):
    from paper_2003_11666_amd.binding import plan_summary
    plan = plan_summary(net, tuning=dict(tile_budget_us=14.0), **kw)
    return {k: int(p) for p, k in re.findall(r"phase (\d+) (ce|fc_bwd_x|fc_bwd_w)\b", plan)}


@pytest.mark.parametrize("net", [_basic(17), _basic(64), _basic(65, 260), _basic(520), _basic(1000, 512, 2)], ids=lambda n: str(n["n_classes"]))
def test_dense_head_follows_the_oracle(net):
    p = _phases(net)
    assert p["fc_bwd_x"] == p["ce"] and p["fc_bwd_w"] == p["ce"] + 1, p
    _follow(net, dict(tile_budget_us=14.0))


@pytest.mark.parametrize("kw", [dict(lwp_form="w"), dict(bwd_weights=1), dict(mitigation=0), dict(update_size=2)], ids=str)
def test_dense_head_with_other_updates(kw):
    net = _basic(40)
    p = _phases(net, **kw)
    assert p["fc_bwd_w"] == p["ce"] + 1 and p["fc_bwd_x"] == p["ce"] + ("update_size" in kw), p
    _follow(net, dict(tile_budget_us=14.0), **kw)


def test_dense_head_without_a_norm_in_front():
    _follow(W._net("dense_head", W.vgg((16, 256), (0, 1), 4, n_classes=33, in_hw=8), 3, 8, 8, 33, 1e-3, 0.9, 8, 3, 8), dict(tile_budget_us=14.0))


@pytest.mark.parametrize("delays", ["larger", "zero"])
def test_dense_head_with_other_delays(delays):
    """Zero delays: the passes of a sample one after the other, the head's backward phases behind all forward ones."""
    from tests.test_gpu_delays import test_delays_in_networks_tiled_for_throughput as follow
    follow(_basic(40), delays, {})


def _without_biases(net):
    return dict(net, stages=[[dict(o, bias=0) for o in st] for st in net["stages"]])


PERCEPTRON = W._net("dense_layers", W.mlp((256, 260, 512, 17)), 256, 1, 1, 17, 1e-2, 0.9, 8, 3, 8)


# (the weight gradient is then the only one of its stage, or the only one that its update waits for)
@pytest.mark.parametrize("kw", [dict(update_size=2), dict(update_size=3, bwd_weights=1), dict(update_size=2, lwp_form="w"), {}], ids=str)
@pytest.mark.parametrize("net", [_basic(40), _basic(40, hw=5), PERCEPTRON], ids=["one-step norm", "two-step norm", "no norm"])
def test_dense_layers_without_a_bias(net, kw):
    _follow(_without_biases(net), dict(tile_budget_us=14.0), **kw)


@pytest.mark.parametrize("kw", [{}, dict(update_size=2)], ids=str)
@pytest.mark.parametrize("delays", ["larger", "zero", "mixed"])
def test_dense_layers_without_a_bias_with_other_delays(delays, kw):
    from tests.test_gpu_delays import test_delays_in_networks_tiled_for_throughput as follow
    for net in (_basic(40), PERCEPTRON):
        follow(_without_biases(net), delays, kw)
