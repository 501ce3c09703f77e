"""Updates in other launches than the planner's first choice: which networks have them, and that none runs ahead of a gradient of its
stage, whichever step writes it."""
import re

import pytest

import pb_workloads as W


def _steps(net, **kw):
    from paper_2003_11666_amd.binding import plan_summary
    return [(int(m[1]), int(m[2]), m[3], l) for l in plan_summary(net, **kw).splitlines() for m in [re.match(r"stage +(\d+) phase (\d+) (\w+)", l)]]


def _last_gradients(steps):
    """Per stage: the launch of the last step that writes a gradient its update reads."""
    last = {}
    for s, p, kind, l in steps:
        if kind in ("gnb_reduce", "gn_bwd", "head", "head_fc", "bias_grad", "conv_bwd_w", "fc_bwd_x", "ce") or (kind == "gemm" and "gm3" in l):
            own = kind == "gemm" and any(k == "gemm" and "gm2" in m and t == s and q < p for t, q, k, m in steps)
            if not own:      # (weight-gradient tiles a phase behind backward data update their weights themselves)
                last[s] = max(last.get(s, 0), p)
    return last


def moved_updates(net, **kw):
    """Updates in another launch than the planner's first choice: behind everything that writes gradients of their stage or, where
    they work out the gradient themselves, with the step that reads the weights (one copy of them: behind it)."""
    steps = _steps(net, **kw)
    last = _last_gradients(steps)
    readers = {s: p for s, p, kind, l in steps if kind == "dot_bwd_x" or (kind == "gemm" and "gm2" in l)}
    return [l for s, p, kind, l in steps if kind == "update" and
            (p > last.get(s, -1) + 1 if " K0x0x0 " in l else not 0 <= p - readers[s] <= 1)]


NETS = {"vgg11": W.config("vgg11"), "resnet50": W.config("resnet50"), "wide": W.config("wide"),
        "resnet50_64": W._net("r50", W.preact_resnet_bottleneck(), 3, 64, 64, 1000, 1e-3, 0.9, 8, 3, 8)}


@pytest.mark.parametrize("name", NETS)
def test_large_updates_move_where_launches_get_shorter(name):
    net = NETS[name]
    steps = _steps(net)
    last = _last_gradients(steps)
    for s, p, kind, l in steps:
        if kind == "update":
            assert p > last.get(s, -1) or any(k == "gn_bwd" and t == s and q == p for t, q, k, _ in steps), l
    # (the other two: no launch gets shorter by it)
    assert bool(moved_updates(net)) == (name in ("vgg11", "resnet50_64"))


def _mlp(*dims):
    return W._net("dense", W.mlp(dims), dims[0], 1, 1, dims[-1], 1e-2, 0.9, 8, 3, 8)


@pytest.mark.parametrize("kw", [dict(update_size=2), dict(update_size=2, bwd_weights=1), dict(update_size=2, lwp_form="w")], ids=str)
@pytest.mark.parametrize("net", [W._net("basic", W.preact_resnet_basic((256,), 1, 4, n_classes=40), 3, 4, 4, 40, 1e-3, 0.9, 8, 3, 8),
                                 _mlp(256, 260, 512, 17), _mlp(1024, 5)], ids=["basic", "mlp", "one-layer"])
def test_updates_wait_for_dense_layers_without_a_bias(net, kw):
    """No other step of such a stage need write a gradient that its update waits for."""
    from paper_2003_11666_amd.binding import plan_summary
    net = dict(net, stages=[[dict(o, bias=0) for o in st] for st in net["stages"]])
    steps = re.findall(r"stage +(\d+) phase (\d+) (\w+)", plan_summary(net, tuning=dict(tile_budget_us=14.0), **kw))
    dense = {s: int(p) for s, p, kind in steps if kind == "fc_bwd_w"}
    assert dense, steps
    for s, p, kind in steps:
        assert kind != "update" or int(p) > dense.get(s, -1), steps


def test_a_plan_whose_update_runs_ahead_of_its_gradients_is_refused(tmp_path):
    """The audit of the step table, on a planner that puts every update into the tick's first launch."""
    from tests import host_stub
    path = host_stub.build(str(tmp_path / "early.so"), {"out.push_back({last_grad_phase + 1, e});": "out.push_back({0, e});"})
    host_stub.run(path, """
try:
    engine(W.config('small_resnet'))
except B.PBError as e:
    assert 'ahead of its gradients' in str(e), e
else:
    raise AssertionError('accepted')
""")
