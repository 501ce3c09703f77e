"""In which launch of a tick updates run: behind everything that writes gradients of their stage, and in large networks not all
in the first one they could."""
import re

import pytest

import pb_workloads as W


def _steps(net):
    from paper_2003_11666_amd.binding import plan_summary
    return [(int(m[1]), int(m[2]), m[3], l) for l in plan_summary(net).splitlines() for m in [re.match(r"stage +(\d+) phase (\d+) (\w+)", l)]]


@pytest.mark.parametrize("net", [W.config("vgg11"), W.config("resnet50"), W.config("wide"),
                                 W._net("r50", W.preact_resnet_bottleneck(), 3, 64, 64, 1000, 1e-3, 0.9, 8, 3, 8)], ids=["vgg11", "resnet50", "wide", "resnet50_64"])
def test_updates_run_behind_their_gradients(net):
    steps, last, moved = _steps(net), {}, 0
    for s, p, kind, l in steps:
        if kind in ("gnb_reduce", "gn_bwd", "head", "head_fc", "bias_grad", "conv_bwd_w") or (kind == "gemm" and "gm3" in l) or (kind == "fc_bwd_x"):
            own = kind == "gemm" and any(k == "gemm" and "gm2" in m and t == s and q < p for t, q, k, m in steps)
            if not own:      # (weight-gradient tiles a phase behind backward data update their weights themselves)
                last[s] = max(last.get(s, 0), p)
    for s, p, kind, l in steps:
        if kind == "update":
            assert p > last.get(s, -1) or any(k == "gn_bwd" and t == s and q == p for t, q, k, _ in steps), l
            moved += p > last.get(s, 0) + 1
    big = [p for s, p, kind, l in steps if kind == "update" and int(re.search(r"tiles +(\d+)", l)[1]) >= 128]
    assert len(set(big)) > 1 or not big, "one launch holds every large update"
