"""Updates that the planner moves to other launches than the first one they could run in, or ahead of the step that reads the
weights where a stage keeps two copies of them (spread_steps; plans of the library's own, no tile budget asked for): weight
stashing, the other form of the weight prediction, plain momentum, larger delays, odd and even numbers of ticks."""
import numpy as np
import pytest

import pb_workloads as W
from tests.test_gpu_conv3 import _follow
from tests.test_moved_update_plans import moved_updates

pytestmark = pytest.mark.gpu

CHAIN = W._net("chain", [[W.conv(3, 48, 3, 1, 1)]] + [[W.gn(4, 48), W.relu(), W.conv(48, 48, 3, 1, 1)] for _ in range(3)] +
               [[W.gn(4, 48), W.relu(), W.gap(), W.linear(48, 5, bias=1), W.ce()]], 3, 40, 40, 5, 1e-3, 0.9, 8, 3, 8)
# (its first 512-channel layer's update runs a launch ahead of the step that reads the weights; without stashing, which has one copy)
VGG = W._net("vgg", W.vgg((64, 128, 256, 512, 512), (0, 1, 2), 8, n_classes=10, in_hw=32), 3, 32, 32, 10, 1e-3, 0.9, 8, 3, 8)
CASES = [(CHAIN, kw) for kw in ({}, dict(bwd_weights=1), dict(lwp_form="w"), dict(mitigation=0))] + \
        [(VGG, kw) for kw in ({}, dict(lwp_form="w"), dict(mitigation=0))]


@pytest.mark.parametrize("net,kw", CASES, ids=lambda v: v.get("name") or "-".join(map(str, v.values())) or "default")
def test_moved_updates_follow_the_oracle(net, kw):
    assert moved_updates(net, **kw)
    # (a ReLU or a pooling window decided the other way by the last bit shows in the gradients of 100 000 activations and more)
    _follow(net, None, tol=2e-3, **kw)


@pytest.mark.parametrize("kw", [{}, dict(lwp_form="w")], ids=str)
@pytest.mark.parametrize("net", [CHAIN, VGG], ids=lambda n: n["name"])
def test_moved_updates_with_larger_delays(net, kw):
    from oracle import pb_oracle as O
    from paper_2003_11666_amd import PBEngine
    assert moved_updates(net, **kw)                    # (delays change the rings, not the launches)
    (xs, ys), S = W.sample_pool(net), len(net["stages"])
    dl, K = [2 * (S - 1 - s) + (0, 3, 1)[s % 3] for s in range(S)], 2 * S + 7
    eng = PBEngine(net, delays=dl, **kw)
    for t in range(K):
        eng.tick(xs[t % len(ys)], ys[t % len(ys)])
    w, v, losses = eng.read_weights().astype(np.float64), eng.read_velocity().astype(np.float64), eng.loss_history()
    eng.close()
    hist, want = O.run_sample_indexed(net, K, xs, ys, delays=dl, mitigation=3, **kw)
    assert np.allclose(losses, np.asarray(want[:len(losses)]), rtol=1e-4, atol=1e-4)
    off = 0
    for s, st in enumerate(net["stages"]):
        params, velocity = hist[s][K - 2 * (S - 1) + s]
        for name, shape, _ in O.stage_param_specs(st):
            n = int(np.prod(shape))
            for got, ref, tol in ((w, params, 1e-5), (v, velocity, 2e-3)):     # (the velocity: a ReLU decided the other way, as above)
                ref = ref[name].numpy().reshape(-1)
                err = np.linalg.norm(got[off:off + n] - ref) / np.linalg.norm(ref)
                assert err <= tol, (s, name, err)
            off += n
    assert off == w.size
