"""The kernel that keeps a perceptron's parameters in registers (pb_mlp.hip) at the edges of its ranges: two stages, one
workgroup per stage and several, columns per lane 2 to 16, ragged rows and columns, a last stage of several workgroups,
the weight-difference form, samples from the pool in pieces and from the host, and the way to single-step launches and
back."""
import numpy as np
import pytest

import pb_workloads as W

pytestmark = pytest.mark.gpu


def _net(dims, lr=0.01):
    return W._net("perceptron", W.mlp(dims), dims[0], 1, 1, dims[-1], lr, 0.9, 16, 5, 16)


def _close(a, b, tol=2e-5):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return np.abs(a - b).max() <= tol * max(np.abs(b).max(), 1e-3)


@pytest.mark.parametrize("dims,form", [((5, 7, 4), "v"), ((5, 7, 6, 4), "w"), ((64, 128, 128, 128, 10), "v"), ((129, 65, 33), "v"),
                                       ((300, 257, 513, 40), "w"), ((1024, 1023, 100), "v"), ((100, 1024, 10), "w"),
                                       ((17,) + (25,) * 10 + (3,), "v"), ((1024,) * 5 + (100,), "v")])
def test_perceptron_follows_the_oracle(dims, form):
    import torch
    from oracle import pb_oracle as O
    from paper_2003_11666_amd import PBEngine
    net = _net(dims, 0.002)
    S, (xs, ys) = len(dims) - 1, W.sample_pool(net)
    orc, a, b = O.PBOracle(net, lwp_form=form), PBEngine(net, lwp_form=form), PBEngine(net, lwp_form=form)
    xd, yd = torch.from_numpy(xs).cuda(), torch.from_numpy(ys).cuda()
    at = 0
    for n in (1, 2, S - 1, 2 * S + 3, 1, 7):
        a.run_resident(xd, yd, at, n)
        for t in range(at, at + n):
            orc.tick(xs[t % len(ys)], ys[t % len(ys)])
            b.tick(xs[t % len(ys)], ys[t % len(ys)])
        at += n
    assert _close(a.read_weights(), orc.read_weights()) and _close(a.loss_history(), orc.loss_history())
    assert _close(a.read_velocity(), orc.read_velocity(), 1e-3)
    for k in ("read_weights", "read_velocity", "loss_history"):
        assert np.array_equal(getattr(a, k)(), getattr(b, k)())
    # single-step launches of the phase kernel take over and hand back
    for mode in (1, 0):
        a.set_launch_mode(mode)
        a.run_resident(xd, yd, at, 5)
        for t in range(at, at + 5):
            orc.tick(xs[t % len(ys)], ys[t % len(ys)])
        at += 5
        assert _close(a.read_weights(), orc.read_weights()) and _close(a.loss_history(), orc.loss_history())
    a.close()
    b.close()


def test_contexts_that_do_not_fit_the_gpu_together_take_turns():
    """Two contexts of 177 workgroups on two streams: launches of one wait for the other's."""
    import torch
    from paper_2003_11666_amd import PBEngine
    net = _net((1024,) * 5 + (100,), 0.002)
    xs, ys = W.sample_pool(net)
    xd, yd = torch.from_numpy(xs).cuda(), torch.from_numpy(ys).cuda()
    torch.cuda.synchronize()
    engines = []
    for _ in range(2):
        with torch.cuda.stream(torch.cuda.Stream()):
            engines.append(PBEngine(net))
    for i in range(4):
        for e in engines:
            e.run_resident(xd, yd, 8 * i, 8)
    a, b = (e.read_weights() for e in engines)
    assert np.array_equal(a, b)
    for e in engines:
        e.close()
