"""The kernel that keeps a perceptron's parameters in registers (pb_mlp.hip) at the edges of its ranges: two stages, one
workgroup per stage and several, columns per lane 2 to 16, ragged rows and columns, a last stage of several workgroups,
the weight-difference form, samples from the pool in pieces and from the host, and the way to single-step launches and
back."""
import numpy as np
import pytest

import pb_workloads as W
from tests.parity_util import per_tensor_errors, tensor_slices

pytestmark = pytest.mark.gpu


def _net(dims, lr=0.01):
    return W._net("perceptron", W.mlp(dims), dims[0], 1, 1, dims[-1], lr, 0.9, 16, 5, 16)


def _tensors_close(eng, orc, net):
    """Every weight matrix and bias, and its velocity, by itself."""
    slices = tensor_slices(net)
    for k, tol in (("read_weights", 2e-5), ("read_velocity", 1e-3)):
        err = per_tensor_errors(getattr(eng, k)(), getattr(orc, k)(), slices)
        assert err.max() <= tol, (k, slices[int(err.argmax())], err.max())


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
    _tensors_close(a, orc, net)
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
        _tensors_close(a, orc, net)
    a.close()
    b.close()


@pytest.mark.parametrize("dims", [(40, 24, 63), (40, 24, 64), (40, 24, 65), (30, 256, 520, 64), (30, 1024, 129)])
def test_classes_around_a_wavefront_and_messages_around_a_workgroup(dims):
    """Up to 64 classes the softmax keeps a lane's exponential, the other logits it reads again; up to 512 partial gradients
    a thread takes one message, above that up to eight."""
    test_perceptron_follows_the_oracle(dims, "v")


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


def test_beside_a_network_that_runs_one_launch_per_tick():
    """A perceptron of 177 workgroups and a convolution network whose ticks are one launch of 248, both with workgroups
    that wait inside a launch, on two streams: the same bits as one after the other."""
    import torch
    from paper_2003_11666_amd import PBEngine
    nets = [_net((1024,) * 5 + (100,), 1e-5), W.config("small_resnet")]
    pools = [[torch.from_numpy(a).cuda() for a in W.sample_pool(n)] for n in nets]
    streams = [torch.cuda.Stream() for _ in nets]
    torch.cuda.synchronize()

    def run(together):
        engines = []
        for n, s in zip(nets, streams):
            with torch.cuda.stream(s):
                engines.append(PBEngine(n))
        out = []
        for rounds in ([[0, 1]] * 40 if together else [[0]] * 40 + [[1]] * 40):
            for i in rounds:
                engines[i].run_resident(*pools[i], engines[i].ticks, 5)
        for e in engines:
            out += [e.read_weights(), e.read_velocity(), e.loss_history()]
            e.close()
        return out
    for a, b in zip(run(True), run(False)):
        assert np.isfinite(a).all() and np.array_equal(a, b)


def test_beside_another_process():
    """While another process has launches of a wide perceptron under way, this one's ticks run as plain phase launches;
    afterwards they run in registers again.  The weights follow the oracle through both."""
    import subprocess
    import sys
    import torch
    from oracle import pb_oracle as O
    from paper_2003_11666_amd import PBEngine
    root = __file__.rsplit("/tests/", 1)[0]
    other = subprocess.Popen([sys.executable, "-c", f"""
import sys; sys.path.insert(0, {root!r})
import torch, pb_workloads as W
from tests.test_gpu_mlp import _net
from paper_2003_11666_amd import PBEngine
net = _net((1024,) * 5 + (100,), 1e-5)
xs, ys = W.sample_pool(net)
e = PBEngine(net)
for t in range(3): e.tick(xs[t], ys[t])
print('ready', flush=True)
sys.stdin.readline()
e.close()
"""], stdin=subprocess.PIPE, stdout=subprocess.PIPE, text=True)
    try:
        assert other.stdout.readline() == "ready\n"
        net = _net((1024,) * 5 + (100,), 1e-5)
        xs, ys = W.sample_pool(net)
        orc, e = O.PBOracle(net), PBEngine(net)

        def launches_per_tick(n):
            e.profile_begin()
            for t in range(e.ticks, e.ticks + n):
                orc.tick(xs[t % len(ys)], ys[t % len(ys)])
                e.tick(xs[t % len(ys)], ys[t % len(ys)])
            return e.profile_end(0)[0] / n
        assert launches_per_tick(70) > 1           # (asked again in between: refused)
        other.communicate("done\n", timeout=60)
        launches_per_tick(64)
        assert launches_per_tick(6) == 1
        assert _close(e.read_weights(), orc.read_weights()) and _close(e.loss_history(), orc.loss_history())
        e.close()
    finally:
        other.kill()


@pytest.mark.parametrize("form", ["v", "w"])
@pytest.mark.parametrize("dims", [(246, 226, 226, 12), (256, 256, 256, 20), (512,) * 9 + (600,)], ids=str)
def test_launches_of_one_tick_give_the_bits_of_longer_ones(dims, form):
    import torch
    from paper_2003_11666_amd import PBEngine
    net, n = _net(dims, 0.002), 2 * len(dims) + 9
    xs, ys = W.sample_pool(net)
    xd, yd = torch.from_numpy(xs).cuda(), torch.from_numpy(ys).cuda()
    longer, host, pool = (PBEngine(net, lwp_form=form) for _ in range(3))
    longer.run_resident(xd, yd, 3, n)
    for t in range(3, 3 + n):
        host.tick(xs[t % len(ys)], ys[t % len(ys)])
        pool.run_resident(xd, yd, t, 1)
    for k in ("read_weights", "read_velocity", "loss_history"):
        want = getattr(longer, k)()
        assert np.isfinite(want).all() and np.array_equal(getattr(host, k)(), want) and np.array_equal(getattr(pool, k)(), want), k
    for e in (longer, host, pool):
        e.close()
