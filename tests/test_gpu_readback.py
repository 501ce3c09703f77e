"""Read-back calls at the edges of their three forms (one small kernel into the staging area, chunks of 512 K floats
through the pinned ring, more chunks than the ring has slots): the initial weights, which library and oracle derive
from the seed independently and round to float once, must come back bit for bit; a short destination gets a prefix."""
import ctypes as C

import numpy as np
import pytest

import pb_workloads as W

pytestmark = pytest.mark.gpu


def _net(dims):
    return W._net("readback", W.mlp(dims), dims[0], 1, 1, dims[-1], 0.01, 0.9, 16, 5, 16)


@pytest.mark.parametrize("dims", [(5, 7, 4), (512, 1000, 10), (512, 1022, 10), (1024, 1024, 10), (2048, 2300, 12)])
def test_initial_weights_come_back_exactly(dims):
    from oracle import pb_oracle as O
    from paper_2003_11666_amd import PBEngine
    net = _net(dims)
    want = O.PBOracle(net).read_weights().astype(np.float32)
    e = PBEngine(net)
    assert np.array_equal(e.read_weights(), want)
    assert not e.read_velocity().any()
    for cap in {1, min(1023, len(want) - 1), len(want) - 1}:
        out = np.full(cap + 8, -7.0, dtype=np.float32)
        assert e.lib.pb_read_weights(e.ctx, out.ctypes.data, C.c_int64(cap)) == cap
        assert np.array_equal(out[:cap], want[:cap]) and np.all(out[cap:] == -7.0)
    e.close()


@pytest.mark.parametrize("capacity,ticks", [(7, 5), (7, 12), (8, 31), (64, 40)])
def test_loss_ring_wraps(capacity, ticks):
    from paper_2003_11666_amd import PBEngine
    net = W.config("tiny_mlp")
    xs, ys = W.sample_pool(net)
    a, b = PBEngine(net, loss_capacity=capacity), PBEngine(net)
    for t in range(ticks):
        for e in (a, b):
            e.tick(xs[t % len(ys)], ys[t % len(ys)])
    got, full = a.loss_history(), b.loss_history()
    assert len(full) == ticks - len(net["stages"]) + 1
    assert np.array_equal(got, full[-capacity:])
    a.close()
    b.close()
