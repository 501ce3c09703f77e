"""Networks tiled for throughput with delays other than the pipeline's own: larger ones (deeper rings of predicted weights)
and smaller ones (the sample-indexed form, whose steps run stage after stage), against the oracle's sample-indexed form.
Direct and dense tiles with the update inside, dot-product layers whose update computes the weight gradient (VGG layers
on 4x4 maps), pooled gradients; updates every sample and every two, both forms of the weight prediction."""
import numpy as np
import pytest

import pb_workloads as W

pytestmark = pytest.mark.gpu


def _net(name, stages, hw):
    return W._net(name, stages, 3, hw, hw, 5, 1e-3, 0.9, 8, 3, 8)


NETS = [_net("basic8", W.preact_resnet_basic((32, 64), 1, 4, in_c=3, n_classes=5), 8),
        _net("basic20", W.preact_resnet_basic((48, 80), 1, 4, in_c=3, n_classes=5), 20),
        _net("bottleneck24", W.preact_resnet_bottleneck((1, 1), 64, 16, n_classes=5), 24),
        _net("vgg21", W.vgg((8, 16, 16), (0, 2), 4, n_classes=5, in_hw=21), 21),
        _net("vgg16", W.vgg((64, 256, 256), (0, 1), 8, n_classes=5, in_hw=16), 16)]


@pytest.mark.parametrize("kw", [dict(), dict(update_size=2), dict(lwp_form="w")], ids=str)
@pytest.mark.parametrize("delays", ["larger", "zero", "mixed"])
@pytest.mark.parametrize("net", NETS, ids=lambda n: n["name"])
def test_delays_in_networks_tiled_for_throughput(net, delays, kw):
    from oracle import pb_oracle as O
    from paper_2003_11666_amd import PBEngine
    (xs, ys), S, r = W.sample_pool(net), len(net["stages"]), np.random.default_rng(1)
    own = [2 * (S - 1 - s) for s in range(S)]
    dl = {"larger": [n + int(r.integers(0, 6)) for n in own], "zero": [0] * S, "mixed": [int(r.integers(0, 5)) for _ in own]}[delays]
    sequential, K, N = any(a < b for a, b in zip(dl, own)), 2 * S + 6, kw.get("update_size", 1)
    eng = PBEngine(net, delays=dl, tuning=dict(tile_budget_us=14.0), **kw)
    for t in range(K):
        eng.tick(xs[t % len(ys)], ys[t % len(ys)])
    w, v, losses = eng.read_weights().astype(np.float64), eng.read_velocity().astype(np.float64), eng.loss_history()
    eng.close()
    hist, want = O.run_sample_indexed(net, K, xs, ys, delays=dl, mitigation=3, **kw)
    assert len(losses) == (K if sequential else K - S + 1)
    assert np.allclose(losses, np.asarray(want[:len(losses)]), rtol=1e-4, atol=1e-4)
    off = 0
    for s, st in enumerate(net["stages"]):
        params, velocity = hist[s][(K if sequential else K - 2 * (S - 1) + s) // N]
        for name, shape, _ in O.stage_param_specs(st):
            n = int(np.prod(shape))
            for got, ref, tol in ((w, params, 1e-5), (v, velocity, 1e-4)):     # (the parity tests' bounds; no decision flips here)
                ref = ref[name].numpy().reshape(-1)
                assert np.linalg.norm(got[off:off + n] - ref) <= tol * np.linalg.norm(ref), (s, name, tol)
            off += n
    assert off == w.size
