"""The work that users of the pipeline-tick engine have it do, as measurable cases.

A pass of a training case is one logging interval: `ticks` pipeline ticks fed from a pool resident on the GPU
(PBEngine.run_resident) or sample by sample from host memory (PBEngine.tick), then what a training program takes at the
end of the interval: the losses of the interval, the weights and the velocity (a checkpoint).  A pass of an "update" case
is one fused optimizer step over flat device arrays (update_standalone).

Learning rate and momentum are those of a training run after its last decay, values for batches of 128 scaled to one
sample per update as the paper does (scale_hyperparameters).  The networks are the benchmark configurations of
pb_workloads and other sizes of the same four families (multilayer perceptron, VGG, ResNet with basic blocks, ResNet with
bottleneck blocks).
"""
import math

import numpy as np
import torch

import pb_workloads as W
from paper_2003_11666_amd import PBEngine
from paper_2003_11666_amd.binding import scale_hyperparameters, update_standalone

VGG_WIDTHS = (1, 2, 4, 4, 8, 8, 8, 8)        # VGG-11's eight conv layers, in units of the first one's channels
VGG_POOLS = (0, 1, 3, 5, 7)                  # layers followed by a 2x2 max-pool, as far as the map can be halved


def _train(name, family, ticks, *, lr_ref=0.001, hw=32, width=64, widths="", layers="", groups=4, extra=0, in_dim=0,
           classes=10, feed="pool", mitigation=3, update_size=1, stash=False, lwp_form="v", dtype="fp32"):
    c = dict(kind="train", family=family, ticks=ticks, lr_ref=lr_ref, hw=hw, width=width, widths=widths, layers=layers,
             groups=groups, extra=extra, in_dim=in_dim, classes=classes, feed=feed, mitigation=mitigation,
             update_size=update_size, stash=stash, lwp_form=lwp_form, dtype=dtype)
    return dict(c, name=name) if name else c


def listed():
    return [
        # online learning with the small perceptron: a handful of samples arrive from the host, then the model is read back
        _train("mlp_online", "mlp", 16, in_dim=64, width=128, layers="3", feed="host"),
        # the perceptron trained from a resident pool: the shortest tick there is
        _train("mlp_pool", "mlp", 1000, in_dim=64, width=128, layers="3"),
        # a wide perceptron: matrix-vector work, every weight touched once per pass and tick
        _train("mlp_wide", "mlp", 256, in_dim=1024, width=1024, layers="4", classes=100),
        # a small ResNet on maps whose rows fit no tile (20x20, 12 and 20 channels)
        _train("resnet_ragged", "basic", 256, hw=20, widths="12-20", layers="2-2", classes=7),
        # the headline: ResNet-20 on 32x32 inputs, spike compensation and weight prediction on
        _train("resnet20", "basic", 512, widths="16-32-64", layers="3-3-3"),
        # the ablation (plain delayed momentum), fed by a data loader on the host
        _train("resnet20_host_plain", "basic", 256, widths="16-32-64", layers="3-3-3", feed="host", mitigation=0),
        # weight stashing with an update every four samples
        _train("resnet20_stash_n4", "basic", 256, widths="16-32-64", layers="3-3-3", update_size=4, stash=True),
        # VGG-11: post-layer GroupNorm, pooling, 512-channel layers on tiny maps
        _train("vgg11", "vgg", 512, lr_ref=1e-4, width=64, groups=8),
        # the wide stress network: ResNet-20 at four times the width and eight more conv stages
        _train("wide_resnet", "basic", 512, widths="64-128-256", layers="3-3-3", extra=8),
        # ResNet-50's stages on small images, fp32 activations
        _train("resnet50_64", "bottleneck", 384, hw=64, width=64, layers="3-4-6-3", groups=32, classes=1000),
        # ResNet-50 at full size, bf16 activations: the largest
        _train("resnet50", "bottleneck", 256, hw=224, width=64, layers="3-4-6-3", groups=32, classes=1000, dtype="bf16"),
        # the optimizer step alone over parameter arrays far beyond the caches
        dict(name="update_64m", kind="update", n=64 << 20, predict=True),
    ]


def _log_int(rng, lo, hi, step=1):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step))


def draw(rng):
    family = rng.choice(["mlp", "mlp", "vgg", "basic", "basic", "basic", "bottleneck", "bottleneck", "update"])
    if family == "update":
        return dict(kind="update", n=_log_int(rng, 1 << 14, 64 << 20, 1024), predict=rng.random() < 0.75)
    opt = dict(feed=rng.choice(["pool", "pool", "host"]), mitigation=rng.choice([3, 3, 3, 2, 1, 0]),
               update_size=rng.choice([1, 1, 1, 1, 2, 4, 8]), stash=rng.random() < 0.15, lwp_form=rng.choice(["v", "v", "v", "w"]))
    if family == "mlp":
        c = _train(None, "mlp", 0, in_dim=_log_int(rng, 16, 1024), width=_log_int(rng, 24, 1024), layers=str(rng.randint(2, 5)),
                   classes=_log_int(rng, 4, 100), **opt)
    elif family == "vgg":
        c = _train(None, "vgg", 0, lr_ref=1e-4, hw=rng.randint(12, 40), width=8 * rng.randint(1, 8), groups=rng.choice([4, 8]),
                   classes=_log_int(rng, 4, 100), **opt)
    elif family == "basic":
        w, n = _log_int(rng, 12, 64, 4), rng.randint(1, 3)
        c = _train(None, "basic", 0, hw=rng.randint(12, 40), widths="-".join(str(w << i) for i in range(n)), groups=rng.choice([2, 4]),
                   layers="-".join(str(rng.randint(1, 3)) for _ in range(n)), extra=rng.choice([0, 0, 2, 8]),
                   classes=_log_int(rng, 4, 100), **opt)
    else:
        base = rng.choice([16, 32, 64, 64])
        c = _train(None, "bottleneck", 0, hw=_log_int(rng, 40, 224), width=base, groups=base // rng.choice([2, 4]),
                   layers="-".join(str(rng.randint(1, n)) for n in (3, 4, 6, 3)[: rng.randint(2, 4)]),
                   classes=_log_int(rng, 10, 1000), dtype=rng.choice(["fp32", "bf16"]), **opt)
    net = _network(c)
    most = listed()[10]
    big = _network(most)
    cap = 0.5 * most["ticks"] * min(_macs(big) / _macs(net), W.count_params(big) / W.count_params(net))
    c["ticks"] = int(max(16, min(cap, _log_int(rng, 64, 1024))))
    return c


def _ints(text):
    return tuple(int(v) for v in text.split("-"))


def _network(case):
    c, hw = case, case["hw"]
    if c["family"] == "mlp":
        st = W.mlp((c["in_dim"],) + (c["width"],) * _ints(c["layers"])[0] + (c["classes"],))
        shape = (c["in_dim"], 1, 1)
    elif c["family"] == "vgg":
        pools, m = [], hw
        for i in VGG_POOLS:
            if m >= 2:
                pools.append(i)
                m //= 2
        st = W.vgg(tuple(c["width"] * k for k in VGG_WIDTHS), tuple(pools), c["groups"], n_classes=c["classes"], in_hw=hw)
        shape = (3, hw, hw)
    elif c["family"] == "basic":
        st = _basic(_ints(c["widths"]), _ints(c["layers"]), c["groups"], c["classes"], c["extra"])
        shape = (3, hw, hw)
    else:
        st = W.preact_resnet_bottleneck(_ints(c["layers"]), c["width"], c["groups"], n_classes=c["classes"])
        shape = (3, hw, hw)
    lr, momentum = scale_hyperparameters(c["lr_ref"], 0.9, 128, c["update_size"])
    return dict(name=c.get("name", c["family"]), stages=st, in_c=shape[0], in_h=shape[1], in_w=shape[2], n_classes=c["classes"],
                lr=lr, momentum=momentum, act_dtype=c["dtype"])


def _basic(widths, blocks, groups, classes, extra):
    """pb_workloads.preact_resnet_basic with a number of blocks of its own for every width."""
    stages, c = [[W.conv(3, widths[0], 3, 1, 1)]], widths[0]
    for gi, (w, n) in enumerate(zip(widths, blocks)):
        for bi in range(n):
            stride = 2 if gi > 0 and bi == 0 else 1
            tap = len(stages)
            stages.append([W.gn(groups, c), W.relu(), W.conv(c, w, 3, stride, 1)])
            stages.append([W.gn(groups, w), W.relu(), W.conv(w, w, 3, 1, 1), W.add(tap, c, w, stride, 1 if stride != 1 or c != w else 0)])
            c = w
    for _ in range(extra):
        stages.append([W.gn(groups, c), W.relu(), W.conv(c, c, 3, 1, 1)])
    stages.append([W.gn(groups, c), W.relu(), W.gap(), W.linear(c, classes, bias=1), W.ce()])
    return stages


def _macs(net):
    """Multiply-accumulates of one forward pass."""
    n = 0
    for st, (i, _) in zip(net["stages"], W.stage_shapes(net)):
        c, h, w = i
        for o in st:
            if o["kind"] == "conv":
                h, w = (h + 2 * o["pad"] - o["k"]) // o["stride"] + 1, (w + 2 * o["pad"] - o["k"]) // o["stride"] + 1
                n += o["cout"] * o["cin"] * o["k"] ** 2 * h * w
            elif o["kind"] == "linear":
                n += o["cin"] * o["cout"]
            elif o["kind"] == "add" and o["proj"]:
                n += o["cin"] * o["cout"] * h * w
    return n


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    if case["kind"] == "update":
        n = case["n"]
        # weights and velocity as training leaves them, gradients of one sample
        w, v, gr = (s * torch.randn(n, device="cuda", generator=g) for s in (0.05, 0.01, 0.01))
        return dict(case=case, w=w, v=v, g=gr, what=w.clone() if case["predict"] else None)
    net = _network(case)
    eng = PBEngine(net, seed=seed, mitigation=case["mitigation"], bwd_weights=int(case["stash"]), update_size=case["update_size"],
                   lwp_form=case["lwp_form"], loss_capacity=case["ticks"])
    elems = net["in_c"] * net["in_h"] * net["in_w"]
    n_pool = max(16, min(256, (4 << 20) // elems))
    s = dict(case=case, eng=eng, at=0)
    if case["feed"] == "pool":
        s["x"] = torch.randn(n_pool, net["in_c"], net["in_h"], net["in_w"], device="cuda", generator=g)
        s["y"] = torch.randint(0, net["n_classes"], (n_pool,), device="cuda", generator=g, dtype=torch.int32)
    else:   # a data loader's output in host memory
        r = np.random.default_rng(seed)
        s["x"] = r.standard_normal((n_pool, net["in_c"], net["in_h"], net["in_w"]), dtype=np.float32)
        s["y"] = r.integers(0, net["n_classes"], n_pool, dtype=np.int32)
    return s


def run(state):
    case = state["case"]
    if case["kind"] == "update":
        # SC coefficients of a stage with delay 20 at momentum 0.9
        a = 0.9 ** 20
        update_standalone(state["w"], state["v"], state["g"], state["what"], 0.005, 0.9, a, (1 - a) / 0.1, 0.005 * 20)
        out = {"weights": state["w"], "velocity": state["v"]}
        return dict(out, predicted=state["what"]) if case["predict"] else out
    eng, x, y, at, n = state["eng"], state["x"], state["y"], state["at"], case["ticks"]
    if case["feed"] == "pool":
        eng.run_resident(x, y, at, n)
    else:
        for i in range(at, at + n):
            eng.tick(x[i % len(y)], y[i % len(y)])
    state["at"] = at + n
    return {"losses": eng.loss_history(), "weights": eng.read_weights(), "velocity": eng.read_velocity()}


def work(case):
    if case["kind"] == "update":
        return {"bytes": (24 if case["predict"] else 20) * case["n"], "flops": 8 * case["n"]}
    net = _network(case)
    p, shapes = W.count_params(net), W.stage_shapes(net)
    acts = sum(c * h * w for (c, h, w), _ in shapes)
    width = 2 if case["dtype"] == "bf16" else 4
    # A tick: weights and velocity read and written (the prediction is a function of both, the gradient can stay on chip);
    # every stage's input written, read by the forward pass and again by the backward pass, and its gradient written and read.
    tick = 16 * p + 5 * width * acts
    return {"bytes": case["ticks"] * tick + 8 * p + 4 * case["ticks"], "flops": case["ticks"] * (6 * _macs(net) + 8 * p)}


def tolerance(case):
    if case["kind"] == "update":
        return {"rel": 1e-6, "max": 1e-5}
    # Sums in 32 bits in another order move a pre-activation by about 1e-7; where that decides a ReLU or a max-pool tie
    # the other way, one sample's gradient changes, and training carries the difference on: the velocity, a sum of
    # gradients, feels it most (weights and losses stay within 1e-4).  bf16 activations add decisions of their own.
    return {"rel": 3e-2, "max": 0.99} if case["dtype"] == "bf16" else {"rel": 5e-3, "max": 0.5}
