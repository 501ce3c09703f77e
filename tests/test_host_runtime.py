"""The host runtime without a GPU: what it does when the system refuses something, and which launches it chooses."""
import os

import pytest

from tests import host_stub


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return host_stub.build(str(tmp_path_factory.mktemp("stub") / "libpb_stub.so"))


def test_read_back_without_the_threads_it_asks_for(lib):
    """4.7 million parameters, ten chunks through the ring of eight: unpacked by as many threads as there are."""
    host_stub.run(lib, """
from oracle import pb_oracle as O
net = mlp(2048, 2300, 12)
e, want = engine(net), O.PBOracle(net).read_weights().astype(np.float32)
for refused in (0, 1, 2, 100):
    put('threads_refused', refused)
    assert np.array_equal(e.read_weights(), want), refused
e.close()
""")


def test_host_memory_that_runs_out_is_an_error_code(lib):
    """A descriptor that asks for more host memory than the process may have: PB_E_NOMEM from every entry that plans a
    network, and the library goes on working."""
    host_stub.run(lib, """
import ctypes as C, resource
net = mlp(5, 7, 4)
desc, keep = B.marshal_net(net)
desc.n_stages = 2 ** 31 - 1
have = int(open('/proc/self/statm').read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (have + (4 << 30),) * 2)
ctx = C.c_void_p()
assert lib.pb_arena_bytes(C.byref(desc), None) == 0
for init in (lib.pb_init, lib.pb_init_static):
    assert init(C.byref(ctx), C.byref(desc), None, 0.1, 0.9, 1) == -3 and not ctx
    assert b'host memory' in lib.pb_last_error()
assert lib.pb_plan_summary(C.byref(desc), None, 0) == -3
e = engine(net)
assert e.read_weights().size == 5 * 7 + 7 + 7 * 4 + 4
e.close()
""")


def test_contexts_work_where_no_memory_can_be_pinned(lib):
    host_stub.run(lib, """
from oracle import pb_oracle as O
for at_init in (1, 0):                     # refused from the start, or only when a large read-back asks for its ring
    for net in (mlp(5, 7, 4), mlp(2048, 600, 12)):
        put('pinned_refused', at_init)
        e = engine(net)
        put('pinned_refused', 1)
        for t in range(9):
            e.tick(np.zeros(net['in_c'], np.float32), 0)
        assert np.array_equal(e.read_weights(), O.PBOracle(net).read_weights().astype(np.float32))
        assert e.loss_history().size == 9 - 2 + 1
        e.close()
""")


def test_launches_that_do_not_fit_the_gpu_together_take_turns(lib):
    """Contexts whose launches hold workgroups that wait for each other: launches of one wait for the other's (an event)
    exactly when their workgroups might not all find a place on the GPU's compute units."""
    host_stub.run(lib, """
wide, small = mlp(1024, 1024, 1024, 1024, 1024, 100), mlp(64, 128, 128, 128, 10)     # 177 and 25 workgroups, one to a compute unit
conv = W.config('small_resnet')                                                     # 248 workgroups, two to a compute unit
for cus, nets, together in [(256, [wide, small], True), (256, [wide, wide], False), (256, [small] * 8, True), (256, [small] * 9, False),
                            (64, [small, small], True), (64, [small] * 3, False), (256, [small, conv], True),
                            (256, [wide, conv], False), (256, [conv] * 2, True), (256, [conv] * 3, False)]:
    print(cus, [n['name'] for n in nets], together, flush=True)
    put('cus', cus)
    for name in ('mlp_launches', 'fused_launches', 'plain_launches', 'waits'):
        put(name, 0)
    engines = [engine(n) for n in nets]
    for _ in range(2):
        for n, e in zip(nets, engines):
            e.tick(np.zeros(n['in_c'] * n['in_h'] * n['in_w'], np.float32), 0)
    assert get('mlp_launches') + get('fused_launches') == 2 * len(nets) and get('plain_launches') == 0
    assert get('waits') == (0 if together else 2 * len(nets) - 1), get('waits')
    for e in engines:
        e.sync()
    put('waits', 0)                     # contexts whose work has been waited for take no room
    for _ in range(3):
        engines[0].tick(np.zeros(nets[0]['in_c'] * nets[0]['in_h'] * nets[0]['in_w'], np.float32), 0)
    assert get('waits') == 0
    for e in engines:
        e.close()
    engines = [engine(n, stream=16) for n in nets]      # nor do launches on one stream wait for each other's events
    for _ in range(2):
        for n, e in zip(nets, engines):
            e.tick(np.zeros(n['in_c'] * n['in_h'] * n['in_w'], np.float32), 0)
    assert get('waits') == 0
    for e in engines:
        e.close()
""")


def test_other_processes_on_the_gpu(lib):
    """While another process has waiting launches under way, ticks that would not fit beside them run as plain phase
    launches; when it has waited for its stream, is gone or was small enough, they don't.  An idle context holds nothing."""
    gpu = f"test-{os.getpid()}"
    other = host_stub.prelude(lib) + """
import os
net = {"wide": mlp(1024, 1024, 1024, 1024, 1024, 100), "small": mlp(64, 128, 128, 128, 10), "conv": W.config("small_resnet")}[sys.argv[1]]
x = np.zeros(net['in_c'] * net['in_h'] * net['in_w'], np.float32)
e = engine(net)
for line in sys.stdin:
    put('mlp_launches', 0), put('fused_launches', 0), put('plain_launches', 0)
    if line == 'tick\\n': e.tick(x, 0)
    if line == 'sync\\n': e.sync()
    if line == 'die\\n': os._exit(0)
    if line == 'fork\\n':                     # a child (a loader's worker, say) that cleans up what it inherited
        pid = os.fork()
        if pid == 0: e.sync(); os._exit(0)
        os.waitpid(pid, 0)
    print(get('mlp_launches'), get('fused_launches'), get('plain_launches'), flush=True)
"""
    try:
        host_stub.run(lib, f"""
import subprocess
class Other:
    def __init__(self, what):
        self.p = subprocess.Popen([sys.executable, '-c', {other!r}, what], stdin=subprocess.PIPE, stdout=subprocess.PIPE, text=True)
    def __call__(self, word):
        self.p.stdin.write(word + chr(10)); self.p.stdin.flush()
        return self.p.stdout.readline().split() if word != 'die' else self.p.wait()
a, b, small, conv, conv2 = Other('wide'), Other('wide'), Other('small'), Other('conv'), Other('conv')
mlp, fused = ['1', '0', '0'], ['0', '1', '0']
def plain(o): r = o('tick'); return r[:2] == ['0', '0'] and int(r[2]) >= 2
assert a('tick') == mlp                                  # six eighths
assert plain(b) and plain(conv)                          # (four eighths)
assert small('tick') == mlp and a('tick') == mlp
a('fork')
for _ in range(64): assert plain(b)
a('sync')
for _ in range(63): r = b('tick')                        # asked again 64 ticks after the refusal
assert r[0] == '0' and b('tick') == mlp and plain(a)
b('die')
for _ in range(63): a('tick')
assert a('tick') == mlp
a('sync'), small('sync')
for _ in range(64): conv('tick')
assert conv('tick') == fused and conv2('tick') == fused and plain(small)
conv('die')
for _ in range(63): small('tick')
assert small('tick') == mlp and a('tick')[0] == '0'
for o in (a, small, conv2): o('die')
""", env=dict(os.environ, STUB_GPU=gpu))
    finally:
        for d in ("/dev/shm", "/tmp"):
            if os.path.exists(f"{d}/pb-tick-{gpu}"):
                os.remove(f"{d}/pb-tick-{gpu}")


def test_a_launch_is_bounded_by_time(lib):
    """A launch that may hold every compute unit ends after 5 ms, at the ticks' measured durations, whatever is asked for."""
    host_stub.run(lib, """
import ctypes as C
pool, labels = np.zeros(4096, np.float32), np.zeros(4, np.int32)
for dims, us in [((64, 128, 128, 128, 10), 3.1), ((256,) * 6 + (10,), 3.4), ((512,) * 6 + (100,), 5.6), ((1024,) * 5 + (1000,), 9.1)]:
    put('mlp_ticks_max', 0), put('mlp_launches', 0)
    e = engine(mlp(*dims))
    assert lib.pb_run_resident(e.ctx, pool.ctypes.data, labels.ctypes.data, 4, 0, 5000) == 0 and e.ticks == 5000
    n, most = get('mlp_launches'), get('mlp_ticks_max')
    assert most * us <= 5000 and n == -(-5000 // most), (dims, n, most)
    e.close()
""")


def test_settings_that_choose_plain_launches(lib):
    """one_launch = -1: no launch of the context has workgroups that wait, in perceptrons and small networks alike."""
    host_stub.run(lib, """
for net in (mlp(1024, 1024, 1024, 100), mlp(64, 128, 10), W.config('small_resnet')):
    for tuning, plain in [(None, False), (dict(one_launch=-1), True)]:
        put('plain_launches', 0), put('mlp_launches', 0), put('fused_launches', 0)
        e = engine(net, tuning=tuning)
        for _ in range(3):
            e.tick(np.zeros(net['in_c'] * net['in_h'] * net['in_w'], np.float32), 0)
        assert (get('mlp_launches') + get('fused_launches') == 0) == plain and (get('plain_launches') > 0) == plain
        e.close()
""")


def test_streams_that_are_kept_to_some_compute_units(lib):
    """A launch of the perceptron kernel needs all of its workgroups resident: not on a stream with a mask."""
    host_stub.run(lib, """
net = mlp(64, 128, 128, 128, 10)
for masked, register_form in [(0, True), (256, True), (224, False), (32, False)]:
    put('masked', masked), put('mlp_launches', 0)
    e = engine(net)
    e.tick(np.zeros(64, np.float32), 0)
    assert (get('mlp_launches') == 1) == register_form, masked
    e.close()
""")


def test_networks_are_planned_side_by_side(lib):
    """Threads that plan different networks at the same time get the plans they get alone; of threads that ask for the
    library's own arena one gets it."""
    host_stub.run(lib, """
import threading
nets = [W.config(n) for n in ('resnet20', 'vgg11', 'mlp', 'wide', 'tiny_vgg', 'resnet50_64')]
alone = [B.plan_summary(n) for n in nets]
bad = []
def work(i):
    for _ in range(10):
        if B.plan_summary(nets[i]) != alone[i]: bad.append(nets[i]['name'])
threads = [threading.Thread(target=work, args=(i,)) for i in range(len(nets))]
[t.start() for t in threads]; [t.join() for t in threads]
assert not bad, bad
got = []
def take():
    try: got.append(PBEngine(W.config('tiny_mlp'), torch_arena=False, static_arena=True))
    except B.PBError: pass
import torch
torch.cuda.current_stream = lambda: type('S', (), dict(cuda_stream=None))
for _ in range(20):
    threads = [threading.Thread(target=take) for _ in range(6)]
    [t.start() for t in threads]; [t.join() for t in threads]
    assert len(got) == 1
    got.pop().close()
""")


def test_weights_in_lane_order_take_no_memory_of_their_own(lib):
    """A network whose 3x3 layers store weights in the order of their tiles' lanes: their read-back in canonical order goes by
    way of the gradients' block, so that what fits the static arena without that order (61.3 MiB) fits with it."""
    host_stub.run(lib, """
import ctypes as C
from oracle import pb_oracle as O
net = W._net("lanes", W.preact_resnet_basic((32, 64, 128), 3, 4, in_c=3, n_classes=5), 3, 20, 20, 5, 1e-3, 0.9, 8, 3, 8)
desc, keep = B.marshal_net(net)
assert lib.pb_arena_bytes(C.byref(desc), None) <= lib.pb_static_arena_bytes()
want = O.PBOracle(net).read_weights().astype(np.float32)
for kw in (dict(), dict(tuning=dict(tile_budget_us=26.0))):
    e = engine(net, **kw)
    for cap in (want.size, 1000):
        got = np.empty(cap, np.float32)
        assert lib.pb_read_weights(e.ctx, got.ctypes.data, cap) == cap and np.array_equal(got, want[:cap])
    assert not e.read_velocity().any()
    e.close()
""")


def test_a_gathered_weight_gradient_is_not_the_end_of_its_launch(lib):
    """The projection of stride 2 in a bottleneck network at 158 pixels: 13 chunks at 4.4 us each, dealt out so that no tile takes
    more than 30."""
    host_stub.run(lib, """
import re
net = W._net("gathered", W.preact_resnet_bottleneck((2, 4), 32, 8, n_classes=340), 3, 158, 158, 340, 1e-3, 0.9, 8, 3, 8)
steps = [l for l in B.plan_summary(net).splitlines() if " k1 s2 " in l and "gm3" in l]
parts = [tuple(map(int, re.search(r"chunks (\\d+)/(\\d+)", l).groups())) for l in steps]
assert parts and all(5.0 + 4.4 * -(-n // p) <= 30.0 for n, p in parts), steps
""")


def test_statistics_that_fit_no_registers_start_early(lib):
    """Groups of 30 x 23 x 23 elements, no multiple of 4, take 35 us: in front of the weight-gradient tiles of 8 us."""
    host_stub.run(lib, """
net = W._net("odd groups", W.preact_resnet_basic((60, 120, 240), 3, 2, in_c=3, n_classes=9), 3, 23, 23, 9, 1e-3, 0.9, 8, 3, 8)
steps = B.plan_summary(net, update_size=8).splitlines()
stats = [i for i, l in enumerate(steps) if "phase 0 gn_stats" in l and "C60x23x23" in l]
tiles = [i for i, l in enumerate(steps) if "phase 0 gemm" in l and "C240x6x6" in l and "gm3" in l]
assert stats and tiles and max(stats) < min(tiles), steps
""")


def test_reductions_the_bf16_tiles_cannot_share_out_stay_on_the_fp32_pipes(lib):
    """224 channels are seven blocks of 32: no two waves share them, and a tile of four waves side by side takes twice the time
    of one that splits the reduction on the fp32 pipes.  256 channels stay on the bf16 pipes."""
    host_stub.run(lib, """
for width, split in ((56, False), (64, True)):
    net = W._net("vgg", W.vgg(tuple(width * k for k in (1, 2, 4, 4, 8, 8, 8, 8)), (0, 1, 3, 5, 7), 4, n_classes=7, in_hw=33), 3, 33, 33, 7, 1e-3, 0.9, 8, 3, 8)
    steps = [l for l in B.plan_summary(net).splitlines() if f"C{4 * width}x8x8 K{4 * width}x8x8" in l and "direct" in l and "gm3" not in l]
    assert len(steps) == 2 and all((" split" in l) == split for l in steps), steps
""")


def test_short_steps_in_the_middle_of_a_network_do_not_shorten_the_others_tiles(lib):
    """A bottleneck network at 222 pixels: the first layer's forward step keeps its 97 tiles of 128 columns."""
    host_stub.run(lib, """
net = W._net("stem", W.preact_resnet_bottleneck((3, 1), 16, 8, n_classes=171), 3, 222, 222, 171, 1e-3, 0.9, 8, 3, 8)
steps = [l for l in B.plan_summary(net, mitigation=0).splitlines() if "C3x222x222" in l and "gm1" in l]
assert len(steps) == 1 and "tile 16x128" in steps[0], steps
""")


def test_layers_left_with_the_least_bf16_tile_run_on_the_fp32_pipes(lib):
    """256 channels on 81 pixels in a crowded launch: 48 and 96 tiles of 16 x 16 on the bf16 pipes, half as many, and no longer
    ones, on the fp32 pipes."""
    host_stub.run(lib, """
net = W._net("vgg", W.vgg(tuple(64 * k for k in (1, 2, 4, 4, 8, 8, 8, 8)), (0, 1, 3, 5, 7), 4, n_classes=70, in_hw=38), 3, 38, 38, 70, 1e-3, 0.9, 8, 3, 8)
steps = [l for l in B.plan_summary(net).splitlines() if "direct" in l and "gm2" in l]
assert len(steps) == 3 and not any("tile 16x16" in l and " split" in l for l in steps), steps
""")
