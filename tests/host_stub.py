"""The host runtime (pb_host.cpp) compiled for the CPU over the stand-in of the HIP runtime in host_stub.cpp."""
import ctypes
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def build(path, planted=None):
    """planted: texts of pb_host.cpp and what stands in their place, for tests of its own checks."""
    csrc = os.path.join(ROOT, "paper_2003_11666_amd", "csrc")
    source = os.path.join(csrc, "pb_host.cpp")
    if planted:
        with open(source) as f:
            text = f.read()
        for old, new in planted.items():
            assert text.count(old) == 1, old
            text = text.replace(old, new)
        source = os.path.join(os.path.dirname(path), "pb_host.cpp")
        with open(source, "w") as f:
            f.write(text.replace('"../../include/', '"%s/include/' % ROOT))
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + csrc, "-w",
                    source, os.path.join(ROOT, "tests", "host_stub.cpp"),
                    # (the library's own pthread_create and hip* functions, whatever else the process has loaded)
                    "-static-libstdc++", "-Wl,-Bsymbolic", "-ldl", "-lpthread", "-o", path], check=True)
    return path


def load(path):
    """The stub library, in place of the HIP library in paper_2003_11666_amd.binding."""
    from paper_2003_11666_amd import binding as B
    B._LIB, B.lib_path = None, lambda: path
    lib = B.load_library()
    lib.stub_get.restype, lib.stub_get.argtypes = ctypes.c_long, [ctypes.c_char_p]
    lib.stub_set.restype, lib.stub_set.argtypes = None, [ctypes.c_char_p, ctypes.c_long]
    return lib


def prelude(path):
    return ("import sys\nsys.path.insert(0, %r)\nimport numpy as np\nimport pb_workloads as W\nfrom tests import host_stub\n"
            "from paper_2003_11666_amd import PBEngine, binding as B\nlib = host_stub.load(%r)\n"
            "get, put = (lambda n: lib.stub_get(n.encode())), (lambda n, v: lib.stub_set(n.encode(), v))\n"
            "def mlp(*dims): return W._net('p', W.mlp(dims), dims[0], 1, 1, dims[-1], 0.01, 0.9, 16, 5, 16)\n"
            "marshal, streams = B.marshal_net, [0]\n"
            "def engine(net, stream=None, **kw):          # (a stream of its own unless one is named)\n"
            "    streams[0] += 1\n"
            "    def on_stream(*a, **k):\n"
            "        d, keep = marshal(*a, **k)\n"
            "        d.stream = 16 * streams[0] if stream is None else stream\n"
            "        return d, keep\n"
            "    B.marshal_net = on_stream\n"
            "    try: return PBEngine(net, torch_arena=False, **kw)\n"
            "    finally: B.marshal_net = marshal\n" % (ROOT, path))


def run(path, body, **kw):
    """A program of its own (a fault of the library must not end the tests): prelude, then `body`."""
    r = subprocess.run([sys.executable, "-c", prelude(path) + body], capture_output=True, text=True, timeout=120, cwd=ROOT, **kw)
    assert r.returncode == 0, f"exit status {r.returncode}\n{r.stdout}\n{r.stderr}"
    return r.stdout
