"""The host interface on a host stand-in for the device runtime (host_runtime.cpp).  Two host
threads that read two lattices of one set at the same time get each its own lattice's values:
the stand-in keeps the first read's launch waiting until the second one's has followed, so a
read that does not hold the set's scratch until its copies are done returns the other's
values."""
import ctypes
import os
import subprocess
import threading

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = "/opt/rocm/bin/amdclang++"


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    from paper_1808_08921_amd import lbdem

    out = str(tmp_path_factory.mktemp("host") / "liblbdem_host.so")
    subprocess.run([CXX, "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-std=c++17", "-O1", "-fPIC", "-shared", "-pthread",
                    "-Wl,-Bsymbolic", "-I/opt/rocm/include", "-o", out,
                    os.path.join(ROOT, "paper_1808_08921_amd", "csrc", "lbdem_api.cpp"),
                    os.path.join(ROOT, "tests", "host_runtime.cpp"), "--rtlib=libgcc"], check=True)
    L = ctypes.CDLL(out)
    L.path = out
    L.lb = lbdem
    return L


def make_set(L, sizes, room):
    lb = L.lb
    lat = (lb.Params * len(sizes))(*[lb.make_params(*s, max_particles=room, max_radius=2.0) for s in sizes])
    cfg = lb.Config()
    L.lbdem_default_config(ctypes.byref(cfg))
    cfg.graph_steps = 0
    h = ctypes.c_void_p()
    assert L.lbdem_create(len(sizes), lat, ctypes.byref(cfg), None, ctypes.c_size_t(0), None, ctypes.byref(h)) == lb.OK
    return h


def place(L, h, lattice, n):
    x, r = np.full((n, 3), 4.0), np.full(n, 2.0)
    dp = ctypes.POINTER(ctypes.c_double)
    assert L.lbdem_particles_set(h, lattice, n, x.ctypes.data_as(dp), None, None, r.ctypes.data_as(dp), None, None) == 0


def doubles(a):
    return a.ctypes.data_as(ctypes.POINTER(ctypes.c_double))


def together(L, readers):
    """Runs the readers on a thread each, the second from the time the first has launched."""
    rc = [None] * len(readers)

    def run(k):
        rc[k] = readers[k]()

    L.host_hold(400)
    threads = [threading.Thread(target=run, args=(k,)) for k in range(len(readers))]
    threads[0].start()
    while L.host_launches() < 1:
        pass
    threads[1].start()
    for t in threads:
        t.join()
    L.host_hold(0)
    assert rc == [0, 0]


@pytest.mark.parametrize("second", ["particles", "fields"])
@pytest.mark.parametrize("first", ["particles", "fields"])
def test_readers_of_one_set_on_two_threads(host, first, second):
    n, shape = 5, (9, 8, 7)
    h = make_set(host, [shape, shape], n)
    cells = shape[0] * shape[1] * shape[2]
    readers, checks = [], []
    for m, kind in enumerate((first, second)):
        place(host, h, m, n)
        if kind == "particles":
            out = np.zeros((5, n, 3))

            def read(m=m, out=out):
                return host.lbdem_particles_get(h, m, n, *[doubles(out[q]) for q in range(5)])

            want = 1000.0 * m * n + np.arange(15.0 * n).reshape(5, n, 3)
        else:
            out = np.zeros((4, cells))

            def read(m=m, out=out):
                return host.lbdem_fields_get(h, m, doubles(out[0]), doubles(out[1:]), None)

            want = np.full((4, cells), m + 1.0)
        readers.append(read)
        checks.append((out, want))
    together(host, readers)
    for out, want in checks:
        assert np.array_equal(out, want)
    host.lbdem_destroy(h)


def test_read_without_host_memory(host):
    """No exception crosses the interface when the host has no memory for a staging copy: the
    read then copies array by array (run in a process of its own, which an exception ends)."""
    code = f"""
import ctypes, sys
sys.path.insert(0, {ROOT!r}); sys.path.insert(0, {os.path.join(ROOT, "tests")!r})
import numpy as np
import test_host_readers as t
from paper_1808_08921_amd import lbdem
L = ctypes.CDLL({host.path!r})
L.lb = lbdem
n = 50
h = t.make_set(L, [(20, 20, 20)], n)
t.place(L, h, 0, n)
out = np.full((5, n, 3), 7.0)
L.host_fail_new(ctypes.c_size_t(1024))
rc = L.lbdem_particles_get(h, 0, n, *[t.doubles(out[q]) for q in range(5)])
L.host_fail_new(ctypes.c_size_t(0))
assert rc == 0, rc
assert (out[0] == 4.0).all() and not out[1:].any()
"""
    r = subprocess.run([os.sys.executable, "-c", code], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]


@pytest.mark.parametrize("precision,es,cs", [("fp64", 8, 8), ("fp32", 4, 4), ("fp16", 2, 4)])
def test_adjoint_workspace_of_one_segment(host, precision, es, cs):
    """A window of one segment starts from the window's start state and keeps no checkpoint:
    per node (rounded up to a wave) the start and one state per step, two adjoint fields, per
    direction a wall term and an FP64 gradient sum, the node map and the slot tables (at most
    32 bytes); then tables by plane, step and workgroup, here below 8 KB."""
    lb = host.lb
    lat = (lb.Params * 1)(lb.make_params(40, 40, 40))
    cfg = lb.Config()
    host.lbdem_default_config(ctypes.byref(cfg))
    cfg.graph_steps, cfg.precision = 0, lb.PRECISIONS[precision]
    h = ctypes.c_void_p()
    assert host.lbdem_create(1, lat, ctypes.byref(cfg), None, ctypes.c_size_t(0), None, ctypes.byref(h)) == lb.OK
    need = ctypes.c_size_t()
    steps = 5
    assert host.lbdem_adj_workspace_size(h, 0, ctypes.c_int64(steps), steps, ctypes.byref(need)) == lb.OK
    node = 19 * es * (1 + steps) + 2 * 19 * cs + 18 * (cs + 8) + 32
    assert need.value <= node * 40 ** 3 + 8192
    host.lbdem_destroy(h)
