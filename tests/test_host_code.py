"""The library's host code -- the C ABI and every kernel launcher -- on the CPU,
linked with a stand-in for the HIP runtime (tests/host/fake_hip.cpp): calls of
the runtime can be made to fail, two devices exist, and the launches are on
record.  Kernels do nothing there, so no field values are tested here.
"""
from __future__ import annotations

import ctypes as C
import os
import re
import subprocess

import numpy as np
import pytest

from paper_1802_04243_amd import sts
from paper_1802_04243_amd import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1802_04243_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")


def _run(*cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, (cmd, r.stdout[-3000:], r.stderr[-3000:])
    return r.stdout


@pytest.fixture(scope="module")
def host_lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("host")
    flags = ["--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-I", os.path.join(ROOT, "include")]
    src = [os.path.join(CSRC, f) for f in ("sts_api.hip", "sts_kernels.hip", "sts_adjoint.hip", "sts3.hip")]
    src.append(os.path.join(ROOT, "tests", "host", "fake_hip.cpp"))
    jobs = [subprocess.Popen([HIPCC, *flags, "-c", s, "-o", str(d / f"{k}.o")], stderr=subprocess.PIPE,
                             text=True) for k, s in enumerate(src)]
    for s, j in zip(src, jobs):
        err = j.communicate()[1]
        assert j.returncode == 0, (s, err[-3000:])
    objs = [str(d / f"{k}.o") for k in range(len(src))]
    # the host objects name a device image each; there is none
    images = sorted(set(re.findall(r"\b__hip_fatbin_\w+", _run("nm", "-u", *objs))))
    (d / "images.c").write_text("".join(f"char {n}[16];\n" for n in images))
    so = str(d / "libsts_host.so")
    # -Bsymbolic: its runtime calls are bound to the stand-in's
    _run("gcc", "-fPIC", "-c", str(d / "images.c"), "-o", str(d / "images.o"))
    _run("g++", "-shared", "-Wl,-Bsymbolic", "-o", so, *objs, str(d / "images.o"), "-lpthread")
    return so


@pytest.fixture
def host(host_lib, monkeypatch):
    """The stand-in's controls; Solver and Solver3 run on the host library."""
    from paper_1802_04243_amd import sts3
    monkeypatch.setattr(sts, "LIB_PATH", host_lib)
    monkeypatch.setattr(sts, "_lib", None)
    monkeypatch.setattr(sts3, "_lib3", None)
    L = sts.lib()
    L.fake_fail.argtypes = [C.c_char_p, C.c_int]
    L.fake_calls.argtypes = [C.c_char_p]
    L.fake_launch.argtypes = [C.c_int, C.POINTER(C.c_uint), C.POINTER(C.c_void_p)]
    L.fake_launch.restype = C.c_char_p
    L.fake_watch.argtypes = [C.c_void_p, C.c_size_t, C.c_double]
    L.fake_watch_bad.restype = C.c_long
    L.fake_reset()
    return L


def _launches(L):
    """(kernel name, grid, third argument of a sum) of every launch."""
    out = []
    for k in range(L.fake_launches()):
        g, p = (C.c_uint * 3)(), C.c_void_p()
        name = L.fake_launch(k, g, C.byref(p)).decode()
        out.append((name, tuple(g), p.value))
    return out


def _solver(nx=120, ny=24, **kw):
    return sts.Solver(W.Problem(nx=nx, ny=ny, lx=0.1 * nx, ly=0.1 * ny, **kw), use_torch=False)


@pytest.mark.parametrize("what", ["hipMalloc", "hipHostMalloc"])
def test_a_drag_after_a_failed_allocation_never_writes_to_address_zero(host, what):
    s = _solver()
    host.fake_fail(what.encode(), 1)
    with pytest.raises(sts.StsError):
        s.drag()
    for _ in range(2):
        try:
            s.drag()
        except sts.StsError:
            pass
        assert all(l[2] for l in _launches(host) if "k_sum" in l[0])
    s.drag()
    assert sum("k_sum" in l[0] for l in _launches(host)) == 3
    s.close()


def _unchanged_until_copied(host, read, arrays):
    for k in range(len(arrays)):
        arrays[k][...] = np.pi
        host.fake_watch(arrays[k].ctypes.data, arrays[k].size, np.pi)
        read()
        assert arrays[k].flat[0] != np.pi  # the copy came
        assert host.fake_watch_bad() == 0, k


def test_reading_fields_writes_to_the_host_arrays_by_its_copies_alone(host):
    """Work that the caller queued earlier on the stream may still read them,
    and a copy that fails leaves them as they were."""
    s = _solver(nx=800, ny=720)  # above 4 MiB a field
    out = [np.zeros(q) for q in s.shapes()]
    p = [sts._ptr(a) for a in out]
    _unchanged_until_copied(host, lambda: sts._check(host.sts_fields(s._h, *p)), out)
    s.adjoint_begin(1)
    _unchanged_until_copied(host, lambda: sts._check(host.sts_adjoint_read_state_grad(s._h, *p)), out)
    for a in out:
        a[...] = np.pi
    host.fake_fail(b"hipMemcpyAsync", 1)
    assert host.sts_fields(s._h, *p) == sts.STS_EDEVICE
    assert all((a == np.pi).all() for a in out)
    s.close()


def test_reading_3d_fields_writes_to_the_host_arrays_by_its_copies_alone(host):
    from paper_1802_04243_amd import sts3
    from paper_1802_04243_amd import workloads3 as W3
    box = W3.Box3(d=tuple(np.full(n, 0.1) for n in (100, 80, 80)))
    s = sts3.Solver3(box, use_torch=False)
    out = [np.zeros(q) for q in box.shapes()]
    p = (sts._D * 5)(*[sts._ptr(a) for a in out])
    _unchanged_until_copied(host, lambda: sts._check(host.sts3_fields(s._h, p)), out)
    s.close()


def test_a_step_graph_is_recorded_for_the_device_of_its_context(host):
    host.hipSetDevice(1)
    s = _solver()
    host.hipSetDevice(0)
    for _ in range(6):
        s.step(1e-3, 4, 0)
    assert host.fake_calls(b"hipGraphLaunch") == 4
    assert host.fake_wrong_device() == 0
    d = C.c_int(-1)
    host.hipGetDevice(C.byref(d))
    assert d.value == 0  # the caller's device is current again
    s.close()


def test_steps_neither_wait_nor_create_streams_whatever_their_arguments(host):
    """Nor do they record a graph in more than every 16th step after the first
    two, or keep more than twice four; a wait lets go of the replaced ones, the
    end of all."""
    s = _solver()
    what = (b"hipStreamCreate", b"hipStreamSynchronize", b"hipEventSynchronize", b"hipMalloc", b"hipHostMalloc")
    before = [host.fake_calls(w) for w in what]
    made = lambda: host.fake_calls(b"hipGraphInstantiate")
    live = lambda: made() - host.fake_calls(b"hipGraphExecDestroy")
    steps = 0
    for k in range(60):  # each time step size for a few steps, then another
        for _ in range(3 + k % 4):
            s.step(1e-3 * (1 + k), 4 + (k % 3 == 0), 0)
            steps += 1
            assert made() <= 2 + steps // 16 and live() <= 8
    assert 4 <= made()
    assert [host.fake_calls(w) for w in what] == before
    s.residuals()
    assert live() <= 4
    s.step(1.0, 65, 0)  # never recorded: too many passes, or timed
    s.timing(True)
    n = host.fake_calls(b"hipGraphLaunch")
    for _ in range(40):
        s.step(1e-3, 4, 0)
    assert host.fake_calls(b"hipGraphLaunch") == n
    s.close()
    assert live() == 0


def test_a_step_whose_graph_cannot_be_made_takes_plain_launches(host):
    for what in ("hipStreamCreate", "hipStreamBeginCapture", "hipGraphInstantiate"):
        host.fake_reset()
        host.fake_fail(what.encode(), 2 if what == "hipStreamCreate" else 1)  # (the first is the context's own)
        s = _solver()
        for _ in range(9):
            n = host.fake_launches()
            s.step(1e-3, 4, 0)
            assert host.fake_launches() >= n + 6  # four passes, the residual's two
        assert host.fake_calls(b"hipGraphLaunch") == 0
        s.close()


# the sizes that sts_workspace_bytes gave before the strips' work items
@pytest.mark.parametrize("nx,ny,size", [(120, 24, 874240), (1600, 640, 122662656)])
def test_a_workspace_without_room_for_work_items_is_taken(host, nx, ny, size):
    import mmap
    mem = mmap.mmap(-1, size + 4096)  # page-aligned, read and written by the library
    base = C.addressof(C.c_char.from_buffer(mem))
    create = host.sts_create

    def smaller(*a):  # the binding's arguments, on this workspace
        return create(*a[:8], base, want, a[10])

    forms = {}
    for want in (size, size - 1, None):
        host.fake_reset()
        host.sts_create = create if want is None else smaller
        if want == size - 1:
            with pytest.raises(sts.StsError, match="workspace needs"):
                _solver(nx, ny)
            continue
        s = _solver(nx, ny)
        s.step(1e-3, 3, 0)
        forms[want] = {n for n, _, _ in _launches(host) if "k_pass" in n or "k_sweep" in n}
        s.close()
    assert not any("k_sweep" in n for n in forms[size])  # tiles
    assert any("k_sweep" in n for n in forms[None]) == (nx * ny > 1e6)


def test_laying_out_strips_among_many_obstacles_is_quick(host):
    """More runs of rows than the chip holds waves: the length of the segments
    is searched by halving.  (One by one, with every run counted for each
    length up to the grid's height, it took seconds.)"""
    import resource
    host.fake_copying(0)
    nx, ny = 300, 20000
    blocks = [(i, j, i, j) for i in range(30, nx - 30, 58) for j in range(10, ny - 10, 10)]
    took = []
    for obstacles in (blocks, ()):
        t = resource.getrusage(resource.RUSAGE_SELF).ru_utime
        _solver(nx, ny, obstacles=obstacles).close()
        took.append(resource.getrusage(resource.RUSAGE_SELF).ru_utime - t)
    print(took)
    assert took[0] < took[1] + 0.5


def test_a_repeated_step_is_a_graph_from_its_third_call_on(host):
    """Of an odd number of passes from its fifth: either buffer has its own."""
    for n, first in ((4, 3), (5, 5)):
        host.fake_reset()
        s = _solver()
        for _ in range(12):
            s.step(1e-3, n, 0)
        assert host.fake_calls(b"hipGraphLaunch") == 12 + 1 - first
        s.close()


def _form(host, s, form):
    return host.sts_internal_pass_form(s._h, form)


@pytest.mark.parametrize("nx,ny,strips", [(120, 24, 0), (1024, 256, 0), (1152, 288, 0), (1280, 288, 1),
                                          (1280, 320, 0), (1420, 284, 1), (1103, 389, 1), (1568, 392, 1),
                                          (5120, 1152, 1), (60, 50000, 0), (100000, 8, 1)])
def test_the_measured_rule_alone_chooses_the_form_of_a_pass(host, nx, ny, strips):
    """Grids on both sides of the rule, past two blocks each; the room for work
    items does not decide."""
    host.fake_copying(0)
    h = max(1, ny // 4)
    s = _solver(nx, ny, obstacles=[(nx // 3, ny // 2, nx // 3 + min(h, nx // 9), ny // 2 + h - 1),
                                   (nx // 2, 1, nx // 2 + min(h, nx // 9), h)])
    assert (_form(host, s, 0) > 0) == bool(strips)
    assert _form(host, s, 2) > 0 or nx * ny < 300_000  # (no room where the rule never asks)
    s.close()


def test_strips_fit_on_every_grid_of_the_rule_s_range(host):
    host.fake_copying(0)
    rng = np.random.default_rng(3)
    for k in range(60):
        v, r = np.exp(rng.uniform(np.log(8e5), np.log(4e6))), np.exp(rng.uniform(-7, 7))
        nx = max(4, int((v * r) ** 0.5))
        ny = max(4, int(v / nx))
        s = _solver(nx, ny, periodic=bool(k % 2))
        assert _form(host, s, 2) > 0, (nx, ny)
        s.close()


def test_contexts_of_a_device_share_the_stream_that_graphs_are_recorded_on(host):
    """One per device while a small context of it lives, none after the last."""
    made = lambda: host.fake_calls(b"hipStreamCreate")
    gone = lambda: host.fake_calls(b"hipStreamDestroy")
    for device in (0, 1, 0):
        host.fake_reset()
        host.hipSetDevice(device)
        s = [_solver() for _ in range(3)]
        assert made() == 3 + 1
        for k in range(6):
            for q in s:
                q.step(1e-3, 4, 0)
        assert host.fake_calls(b"hipGraphLaunch") == 3 * 4 and host.fake_wrong_device() == 0
        for q in s:
            q.close()
        assert gone() == made()


def test_threads_that_step_at_once_each_get_their_graph(host):
    import threading
    s = [_solver() for _ in range(4)]

    def run(q):
        for _ in range(60):
            q.step(1e-3, 4, 0)

    threads = [threading.Thread(target=run, args=(q,)) for q in s]
    [t.start() for t in threads], [t.join() for t in threads]
    assert host.fake_calls(b"hipGraphInstantiate") == 4
    for q in s:
        q.close()


@pytest.mark.parametrize("n", [(4, 4, 20000), (4, 70000, 4), (4, 4, 65533), (5, 16385, 5)])
@pytest.mark.parametrize("periodic", [False, True])
def test_launches_of_long_boxes_keep_to_the_grid_limits(host, n, periodic):
    """At most 65535 blocks along y and z, whatever the box's proportions."""
    from paper_1802_04243_amd import sts3
    from paper_1802_04243_amd import workloads3 as W3
    host.fake_copying(0)
    bc = (W3.PERIODIC,) * 3 if periodic else (W3.INLET_OUTLET, W3.WALLS, W3.WALLS)
    s = sts3.Solver3(W3.Box3(d=tuple(np.full(m, 0.1) for m in n), bc=bc), use_torch=False)
    for scheme in W.SCHEMES.values():
        s.step(1e-3, 2, scheme)
    for name, grid, _ in _launches(host):
        assert all(1 <= g <= 65535 for g in grid[1:]), (name, grid)
    s.close()


def test_reading_a_small_box_queues_no_copies(host):
    """(One of 5 x 20 us to pageable memory each took twice as long as the
    copies of the padded fields had.)"""
    from paper_1802_04243_amd import sts3
    from paper_1802_04243_amd import workloads3 as W3
    s = sts3.Solver3(W3.Box3(d=tuple(np.full(m, 0.1) for m in (8, 6, 5))), use_torch=False)
    n = host.fake_calls(b"hipMemcpyAsync") + host.fake_calls(b"hipMemcpy")
    s.fields()
    assert host.fake_calls(b"hipMemcpyAsync") + host.fake_calls(b"hipMemcpy") == n
    s.close()


def test_a_refused_workspace_is_reported_with_the_size_it_needs(host):
    """The message is made before the context is given back."""
    M_PERTURB = -6  # freed memory is overwritten
    libc = C.CDLL(None)
    create = host.sts_create
    g = sts._Grid(120, 24, 1.0, 1.0, None, None)
    need = C.c_size_t()
    sts._check(host.sts_workspace_bytes(C.byref(g), C.byref(need)))
    mem = np.zeros(512)
    base = (mem.ctypes.data + 255) // 256 * 256
    libc.mallopt(M_PERTURB, 0xA5)
    try:
        host.sts_create = lambda *a: create(*a[:8], base, 256, a[10])
        with pytest.raises(sts.StsError, match=f"needs {need.value} bytes"):
            _solver()
        host.sts_create = create
        host.fake_fail(b"hipMalloc", 1)
        with pytest.raises(sts.StsError, match=f"hipMalloc of {need.value} bytes"):
            _solver()
    finally:
        libc.mallopt(M_PERTURB, 0)
        host.sts_create = create
