"""The library's host code on a HIP runtime without a device (hip_host.cpp): what it does when an
allocation or a launch fails, or when a resident solve reports that it could not finish."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.dirname(os.path.abspath(__file__))
OK, OOM, DEVICE, INTERNAL = 0, -2, -3, -5
MiB = 1 << 20
STATIC_OR, SIMPLE_OR = 6, 24


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    from paper_1903_12085_amd import build
    objs = [os.path.join(build.HERE, "_build", s.replace(".hip", ".o")) for s in build.SOURCES]
    newest = max(os.path.getmtime(os.path.join(build.CSRC, f)) for f in os.listdir(build.CSRC))
    if any(not os.path.exists(o) or os.path.getmtime(o) < newest for o in objs):
        build.build()
    d = tmp_path_factory.mktemp("host")
    rt, so = str(d / "hip_host.o"), str(d / "libhost.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-c",
                    os.path.join(HERE, "hip_host.cpp"), "-o", rt], check=True)
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", "-Wl,-z,defs", "-o", so] + objs + [rt], check=True)
    L = ctypes.CDLL(so)
    L.host_reset.argtypes = [ctypes.c_size_t]
    L.host_used.restype = L.host_peak.restype = ctypes.c_size_t
    L.host_log.restype = L.sssp_last_error.restype = ctypes.c_char_p
    L.sssp_graph_create.argtypes = [ctypes.c_uint32, ctypes.c_uint64] + [ctypes.c_void_p] * 3 + [
        ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p]
    L.sssp_delta_step.argtypes = [ctypes.c_void_p, ctypes.c_uint32, ctypes.c_uint64, ctypes.c_void_p, ctypes.c_void_p]
    L.host_reset(1 << 40)
    return L


def ptr(a):
    return a.ctypes.data_as(ctypes.c_void_p)


class Host:
    """A graph of n vertices and m edges on the host runtime, and calls on it."""

    def __init__(self, lib, n=9, m=16):
        rng = np.random.default_rng(1)
        self.lib, self.n = lib, n
        rp = (np.arange(n + 1, dtype=np.uint64) * m) // n
        col, w = rng.integers(0, n, m).astype(np.uint32), np.ones(m, np.uint32)
        self.h = ctypes.c_void_p()
        self.rc = lib.sssp_graph_create(n, m, ptr(rp), ptr(col), ptr(w), 0, None, ctypes.byref(self.h))
        self.dist, self.phases = np.zeros(n, np.uint64), ctypes.c_uint32(99)

    def solve(self, crit=STATIC_OR, call="sssp_solve"):
        return getattr(self.lib, call)(self.h, 0, crit, ptr(self.dist), ctypes.byref(self.phases))

    def delta(self):
        return self.lib.sssp_delta_step(self.h, 0, 100, ptr(self.dist), ctypes.byref(self.phases))

    def batch(self, nq=2, shape=(0, 0, 0, 0, 0)):
        hs = (ctypes.c_void_p * nq)(*[self.h.value] * nq)
        ds = [np.zeros(self.n, np.uint64) for _ in range(nq)]
        outs = (ctypes.c_void_p * nq)(*[ptr(d).value for d in ds])
        src = np.zeros(nq, np.uint32)
        return self.lib.sssp_solve_batch_ex(hs, ptr(src), nq, STATIC_OR, outs, None, (ctypes.c_uint32 * 5)(*shape))

    def learned(self):
        w, sel, none = np.zeros(5382, np.float32), ctypes.c_void_p(), ctypes.c_void_p()
        assert self.lib.sssp_selector_create(ptr(w), ctypes.byref(sel)) == OK
        rc = self.lib.sssp_solve_learned_checkpoint(self.h, 0, sel, ptr(self.dist), none, none, none, 0, none)
        self.lib.sssp_selector_destroy(sel)
        return rc

    def log(self):
        return self.lib.host_log().decode().split()

    def message(self):
        return self.lib.sssp_last_error().decode()

    def close(self):
        self.lib.sssp_graph_destroy(self.h)


SOLVES = {"static": lambda g: g.solve(), "simple": lambda g: g.solve(SIMPLE_OR), "delta": lambda g: g.delta(),
          "noalloc": lambda g: g.solve(call="sssp_solve_noalloc"), "batch": lambda g: g.batch(),
          "learned": lambda g: g.learned()}


@pytest.mark.parametrize("name", list(SOLVES))
def test_broken_phase_bound_is_an_error(lib, name):
    """A resident solve that ran for more phases than there can be has broken an invariant: that is
    reported, not covered up by a second solve with other kernels."""
    g = Host(lib)
    assert g.rc == OK
    lib.host_reset(1 << 40)
    lib.host_coop(0, 2, 5, 6 if name == "batch" else 0)
    assert SOLVES[name](g) == INTERNAL and "phase bound" in g.message()
    after = g.log()[g.log().index("coop"):]
    assert after.count("kernel") == (name == "learned")  # its counts are queued before the read-back
    if name != "learned":  # its second stage would need the kernels
        lib.host_coop(0, 0, 5, 6 if name == "batch" else 0)
        assert SOLVES[name](g) == OK and (name == "batch" or g.phases.value == 5)
    g.close()


def keep_block(lib):
    """Destroys a graph of about 80 MB, whose block the library keeps."""
    lib.host_reset(1 << 40)
    lib.sssp_graph_destroy(None)
    big = Host(lib, 1 << 20, 6 << 20)
    assert big.rc == OK
    before = lib.host_used()
    big.close()
    assert before - lib.host_used() < MiB  # still held


def create(lib, g):
    made = Host(lib, 5, 7)
    made.close()
    return made.rc


def one_workgroup(lib, g):
    cfg = (ctypes.c_uint32 * 6)()
    lib.sssp_get_launch(g.h, cfg)
    cfg[5] = 1
    assert lib.sssp_set_launch(g.h, cfg) == OK
    return g.solve()


def batch_shape(lib, g, nq=1):
    return g.batch(nq, (256, 0, 0, 0, 0))


def traced(lib, g):
    trace, st = np.zeros(64, np.uint64), np.zeros(64, np.uint64)
    return lib.sssp_solve_ex(g.h, 0, SIMPLE_OR, ptr(g.dist), ptr(st), None, ptr(trace), 2)


def selector(lib, g):
    sel = ctypes.c_void_p()
    rc = lib.sssp_selector_create(ptr(np.zeros(5382, np.float32)), ctypes.byref(sel))
    if rc == OK:
        x, y = np.zeros((4, 12), np.float32), np.zeros((4, 6), np.float32)
        rc = lib.sssp_selector_forward(sel, ptr(x), 4, ptr(y))
        lib.sssp_selector_destroy(sel)
    return rc


ALLOCATING = {"create": create, "static": (lambda lib, g: g.solve()), "simple": (lambda lib, g: g.solve(SIMPLE_OR)),
              "delta": (lambda lib, g: g.delta()), "batch": (lambda lib, g: g.batch()), "batch_shape": batch_shape,
              "one_workgroup": one_workgroup, "traced": traced, "learned": (lambda lib, g: g.learned()),
              "selector": selector}


@pytest.mark.parametrize("name", list(ALLOCATING))
def test_kept_block_is_given_back_whichever_allocation_fails(lib, name):
    """With memory for all but the last k bytes of what a call allocates, k from 1 to all of it: one of its
    allocations fails first, the kept block goes, and the call succeeds as with memory to spare. (Solves
    that need the phase kernels end in their phase bound here, since kernels do nothing.)"""
    def attempt(slack):
        g = Host(lib)
        assert g.rc == OK
        lib.host_reset(lib.host_used() + slack)
        rc = ALLOCATING[name](lib, g)
        log, msg, peak = g.log(), g.message(), lib.host_peak()
        lib.host_reset(1 << 40)
        g.close()
        return rc, log, msg, peak

    keep_block(lib)
    expect, log, _, need = attempt(1 << 30)
    assert expect in (OK, INTERNAL) and "oom" not in log and need > 0
    for i in range(24):
        keep_block(lib)
        rc, log, msg, _ = attempt((need - 1) * i // 24)
        assert rc == expect, (i, rc, msg)
        assert log.count("oom") == 1, (i, log[:20])
    lib.sssp_graph_destroy(None)


def phase_kernels(lib, g):
    cfg = (ctypes.c_uint32 * 6)()
    lib.sssp_get_launch(g.h, cfg)
    cfg[5] = 2
    assert lib.sssp_set_launch(g.h, cfg) == OK


# the call, and the same work by kernels without resident scratch
WITHOUT = {"static": (ALLOCATING["static"], phase_kernels, ALLOCATING["static"]),
           "simple": (ALLOCATING["simple"], phase_kernels, ALLOCATING["simple"]),
           "delta": (ALLOCATING["delta"], phase_kernels, ALLOCATING["delta"]),
           "learned": (ALLOCATING["learned"], phase_kernels, ALLOCATING["learned"]),
           "batch": (lambda lib, g: g.batch(), lambda lib, g: None, lambda lib, g: batch_shape(lib, g, 2)),
           "single": (lambda lib, g: g.batch(1), lambda lib, g: None, batch_shape),
           "one_workgroup": (one_workgroup, lambda lib, g: None, one_workgroup),
           "traced": (traced, lambda lib, g: None, traced)}


@pytest.mark.parametrize("name", list(WITHOUT))
@pytest.mark.parametrize("held", [False, True])
def test_no_memory_for_resident_scratch_is_no_refusal(lib, name, held):
    """With the memory that the other kernels need and no more, and (held) with scratch on the handle from
    an earlier resident solve: the call is served by them."""
    call, choose, other = WITHOUT[name]
    lib.host_reset(1 << 40)
    lib.sssp_graph_destroy(None)
    g = Host(lib, 4000, 9000)
    choose(lib, g)
    lib.host_reset(1 << 40)
    expect, need = other(lib, g), lib.host_peak()
    g.close()
    assert expect in (OK, INTERNAL) and need > 0
    g = Host(lib, 4000, 9000)
    base = lib.host_used()
    if held:
        assert g.solve() == OK
        assert lib.host_used() > base
    lib.host_reset(base + need)
    rc = call(lib, g)
    assert rc != OOM, g.message()
    if name in (("one_workgroup", "traced", "batch") if held else ("simple", "learned", "batch", "single")):
        assert "oom" in g.log()
    assert rc == expect or name in ("static", "simple", "delta", "learned"), (rc, g.message())
    lib.host_reset(1 << 40)
    g.close()


@pytest.mark.parametrize("what", ["staging", "event"])
def test_failed_creation_waits_before_its_block_is_kept(lib, what):
    """Creation that fails after work was queued on its block: the block may serve the next graph, on
    another stream, so that work has to be over."""
    lib.host_reset(1 << 40)
    lib.sssp_graph_destroy(None)
    n, m = 1 << 20, 6 << 20
    base = lib.host_used()
    whole = Host(lib, n, m)
    block = lib.host_used() - base
    whole.close()
    lib.sssp_graph_destroy(None)
    lib.host_reset(lib.host_used() + block + (MiB if what == "staging" else 1 << 30))
    lib.host_fail_events(1 if what == "event" else 0)
    failed = Host(lib, n, m)
    assert failed.rc == (OOM if what == "staging" else DEVICE)
    log = failed.log()
    queued = max(i for i, x in enumerate(log) if x in ("set", "kernel"))
    assert "wait" in log[queued:], log
    lib.host_reset(1 << 40)
    lib.sssp_graph_destroy(None)


@pytest.mark.parametrize("name", list(SOLVES))
def test_launch_that_does_not_fit_falls_back(lib, name):
    """The device cannot hold the workgroups at once (error 720): the other kernels are launched. Here they
    do nothing, so that all but the batch end in their phase bound."""
    g = Host(lib)
    lib.host_reset(1 << 40)
    lib.host_coop(720, 0, 0, 0)
    rc = SOLVES[name](g)
    assert rc == (OK if name == "batch" else INTERNAL), g.message()
    assert "terminate" in g.message() or rc == OK
    assert "kernel" in g.log()[g.log().index("coop"):]
    lib.host_reset(1 << 40)
    form = ctypes.c_uint32(9)
    assert lib.sssp_last_form(g.h, ctypes.byref(form)) == OK and form.value == (3 if name == "batch" else 0)
    g.close()
