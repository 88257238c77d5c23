"""The library's host code under failures that a GPU run cannot bring about at
will: a device allocation that fails in the middle of a call, and the calls
after it.  The library's sources are compiled for the host only and linked with
tests/host_runtime/fake_hip.hip, whose kernels are recorded and do nothing, so
this runs without a GPU and checks no numbers."""
import ctypes
import os
import re
import subprocess
import threading
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

from conftest import ROOT
from paper_2605_07391_amd import build as hipbuild
from paper_2605_07391_amd import merbit as mb

vp = ctypes.c_void_p
N = 300


@pytest.fixture(scope="session")
def lib(tmp_path_factory):
    """The library on the fake runtime."""
    out = tmp_path_factory.mktemp("host_runtime")
    flags = [f for f in hipbuild.FLAGS if f.startswith(("--offload-arch", "-std", "-fPIC", "-I"))]
    sources = [os.path.join(hipbuild.CSRC, s) for s in hipbuild.SOURCES]
    sources.append(os.path.join(ROOT, "tests", "host_runtime", "fake_hip.hip"))

    def compile_(src):
        obj = str(out / (os.path.basename(src) + ".o"))
        subprocess.run([hipbuild.HIPCC, *flags, "-O0", "--offload-host-only", "-w",
                        f"-I{hipbuild.CSRC}", "-c", src, "-o", obj], check=True)
        return obj

    with ThreadPoolExecutor(8) as pool:
        objs = list(pool.map(compile_, sources))
    # the device code that a host-only object refers to does not exist
    names = subprocess.run(["nm", "-u", *objs], check=True, capture_output=True, text=True).stdout
    stub = out / "fatbin.c"
    stub.write_text("".join(f"char {n}[8];\n" for n in
                            sorted(set(re.findall(r"\b__hip_fatbin_\w+", names)))))
    so = str(out / "libmerbit_host.so")
    wrap = ["_ZN6merbit15dev_alloc_bytesEPPvm", "_ZN6merbit8dev_freeEPv",
            "_ZN6merbit14dev_free_afterE10hipError_tPv"]
    subprocess.run(["g++", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-Wl,-z,defs",
                    *[f"-Wl,--wrap={w}" for w in wrap], "-o", so, str(stub), *objs, "-lpthread"],
                   check=True)
    lib = ctypes.CDLL(so)
    lib.fake_log.restype = ctypes.c_char_p
    lib.fake_device_bytes.argtypes = [ctypes.c_size_t]
    lib.fake_live_bytes.restype = ctypes.c_size_t
    for f in ("fake_mallocs", "fake_frees", "fake_early_frees", "fake_held",
              "fake_gate_timeouts", "fake_gate_waiting"):
        getattr(lib, f).restype = ctypes.c_long
    lib.fake_fail_new.argtypes, lib.fake_fail_new.restype = [ctypes.c_long], ctypes.c_long
    lib.fake_capture.argtypes = [vp, ctypes.c_int]
    lib.fake_spmv_y.restype = vp
    lib.merbit_release_memory.restype = ctypes.c_int64
    lib.merbit_last_error.restype = ctypes.c_char_p
    lib.merbit_plan_destroy.restype = None
    return lib


def _csr(n=N, per_row=3):
    rp = (np.arange(n + 1) * per_row).astype(np.int32)
    col = (np.arange(n * per_row) * 7 % n).astype(np.int32)
    return rp, col, np.ones(len(col), np.float32)


def _p(a):
    return vp(a.ctypes.data)


class HostPlan:
    def __init__(self, lib, n=N, per_row=3, **kw):
        self.lib, self.n = lib, n
        self.keep = _csr(n, per_row)
        rp, col, val = self.keep
        o = mb.Opts()
        lib.merbit_opts_init(ctypes.byref(o))
        for k, v in {"hot_columns": 0, "validate": 0, "eager_loops": 1, **kw}.items():
            setattr(o, k, v)
        self.h = vp()
        i64 = ctypes.c_int64
        self.rc = lib.merbit_plan_create(i64(n), i64(n), i64(len(col)), _p(rp), _p(col), _p(val),
                                         0, ctypes.byref(o), None, ctypes.byref(self.h))

    def close(self):
        self.lib.merbit_plan_destroy(self.h)
        self.h = vp()


def _launches(lib, call):
    """(return code, [(kernel, what its line says of it)]) of one call."""
    lib.fake_reset_log()
    rc = call()
    lines = lib.fake_log().decode().splitlines()
    return rc, [tuple(x.split(" null:")) for x in lines]


def _pagerank(lib, plan, x):
    return lib.merbit_pagerank(plan.h, ctypes.c_double(0.85), ctypes.c_double(0.0), 3, 10, _p(x),
                               None, None, None)


# ------------------------------------------ calls after a failed one --

@pytest.mark.parametrize("fault", ["first allocation", "second allocation", "synchronisation"])
def test_dangling_mask_is_not_kept_unless_it_was_built(lib, fault):
    """The mask of the dangling vertices is shared by all later calls: a call
    that fails before its kernels have run must not leave it behind."""
    plan = HostPlan(lib)
    assert plan.rc == mb.OK
    x = np.ones(N, np.float32)
    if fault == "synchronisation":
        lib.fake_fail_sync(1)
    else:
        lib.fake_fail_alloc(1 if fault == "first allocation" else 2)
    rc, _ = _launches(lib, lambda: _pagerank(lib, plan, x))
    assert rc == (mb.EHIP if fault == "synchronisation" else mb.ENOMEM)
    rc, run = _launches(lib, lambda: _pagerank(lib, plan, x))
    assert rc == mb.OK
    assert "pack_dangling_kernel" in [k for k, _ in run], run
    rc, run = _launches(lib, lambda: _pagerank(lib, plan, x))  # once built it is kept
    assert rc == mb.OK and "pack_dangling_kernel" not in [k for k, _ in run]
    plan.close()


def _check_calls_after_failures(lib, call, before=None):
    """Fail each device allocation of `call` in turn on a new plan (which
    `before` has used): the call reports it, and the calls after it, `call` or
    `before` first, succeed and give every kernel the operands that it has on a
    plan which saw no failure."""
    good = {}
    plan = HostPlan(lib)
    for c in [before, call] if before else [call]:
        rc, run = _launches(lib, lambda: c(plan))
        assert rc == mb.OK
        good[c] = set(run)
    plan.close()
    failures = 0
    for nth in range(1, 40):
        for then in ([call, before], [before, call]) if before else ([call],):
            plan = HostPlan(lib)
            if before:
                assert before(plan) == mb.OK
            lib.fake_fail_alloc(nth)
            rc = call(plan)
            lib.fake_fail_alloc(0)
            if rc == mb.OK:  # fewer allocations than that
                plan.close()
                return failures
            assert rc == mb.ENOMEM, lib.merbit_last_error()
            for c in then:
                rc, run = _launches(lib, lambda: c(plan))
                assert rc == mb.OK, lib.merbit_last_error()
                assert set(run) <= good[c], (nth, set(run) - good[c])
            plan.close()
        failures += 1


def test_pagerank_after_a_failed_allocation(lib):
    x = np.ones(N, np.float32)
    n = _check_calls_after_failures(lib, lambda plan: _pagerank(lib, plan, x))
    assert n == 7  # the mask and its work space, three vectors, two pair arrays
def _pagerank_personalized(lib, plan, x, k):
    src = (np.arange(k) % plan.n).astype(np.int32)
    return lib.merbit_pagerank_personalized(plan.h, ctypes.c_double(0.85), ctypes.c_double(0.0), 3,
                                            10, _p(src), k, _p(x), None, None, None)


@pytest.mark.parametrize("before_k", [0, 3, 40], ids=["new plan", "after k=3", "after k=40"])
@pytest.mark.parametrize("k", [5, 64])
def test_personalized_pagerank_after_a_failed_allocation(lib, k, before_k):
    """Also with buffers of another width on the plan, and with a call of that
    width after the failed one."""
    x = np.ones((N, 64), np.float32)

    def ppr(width):
        return lambda plan: _pagerank_personalized(lib, plan, x, width)

    n = _check_calls_after_failures(lib, ppr(k), ppr(before_k) if before_k else None)
    # two or three vectors, and on a new plan the mask and its work space, the
    # parts, two sums and the sources
    assert n == (3 if k == 64 else 2) + (0 if before_k else 6)


@pytest.mark.parametrize("driver", ["pagerank", "multi", "adjoint", "personalized"])
def test_output_buffers_after_a_loop_that_failed(lib, driver):
    """A driver's two output buffers take turns at being zero where the next
    product adds onto them; a call that fails between two chunks of its loop
    leaves that unknown, and the next one clears a buffer first."""
    D = ctypes.c_double
    plan = HostPlan(lib, eager_loops=0)
    x, g = np.ones(N, np.float32), np.ones(N, np.float32)
    gp = np.array([0, 100, N], np.int64)
    src, X = np.zeros(3, np.int32), np.ones((N, 3), np.float32)
    clear = "spmm_zero" if driver == "personalized" else "zero_boundary"

    def call(alpha):
        if driver == "personalized":
            return lib.merbit_pagerank_personalized(plan.h, D(alpha), D(0.0), 25, 5, _p(src), 3,
                                                    _p(X), None, None, None)
        if driver == "pagerank":
            return lib.merbit_pagerank(plan.h, D(alpha), D(0.0), 25, 5, _p(x), None, None, None)
        if driver == "multi":
            return lib.merbit_pagerank_multi(plan.h, _p(gp), 2, D(alpha), D(0.0), 25, 5, _p(x),
                                             None, None, None)
        return lib.merbit_pagerank_adjoint(plan.h, plan.h, D(alpha), D(0.0), 25, 5, _p(g), _p(x),
                                           None, None, None)

    assert call(0.85) == mb.OK
    rc, run = _launches(lib, lambda: call(0.85))
    assert rc == mb.OK and not any(k.startswith(clear) for k, _ in run)
    lib.fake_fail_graph(2)
    assert call(0.5) == mb.ENOMEM  # the second chunk, after one of 5 steps
    rc, run = _launches(lib, lambda: call(0.85))
    assert rc == mb.OK and any(k.startswith(clear) for k, _ in run)
    plan.close()


def test_stacked_buffers_after_a_chunk_that_was_not_run(lib):
    """A striped plan's two buffers of the stacked products take turns as well: a
    chunk that was recorded and could not be instantiated has not used them."""
    lib.fake_fill(1)
    plan = HostPlan(lib, stripes=8, eager_loops=0)
    lib.fake_fill(0)
    assert plan.rc == mb.OK
    x, y = np.ones(N, np.float32), np.ones(N, np.float32)

    def buffer():
        assert lib.merbit_spmv(plan.h, _p(x), _p(y), None) == mb.OK
        return lib.fake_spmv_y()

    first, second = buffer(), buffer()
    assert first != second
    lib.fake_fail_graph(1)
    assert lib.merbit_pagerank(plan.h, ctypes.c_double(0.85), ctypes.c_double(0.0), 5, 5, _p(x),
                               None, None, None) == mb.ENOMEM
    assert buffer() == first
    plan.close()


def _tune(lib):
    rp, col, val = _csr()
    o = mb.Opts()
    lib.merbit_opts_init(ctypes.byref(o))
    i64 = ctypes.c_int64
    return lib.merbit_tune(i64(N), i64(N), i64(len(col)), _p(rp), _p(col), _p(val), 0, None, 0,
                           None, 0, 2, ctypes.byref(o), None, None)


# ------------------------------------------------- memory and pending work --

@pytest.mark.parametrize("call", ["pagerank", "tune"])
def test_host_memory_runs_out_during_a_call(lib, call):
    """No device memory is lost to a host allocation that fails."""
    x = np.ones(N, np.float32)
    held = lib.fake_held()
    for nth in range(1, 300):
        plan = HostPlan(lib)
        lib.fake_fail_new(nth)
        rc = _pagerank(lib, plan, x) if call == "pagerank" else _tune(lib)
        came = lib.fake_fail_new(0) == 0
        plan.close()
        assert lib.fake_held() == held, nth
        assert rc in (mb.OK, mb.ENOMEM) if came else rc == mb.OK
        if not came:  # fewer host allocations than that
            break
    assert not came and nth > 5

def test_host_memory_runs_out_during_a_striped_build(lib):
    """The build's temporaries go back while an exception unwinds it: only
    after its queued work, and all of them."""
    lib.fake_fill(1)  # one (stripe, row) pair and one more: a plan of two rows
    failures = 0
    for nth in range(1, 400):
        held, early = lib.fake_held(), lib.fake_early_frees()
        lib.fake_fail_new(nth)
        plan = HostPlan(lib, stripes=8, hot_columns=-1)
        if lib.fake_fail_new(0) > 0:  # fewer host allocations than that
            break
        failures += plan.rc == mb.ENOMEM
        plan.close()
        assert lib.fake_early_frees() == early, nth
        assert lib.fake_held() == held, nth
    lib.fake_fill(0)
    assert failures >= 20


@pytest.mark.parametrize("call", ["plan_create", "transpose"])
def test_calls_that_allocate_are_refused_under_capture(lib, call):
    """While a stream is captured hipMalloc is refused, and with it every call
    that needs memory -- also where a kept block would do: its kernels would
    only be recorded, and the recording would outlive the block."""
    rp_t, col_t, perm = np.zeros(N + 1, np.int32), np.zeros(3 * N, np.int32), np.zeros(3 * N, np.int32)

    def transpose(plan):
        return lib.merbit_transpose(plan.h, _p(rp_t), _p(col_t), _p(perm), None)

    plan = HostPlan(lib)
    assert transpose(plan) == mb.OK
    HostPlan(lib).close()  # blocks of every size are kept now
    held = lib.fake_held()
    lib.fake_capture(None, 1)
    if call == "plan_create":
        again = HostPlan(lib)
        rc, launched = again.rc, bool(again.h)
    else:
        rc, run = _launches(lib, lambda: transpose(plan))
        launched = bool(run)
    lib.fake_capture(None, 0)
    assert rc == mb.EHIP and not launched
    assert lib.fake_held() == held
    assert transpose(plan) == mb.OK
    plan.close()


@pytest.mark.parametrize("call", ["plan_destroy", "transpose", "dangling mask", "tune"])
def test_blocks_whose_work_was_not_waited_for_are_not_reused(lib, call):
    """A wait that fails (or is refused, under capture) leaves work pending:
    the blocks it uses go back to the device and not to the next caller."""
    x = np.ones(N, np.float32)
    rp_t, col_t, perm = np.zeros(N + 1, np.int32), np.zeros(3 * N, np.int32), np.zeros(3 * N, np.int32)
    plan = HostPlan(lib)
    early, frees = lib.fake_early_frees(), lib.fake_frees()
    if call == "plan_destroy":
        assert lib.merbit_spmv(plan.h, _p(x), _p(np.ones(N, np.float32)), None) == mb.OK
        lib.fake_fail_sync(1)
        plan.close()
    elif call == "transpose":
        lib.fake_fail_sync(1)
        lib.merbit_transpose(plan.h, _p(rp_t), _p(col_t), _p(perm), None)
    elif call == "dangling mask":
        lib.fake_fail_sync(1)
        assert _pagerank(lib, plan, x) == mb.EHIP
    else:
        lib.fake_fail_sync(1)
        _tune(lib)
    assert lib.fake_early_frees() == early
    assert lib.fake_frees() > frees
    lib.fake_fail_sync(0)
    plan.close()


MIB = 1 << 20


def _solve(lib, n):
    """A plan of n rows without nonzeros and one solver call: 8 vectors."""
    plan = HostPlan(lib, n=n, per_row=0)
    b = x = np.empty(n, np.float32)
    lib.merbit_bicgstab(plan.h, _p(b), vp(x.ctypes.data + 4), ctypes.c_double(0.0), 0, 1, None,
                        None, None)
    plan.close()


def test_kept_memory_is_bounded_and_ages(lib):
    lib.merbit_release_memory()
    base = lib.fake_live_bytes()
    _solve(lib, 20_000_000)  # 8 x 80 MB
    kept = lib.fake_live_bytes() - base
    assert 256 * MIB < kept <= 512 * MIB
    for _ in range(60):  # over 512 allocations and frees that cannot use those blocks
        HostPlan(lib).close()
    assert lib.fake_live_bytes() - base < MIB


def test_kept_memory_goes_back_when_an_allocation_fails_and_on_request(lib):
    lib.merbit_release_memory()
    base = lib.fake_live_bytes()
    _solve(lib, 10_000_000)
    kept = lib.fake_live_bytes() - base
    assert kept > 256 * MIB
    # a plan whose vectors fit only without the kept ones, which are too small
    lib.fake_device_bytes(base + kept + 64 * MIB)
    plan = HostPlan(lib, n=15_000_000, per_row=0)
    assert plan.rc == mb.OK
    x = np.empty(15_000_000, np.float32)
    assert _pagerank(lib, plan, x) == mb.OK
    lib.fake_device_bytes(1 << 40)
    plan.close()
    kept = lib.fake_live_bytes() - base
    assert kept > 0 and lib.merbit_release_memory() == kept
    assert lib.fake_live_bytes() == base and lib.merbit_release_memory() == 0


def test_other_threads_go_on_while_memory_goes_back(lib):
    """hipFree waits for the device: not with the lock that every allocation
    takes."""
    HostPlan(lib).close()
    timeouts, waiting = lib.fake_gate_timeouts(), lib.fake_gate_waiting()
    lib.fake_gate(1)
    releasing = threading.Thread(target=lib.merbit_release_memory)
    releasing.start()
    while lib.fake_gate_waiting() == waiting:
        assert releasing.is_alive()
    plan = HostPlan(lib)  # needs the lock; hipFree is still waiting
    lib.fake_gate(0)
    releasing.join()
    assert plan.rc == mb.OK and lib.fake_gate_timeouts() == timeouts
    plan.close()


# ------------------------------------------------------------ launch shape --

def _launch_shape(lib, plan):
    x, y = np.ones(plan.n, np.float32), np.ones(plan.n, np.float32)
    rc, run = _launches(lib, lambda: lib.merbit_spmv(plan.h, _p(x), _p(y), None))
    assert rc == mb.OK
    last = [what for k, what in run if k.startswith("spmv")][-1]
    return tuple(int(v) for v in re.search(r"block: (\d+) grid: (\d+)", last).groups())


@pytest.mark.parametrize("options,shape", [
    (dict(blocks_per_cu=1), (1024, 256)),
    (dict(blocks_per_cu=1, desc_bits=64, sigma=16), (512, 256)),
    (dict(blocks_per_cu=1, block_lanes=256), (256, 256)),
    (dict(), (256, 4 * 256)),
], ids=["default lanes", "default lanes, 64 bits", "256 lanes", "no limit"])
def test_blocks_per_cu_counts_blocks_of_the_plans_size(lib, options, shape):
    """One resident block per CU is one of block_lanes (of its default when not
    given), on a plan with more tiles than the 256 CUs can hold."""
    plan = HostPlan(lib, n=3_000_000, per_row=1, **options)
    assert plan.rc == mb.OK
    assert _launch_shape(lib, plan) == shape
    plan.close()


@pytest.mark.parametrize("options", [dict(), dict(blocks_per_cu=1), dict(block_lanes=512),
                                     dict(desc_bits=64, sigma=16), dict(commit=1)],
                         ids=["default", "limit", "512 lanes", "64 bits", "block commit"])
def test_plan_info_describes_the_launch(lib, options):
    plan = HostPlan(lib, n=100_000, **options)
    info = mb.PlanInfo()
    assert lib.merbit_plan_info(plan.h, ctypes.byref(info)) == mb.OK
    assert (info.block_lanes, info.grid) == _launch_shape(lib, plan)
    # one FP32 value per merge-path step of the block, and the kernel's few words
    assert 0 <= info.lds_bytes - 4 * info.block_lanes * info.sigma <= 64 + 4 * 33
    plan.close()
