"""The host driver (spff_api.cpp) against a stand-in device: launch plans,
step queues and blocks of ticks, without a GPU."""

import ctypes
import os
import shutil
import subprocess

import pytest

from paper_2203_16467_amd import spff

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = "/opt/rocm/include"


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    """The driver compiled for the host and linked with tests/fake_device.cpp."""
    cxx = shutil.which("g++")
    if cxx is None or not os.path.exists(os.path.join(ROCM, "hip", "hip_runtime.h")):
        pytest.skip("needs g++ and the HIP headers")
    csrc = os.path.join(ROOT, "paper_2203_16467_amd", "csrc")
    out = str(tmp_path_factory.mktemp("driver") / "driver.so")
    subprocess.run([cxx, "-std=c++17", "-O1", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__", "-I", ROCM, "-I",
                    os.path.join(ROOT, "include"), "-I", csrc, os.path.join(csrc, "spff_api.cpp"),
                    os.path.join(ROOT, "tests", "fake_device.cpp"), "-Wl,-z,defs", "-Wl,-Bsymbolic",
                    "-o", out], check=True)
    L = ctypes.CDLL(out)
    for name, (res, args) in spff._SIGS.items():
        getattr(L, name).restype, getattr(L, name).argtypes = res, args
    return L


class Handle:
    """A handle of the driver over host memory."""

    def __init__(self, L, B=1, **kw):
        L.fake_reset()
        self.L, self.B, self.cfg = L, B, spff.default_config(**kw)
        n = ctypes.c_size_t()
        assert L.spff_workspace_bytes(ctypes.byref(self.cfg), B, ctypes.byref(n)) == 0
        self.mem = ctypes.create_string_buffer(n.value + 512)
        ws = (ctypes.addressof(self.mem) + 255) // 256 * 256
        self.h = ctypes.c_void_p()
        assert L.spff_create_batch(ctypes.byref(self.cfg), B, ctypes.c_void_p(ws), None, ctypes.c_void_p(ws), n.value,
                                   None, ctypes.byref(self.h)) == 0

    def need(self, *ticks):
        self.L.fake_need(len(ticks), (ctypes.c_int * len(ticks))(*ticks))

    def counts(self):
        c = (ctypes.c_int * 3)()
        self.L.fake_counts(c)
        return list(c)

    def sequence(self, K):
        stats = (spff.StepStats * (self.B * K))()
        st = self.L.spff_run_sequence(self.h, K, (ctypes.c_double * (3 * self.B * K))(), stats)
        return st, [[stats[b * K + k].to_dict() for k in range(K)] for b in range(self.B)]

    def close(self):
        self.L.spff_destroy_problem(self.h)


def test_step_records_survive_a_failed_allocation(driver):
    """The pinned staging of step records grows with the queue.  If its
    allocation fails the call reports it, and a later queue no longer than
    an earlier one works."""
    p = Handle(driver, 2)
    p.need(3, 5)
    assert p.sequence(2)[0] == 0
    driver.fake_fail_alloc(1)
    assert p.sequence(6)[0] == spff.E_DEVICE
    st, s = p.sequence(2)
    assert st == 0 and [[x["ticks"] for x in row] for row in s] == [[3, 3], [5, 5]]
    st, s = p.sequence(6)
    assert st == 0 and [len(row) for row in s] == [6, 6] and s[1][5]["ticks"] == 5
    p.close()


@pytest.mark.parametrize("nx,ny,B", [(512, 512, 1), (256, 128, 8), (64, 1024, 3), (1024, 64, 1), (32, 32, 2)])
@pytest.mark.parametrize("precision", [spff.FP32, spff.FP64])
def test_installing_the_reported_plan_changes_nothing(driver, nx, ny, B, precision):
    """The plan that a handle reports, given back, leaves the geometry that
    it launches as it was; any other LDS plan is launched as it says, and
    removing the plan restores the built-in geometry."""
    p = Handle(driver, B, nx=nx, ny=ny, precision=precision)

    def launched():
        g = (ctypes.c_int * 6)()
        p.sequence(1)
        driver.fake_geom(g)
        return list(g)

    count = ctypes.c_int32()
    driver.spff_plan_buckets(p.h, ctypes.byref(count), None)
    last = count.value - 1
    built_in = launched()
    if precision == spff.FP64 and nx == ny == 512:
        assert built_in[0] and built_in[3]  # register kernels
    plan = spff.Plan()
    assert driver.spff_get_plan(p.h, last, ctypes.byref(plan)) == 0
    assert driver.spff_set_plan(p.h, last, ctypes.byref(plan)) == 0
    assert launched() == built_in
    other = spff.Plan.from_dict(dict(row_kind=spff.FFT_LDS, rows=1, row_threads=128, col_kind=spff.FFT_LDS, cols=1,
                                     col_threads=128))
    assert driver.spff_set_plan(p.h, last, ctypes.byref(other)) == 0
    assert launched() == [0, 1, 128, 0, 1, 128]
    assert driver.spff_set_plan(p.h, last, None) == 0
    assert launched() == built_in
    p.close()


@pytest.mark.parametrize("K", [1, 2, 4, 8, 12, 16, 64])
def test_static_step_checks_no_oftener_than_its_blocks(driver, K):
    """A phase-field solve ends with a tick that finds it converged, so a
    step whose other ticks fill m blocks of ticks_per_sync takes one tick
    more.  It must not cost a block: the static step checks m times (once
    more where it splits a long second block), and enqueues no tick beyond
    the blocks."""
    for m in (1, 2, 3, 7):
        T = m * K + 1
        driver.fake_reset()
        driver.fake_need(1, (ctypes.c_int * 1)(T))
        cfg = spff.default_config(nx=16, ny=16, ticks_per_sync=K)
        buf = ctypes.create_string_buffer(16 * 16 * 4 * 6)
        stats, c = spff.StepStats(), (ctypes.c_int * 3)()
        assert driver.spff_load_step_static(ctypes.byref(cfg), buf, ctypes.addressof(buf), (ctypes.c_double * 3)(),
                                            ctypes.byref(stats), None) == 0
        driver.fake_counts(c)
        checks, rows, cols = c[0] - 2, c[1], c[2]  # two synchronisations of uploads
        assert stats.ticks == T
        assert checks <= m + (K >= 16 and m > 1), (m, checks)
        assert cols == T and rows == T + 1


def test_memory_that_kernels_post_to_is_coherent(driver):
    """The progress words are read while the kernel that posts them runs, so
    the pinned memory asks for coherence (0x40000000, hipHostMallocCoherent)
    instead of relying on the process's default."""
    p = Handle(driver, 3)
    assert driver.fake_alloc_flags() & 0x40000000
    p.close()


@pytest.mark.parametrize("nx,ny,B,row,col", [
    (256, 128, 1, 2, 0), (512, 256, 1, 2, 0), (1024, 512, 1, 1, 1), (1024, 256, 1, 0, 1), (64, 1024, 1, 0, 1),
    (512, 512, 5, 2, 1), (512, 512, 8, 1, 1), (256, 256, 9, 2, 1), (256, 256, 32, 1, 1), (128, 128, 128, 1, 1)])
def test_fp64_built_in_kernels(driver, nx, ny, B, row, col):
    """Which kernels FP64 batches run as built in (rows: 0 LDS, 1 eight, 2
    four points per lane; columns: 0 LDS, 1 registers): the sizes at which
    the GPU tests compare them."""
    p = Handle(driver, B, nx=nx, ny=ny, precision=spff.FP64)
    p.need(*[3] * B)
    g = (ctypes.c_int * 6)()
    p.sequence(1)
    driver.fake_geom(g)
    assert [g[0], g[3]] == [row, col]
    p.close()


@pytest.mark.parametrize("nx,ny,B,rows", [(64, 64, 1, 1), (64, 256, 1, 1), (64, 512, 1, 2), (32, 1024, 1, 4),
                                          (64, 2048, 1, 4), (64, 64, 32, 1), (64, 64, 33, 2), (64, 512, 13, 4),
                                          (64, 512, 64, 8), (8, 8, 512, 2), (8, 8, 8192, 8)])
@pytest.mark.parametrize("precision", [spff.FP32, spff.FP64])
def test_short_rows_take_one_wavefront_a_group(driver, nx, ny, B, rows, precision):
    """Rows below 64 pixel pairs: 64 threads a group, at most 256 groups a
    problem and 2048 (with four or more rows a group 4096) in all, up to
    eight rows a group; explicit overrides stand."""
    p = Handle(driver, B, nx=nx, ny=ny, precision=precision)
    count, plan = ctypes.c_int32(), spff.Plan()
    driver.spff_plan_buckets(p.h, ctypes.byref(count), None)
    assert driver.spff_get_plan(p.h, count.value - 1, ctypes.byref(plan)) == 0
    assert (plan.row_kind, plan.rows, plan.row_threads) == (spff.FFT_LDS, rows, 64)
    p.close()
    p = Handle(driver, 1, nx=nx, ny=ny, precision=precision, plan_rows=2)
    assert driver.spff_get_plan(p.h, 0, ctypes.byref(plan)) == 0
    assert (plan.rows, plan.row_threads) == (2, 256)
    p.close()


@pytest.mark.parametrize("K", [1, 2, 4, 16])
@pytest.mark.parametrize("need", [(6,), (7,), (8,), (15,), (3, 10), (21, 4, 9)])
def test_no_block_runs_after_every_problem_is_idle(driver, K, need):
    """A problem's end is known from the row kernel after its last tick.  The
    driver enqueues no block once that has been seen for every problem; with
    a device that runs each block at once, the row kernels are those of the
    blocks that hold the last end."""
    p = Handle(driver, len(need), ticks_per_sync=K)
    p.need(*need)
    p.counts()
    st, s = p.sequence(1)
    assert st == 0 and [row[0]["ticks"] for row in s] == list(need)
    k = min(K, 4)
    _, rows, cols = p.counts()
    assert rows == cols == -(-(max(need) + 1) // k) * k
    p.close()
