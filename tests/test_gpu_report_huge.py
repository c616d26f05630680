"""The report of an LP whose two products together take more threads than one
launch can have (2^32): 33.6 million rows and columns of 33 entries, 64 lanes
each, 1.1 billion entries.  A is 33 copies of one block of rows, so that numpy
has both products from the block."""
import ctypes as C

import numpy as np
import pytest

from paper_2511_13894_amd import pdhg

pytestmark = pytest.mark.gpu

PER = 33  # entries of a row and of a column, copies of the block
ROWS = 1016802  # rows of the block
M = PER * ROWS  # rows and columns


def _device(hip, ptr, name, size):
    ptr[name] = C.c_void_p()
    assert hip.hipMalloc(C.byref(ptr[name]), C.c_size_t(size)) == 0, name


def _huge_lp(hip, val):
    lp = pdhg.DeviceLP.__new__(pdhg.DeviceLP)
    lp.m = lp.n = M
    lp.nnz = M * PER
    lp.ptr = {}
    col = (np.arange(ROWS, dtype=np.int32)[:, None] + ROWS * np.arange(PER, dtype=np.int32)[None, :]).reshape(-1)
    for name, block in (("col", col), ("val", val.reshape(-1))):  # row i has the columns i mod ROWS + k ROWS
        _device(hip, lp.ptr, name, PER * block.nbytes)
        for k in range(PER):
            dst = C.c_void_p(lp.ptr[name].value + k * block.nbytes)
            src = block.ctypes.data_as(C.c_void_p) if k == 0 else lp.ptr[name]
            assert hip.hipMemcpy(dst, src, C.c_size_t(block.nbytes), 1 if k == 0 else 3) == 0
    inf = np.full(M, np.inf)
    for name, a in (("row_ptr", np.arange(M + 1, dtype=np.int64) * PER), ("b", np.zeros(M)), ("c", np.zeros(M)),
                    ("l", -inf), ("u", inf), ("sense", np.full(M, ord("="), dtype=np.uint8))):
        _device(hip, lp.ptr, name, a.nbytes)
        assert hip.hipMemcpy(lp.ptr[name], a.ctypes.data_as(C.c_void_p), C.c_size_t(a.nbytes), 1) == 0
    return lp


def test_report_past_one_launch_of_threads():
    hip = pdhg._hip_runtime()
    free, total = C.c_size_t(), C.c_size_t()
    assert hip.hipMemGetInfo(C.byref(free), C.byref(total)) == 0
    if free.value < 150 << 30:
        pytest.skip(f"{free.value >> 30} GiB of GPU memory free, about 110 needed")
    rng = np.random.default_rng(3)
    val = rng.integers(1, 9, (ROWS, PER)).astype(np.float64)
    print(f"[huge report] m = n = {M}, nnz = {M * PER}", flush=True)
    lp = _huge_lp(hip, val)
    s = pdhg.Solver(lp, ruiz_iters=1, pc_alpha=-1.0, power_iters=1)
    lp.free()
    print("[huge report] created", flush=True)
    x, y = rng.integers(-4, 5, M).astype(np.float64), rng.integers(-4, 5, M).astype(np.float64)
    k = s.kkt(x, y)
    ax = (val * x.reshape(PER, ROWS).T).sum(axis=1)  # of the block; every copy has the same
    aty = val * y.reshape(PER, ROWS).sum(axis=0)[:, None]
    # integers below 2^53 up to the square root
    assert k.rpinf == np.abs(ax).max() and k.rdinf == np.abs(aty).max()
    assert k.rp2 == pytest.approx(np.sqrt(PER * (ax * ax).sum()), rel=1e-14)
    assert k.rd2 == pytest.approx(np.sqrt((aty * aty).sum()), rel=1e-14)
