"""GPU tests of the merge rows (rows of few A entries, whose B rows are merged
in LDS): run counts and lengths around every edge of the kernel, against the
CPU oracle, through the two phases and through the single pass."""
from __future__ import annotations

import numpy as np
import pytest

import matgen
import oracle
from gpu_util import assert_matches, run_gpu

pytestmark = pytest.mark.gpu


def _b(lengths, ncols, dtype, seed):
    """A B whose row j holds lengths[j] columns: every third row's packed at the start, the others' spread."""
    rng = np.random.default_rng(seed)
    cols = [np.arange(n) if j % 3 == 0 else np.sort(rng.choice(ncols, size=n, replace=False))
            for j, n in enumerate(lengths)]
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    val = (1.0 - rng.random(rp[-1])).astype(dtype) * np.where(rng.random(rp[-1]) < 0.5, -1, 1).astype(dtype)
    return matgen.CSR(len(lengths), ncols, rp, np.concatenate(cols).astype(np.int32), val)


def _a(rows, ncols, dtype, seed):
    rng = np.random.default_rng(seed)
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    ci = np.concatenate([np.sort(r) for r in rows]).astype(np.int32)
    return matgen.CSR(len(rows), ncols, rp, ci, (1.0 - rng.random(len(ci))).astype(dtype))


# lengths of B's rows: empty, around the places a thread takes (4, 8, 16), a wave's 64, and long ones
LENGTHS = [0, 1, 3, 4, 5, 7, 8, 9, 15, 16, 17, 63, 64, 65, 0, 120, 200, 255, 256, 257, 500, 513, 1000, 1024, 2047,
           2500, 4000, 4090, 6000, 8100] + [30] * 70


@pytest.mark.parametrize("ncols", [9000, 400_000, 3_000_000])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_runs(ncols, dtype):
    # one run of every length; pairs whose sum lies around each size of the kernel; 3, 5, 8, 33, 63 .. 65 runs,
    # empty ones among them; the same B row's columns again and again (a row of equal columns per run)
    B = _b(LENGTHS, ncols, dtype, 5)
    n = len(LENGTHS)
    rng = np.random.default_rng(6)
    rows = [[j] for j in range(n)]
    rows += [[15, j] for j in range(n)] + [[0, 14, j] for j in range(16, 30)]
    rows += [[21, 22], [18, 19], [17, 18, 20], [23, 24, 22], [26, 25, 24], [28, 24], [29, 1], [29, 11], [29, 2]]
    rows += [[0, 3, 6, 9, 12]] * 3 + [list(range(30, 30 + k)) for k in (2, 8, 33, 62, 63, 64, 65, 70)]
    rows += [list(rng.choice(n, size=k, replace=False)) for k in (3, 4, 5, 7, 8, 9, 16, 17, 31, 33, 63, 64, 65)]
    rows = [np.unique(r) for r in rows]
    A = _a(rows, n, dtype, 7)
    ref = oracle.spgemm(A, B)
    got, sym, num = run_gpu(A, B)
    assert_matches(got, ref, A.val.dtype, what="two phases")
    # rows of up to 64 products are the register tier's
    assert num["merged_rows"] > 40 and sym["merged_rows"] > 40
    off, _, noff = run_gpu(A, B, dict(tiny_max=-1))
    assert_matches(off, ref, A.val.dtype, what="no register tier")
    # equal columns are summed in the order of A's entries, so a second call gives the same bits: for the merged
    # rows, of at most 64 A entries, fewer than the 2048 entries the dense tier starts at and at most 4096 products
    # (longer ones and rows of more A entries sum with LDS atomics, in any order)
    again, _, _ = run_gpu(A, B)
    count = np.diff(ref.row_ptr)
    light = np.repeat((np.diff(A.row_ptr) <= 64) & (count < 2048) & (ref.products <= 4096), count)
    assert np.array_equal(again.val[light], got.val[light])
    import torch
    from paper_2606_20855_amd import wingspan as ws
    dA, dB = ws.DeviceCSR.from_host(A, "cuda:0"), ws.DeviceCSR.from_host(B, "cuda:0")
    S = ws.spgemm_sharded(dA, dB)
    C = ws.sharded_to_csr(S)
    torch.cuda.synchronize()
    assert_matches(C.to_host(), ref, A.val.dtype, what="single pass")
