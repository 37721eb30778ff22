"""GPU tests of the register tier: segments of every width, several rows per
segment, ragged row counts, rows with many empty B rows, runs of equal columns
up to a whole segment, and columns too many for 32-bit sort keys, against a
plain numpy sum of the products in order."""
from __future__ import annotations

import numpy as np
import pytest

import matgen
from gpu_util import run_gpu

pytestmark = pytest.mark.gpu


def _reference(A, B):
    """Row by row: products in the order of A's entries, equal columns added in that order in double."""
    rp, cols, vals = [0], [], []
    for i in range(A.nrows):
        k, a = A.row(i)
        c = np.concatenate([B.row(j)[0] for j in k] + [np.zeros(0, np.int32)]).astype(np.int64)
        p = np.concatenate([float(x) * B.row(j)[1].astype(np.float64) for j, x in zip(k, a)] + [np.zeros(0)])
        u, inv = np.unique(c, return_inverse=True)
        s = np.zeros(len(u))
        np.add.at(s, inv, p)
        cols.append(u)
        vals.append(s)
        rp.append(rp[-1] + len(u))
    return np.array(rp), np.concatenate(cols), np.concatenate(vals).astype(A.val.dtype)


def _matrices(m, ncols, dtype, seed):
    rng = np.random.default_rng(seed)
    # B: empty rows, rows of 1 to 64 columns; every fourth row starts at column 0 (runs of equal columns)
    lens = np.concatenate([np.zeros(100, int), rng.integers(1, 9, 60), rng.integers(9, 65, 30), [64, 32, 16, 8]])
    span = min(ncols, 1 << 40)
    cols = [np.arange(n) if j % 4 == 0 else np.unique(np.concatenate([rng.integers(0, span, 2 * n + 8), [span - 1]]))[-n:]
            if n else np.zeros(0, int) for j, n in enumerate(lens)]
    cols = [np.sort(rng.permutation(c)[:n]) for c, n in zip(cols, lens)]
    bp = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
    B = matgen.CSR(len(lens), ncols, bp, np.concatenate(cols).astype(np.int32), (rng.random(bp[-1]) - 0.5).astype(dtype))
    size = np.diff(bp)
    rows = []
    for i in range(m):
        # entries added while the products stay within 8, 16, 32 or 64; every eighth row takes all the empty B rows
        room = (8, 16, 32, 64)[i % 4]
        r = list(range(100)) if i % 8 == 0 else []
        for j in rng.permutation(np.arange(0 if i % 3 else 100, len(lens))):
            if j not in r and size[r].sum() + size[j] <= room:
                r.append(j)
            if len(r) > 130 or (size[r].sum() == room and rng.random() < 0.5):
                break
        rows.append(np.sort(r))
    rows[m // 2] = np.arange(0)
    ap = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    return matgen.CSR(m, len(lens), ap, np.concatenate(rows).astype(np.int32), (rng.random(ap[-1]) - 0.5).astype(dtype)), B


# 67,108,864 and 2^27 columns on: wider keys for segments of 64 and of 32 lanes; 2^30: for all
@pytest.mark.parametrize("m,ncols", [(37, 500), (301, 100_000), (203, (1 << 26) - 1), (203, 1 << 26), (150, 1 << 27),
                                     (150, (1 << 30) + 5)])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_small_rows(m, ncols, dtype):
    A, B = _matrices(m, ncols, dtype, m + ncols % 97)
    rp, col, val = _reference(A, B)
    got, sym, num = run_gpu(A, B, dict(cache_mib=-1))
    assert num["rows"]["tiny"] == int(np.sum(np.diff(rp) > 0))
    assert np.array_equal(got.row_ptr, rp) and np.array_equal(got.col_idx, col)
    assert np.array_equal(got.val, val)   # the same products added in the same order


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_many_rows(dtype):
    # enough rows of every width for several rows per segment, and not a multiple of them
    A, B = _matrices(400, 9000, dtype, 11)
    rp, col, val = _reference(A, B)
    times = 401
    rows = np.tile(A.col_idx, times)
    ap = np.concatenate([[0], np.cumsum(np.tile(np.diff(A.row_ptr), times))])[: 400 * times - 2].astype(np.int32)
    big = matgen.CSR(len(ap) - 1, A.ncols, ap, rows[: ap[-1]], np.tile(A.val, times)[: ap[-1]])
    got, sym, num = run_gpu(big, B)
    want = np.tile(np.diff(rp), times)[: big.nrows]
    assert np.array_equal(np.diff(got.row_ptr), want)
    n = int(got.row_ptr[-1])
    assert np.array_equal(got.col_idx, np.tile(col, times)[:n])
    assert np.array_equal(got.val, np.tile(val, times)[:n])
