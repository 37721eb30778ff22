"""GPU tests of the outer product's row buckets: bucket lengths around every size
of the coalesce, A entries whose B rows are empty, equal columns across a whole
bucket, and columns too many for 32-bit sort keys, against a plain numpy sum."""
from __future__ import annotations

import numpy as np
import pytest

import matgen

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 2, 31, 32, 33, 63, 64, 65, 100, 127, 128, 129, 200, 255, 256, 257, 300, 1000, 4095, 4096, 4097, 9000]


def _matrices(ncols, dtype, seed):
    """Row i's bucket holds LENGTHS[i] entries: rows of B of 1, 7 and 50 columns, spread over all columns, packed at
    the start or at the end, picked to fill it; among them empty ones."""
    rng = np.random.default_rng(seed)
    sizes = [0] * 20 + [1] * 60 + [7] * 400 + [50] * 300
    cols = []
    for j, n in enumerate(sizes):
        if j % 3 == 0:
            cols.append(np.arange(n))
        elif j % 3 == 1:
            cols.append(ncols - n + np.arange(n))
        else:
            cols.append(np.unique(np.concatenate([rng.integers(0, ncols, 3 * n)]))[:n])
    sizes = np.array([len(c) for c in cols])
    bp = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    B = matgen.CSR(len(sizes), ncols, bp, np.concatenate(cols).astype(np.int32), (rng.random(bp[-1]) - 0.5).astype(dtype))
    rows = []
    for want in LENGTHS:
        left, r = want, list(rng.choice(20, size=3, replace=False))
        for j in np.concatenate([rng.permutation(np.nonzero(sizes == s)[0]) for s in (50, 7, 1)]):
            if sizes[j] <= left:
                r.append(j)
                left -= sizes[j]
        assert left == 0, want
        rows.append(np.sort(r))
    ap = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    A = matgen.CSR(len(rows), len(sizes), ap, np.concatenate(rows).astype(np.int32), (rng.random(ap[-1]) - 0.5).astype(dtype))
    return A, B


@pytest.mark.parametrize("ncols", [400, 100_000, (1 << 27) - 1, 1 << 27, (1 << 31) - 2])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_bucket_lengths(ncols, dtype):
    import torch
    from paper_2606_20855_amd import wingspan as ws
    A, B = _matrices(ncols, dtype, 3 + ncols % 11)
    At = ws.DeviceCSR.from_host(matgen.transpose(A), "cuda:0")
    C = ws.spgemm_outer(At, ws.DeviceCSR.from_host(B, "cuda:0"))
    torch.cuda.synchronize()
    got = C.to_host()
    tol = 1e-12 if dtype == np.float64 else 1e-5
    for i in range(A.nrows):
        k, a = A.row(i)
        c = np.concatenate([B.row(j)[0] for j in k]).astype(np.int64)
        p = np.concatenate([float(x) * B.row(j)[1].astype(np.float64) for j, x in zip(k, a)])
        assert len(c) == LENGTHS[i]
        u, inv = np.unique(c, return_inverse=True)
        s, mag = np.zeros(len(u)), np.zeros(len(u))
        np.add.at(s, inv, p)
        np.add.at(mag, inv, np.abs(p))
        lo, hi = got.row_ptr[i], got.row_ptr[i + 1]
        assert np.array_equal(got.col_idx[lo:hi], u), f"row {i}"
        assert np.all(np.abs(got.val[lo:hi].astype(np.float64) - s) <= tol * mag), f"row {i}"
