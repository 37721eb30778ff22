"""GPU tests of the outer product where C has few columns or rows repeat them:
buckets summed in LDS accumulators, by pieces and not; long runs of equal columns
in the sorted buckets; rows of which many entries claim places at once. Sums of
small whole numbers, exact in any order."""
from __future__ import annotations

import numpy as np
import pytest

import matgen

pytestmark = pytest.mark.gpu


def _csr(rows, ncols, rng, dtype):
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    ci = np.concatenate(rows).astype(np.int32) if rp[-1] else np.zeros(0, np.int32)
    return matgen.CSR(len(rows), ncols, rp, ci, rng.integers(-3, 4, len(ci)).astype(dtype))


def _outer(A, B):
    import torch
    from paper_2606_20855_amd import wingspan as ws
    print(f"outer: A {A.nrows}x{A.ncols} nnz={A.nnz} B {B.nrows}x{B.ncols} nnz={B.nnz}", flush=True)
    C = ws.spgemm_outer(ws.DeviceCSR.from_host(matgen.transpose(A), "cuda:0"), ws.DeviceCSR.from_host(B, "cuda:0"))
    torch.cuda.synchronize()
    return C.to_host()


def _check(A, B):
    got = _outer(A, B)
    for i in range(A.nrows):
        k, a = A.row(i)
        cols, sums = np.zeros(0, np.int64), np.zeros(0)
        if len(k):
            c = np.concatenate([B.row(j)[0] for j in k]).astype(np.int64)
            p = np.concatenate([float(x) * B.row(j)[1].astype(np.float64) for j, x in zip(k, a)])
            cols, inv = np.unique(c, return_inverse=True)
            sums = np.bincount(inv, p, len(cols))
        lo, hi = got.row_ptr[i], got.row_ptr[i + 1]
        assert np.array_equal(got.col_idx[lo:hi], cols), f"row {i}"
        assert np.array_equal(got.val[lo:hi], sums), f"row {i}"


# C's columns: the least, around a window of 4096 and two of them, the last number summed by pieces and the first sorted
@pytest.mark.parametrize("n", [1, 2, 33, 300, 4095, 4096, 4097, 8192, 8193, 20_000, 65_536, 65_537])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_bucket_lengths(n, dtype):
    rng = np.random.default_rng(n)
    wide = min(50, n)
    fill = [np.sort(rng.choice(n, wide, replace=False)) for _ in range(80_000 // wide if wide < 50 else 1600)]
    fill += [np.arange(wide), n - wide + np.arange(wide)] * 20
    one = [np.array([n // 2])] * 9000                       # rows of one entry, all in one column
    ends = [np.array([0]), np.array([n - 1]), np.zeros(0, np.int64)] * 100
    B = _csr(fill + one + ends, n, rng, dtype)
    nf, no = len(fill), len(one)
    rows = []
    # around the buckets' sizes, a piece of 8192 places, and C's columns
    for want in [0, 32, 256, 257, 4095, 4096, 4097, 8191, 8192, 8193, 12_289, 40_000, n - 1, n, n + 1]:
        picks = rng.permutation(nf)[:min(want // wide, nf)]
        left = want - len(picks) * wide
        rows.append(np.sort(np.concatenate([picks, nf + rng.choice(no, min(left, no), replace=False)])))
    # one column alone: in a wave's registers, in LDS, past it
    for want in [17, 33, 64, 65, 200, 256, 2000, 4096, 4097, 9000]:
        rows.append(np.sort(nf + rng.choice(no, want, replace=False)))
    rows.append(np.arange(B.nrows))
    A = _csr(rows, B.nrows, rng, dtype)
    _check(A, B)


def test_runs_of_equal_columns():
    # runs of 1 to 120 equal columns in sorted buckets, which cross lanes, registers, waves and blocks of the scans
    rng = np.random.default_rng(5)
    n = 100_000
    cols = [np.full(1, c) for c in rng.choice(n, 400, replace=False) for _ in range(rng.integers(1, 121))]
    B = _csr(cols, n, rng, np.float64)
    rows = [np.sort(rng.choice(B.nrows, want, replace=False))
            for want in (40, 64, 100, 128, 180, 256, 300, 1000, 2500, 4096, 4097, 10_000)] + [np.arange(B.nrows)]
    # runs that end with the bucket, and one run over all of it
    rows += [np.arange(k) for k in (60, 120, 250, 1030, 4090, 4200)]
    _check(_csr(rows, B.nrows, rng, np.float64), B)


def test_sorted_buckets_of_many_merge_passes():
    # C of more columns than are summed by pieces: 2 to 42 runs sorted in LDS, one to six merge passes
    rng = np.random.default_rng(6)
    n = 100_000
    B = _csr([np.sort(rng.choice(n, 50, replace=False)) for _ in range(3500)], n, rng, np.float64)
    rows = [np.sort(rng.choice(B.nrows, want, replace=False)) for want in (82, 164, 170, 330, 700, 1400, 3400)]
    _check(_csr(rows, B.nrows, rng, np.float64), B)


@pytest.mark.parametrize("hot", [[0], [7, 2054, 4101], list(range(16)), list(range(0, 40_000, 2048))], ids=len)
def test_rows_claimed_by_many_entries(hot):
    # every index has a few of the hot rows (among them rows of one slot of the claims' table) and one other
    rng = np.random.default_rng(len(hot))
    K, m, n = 30_000, 50_000, 70_000
    at = [np.unique(np.append(rng.choice(hot, min(3, len(hot)), replace=False), rng.integers(m))) for _ in range(K)]
    At = _csr(at, m, rng, np.float64)
    B = _csr([np.unique(rng.integers(0, n, rng.integers(0, 4))) for _ in range(K)], n, rng, np.float64)
    A = matgen.transpose(At)
    got = _outer(A, B)
    import scipy.sparse as sp
    one = [sp.csr_matrix((np.ones(X.nnz), X.col_idx, X.row_ptr), (X.nrows, X.ncols)) for X in (A, B)]
    val = [sp.csr_matrix((X.val, X.col_idx, X.row_ptr), (X.nrows, X.ncols)) for X in (A, B)]
    S = (one[0] @ one[1]).tocsr()
    S.sort_indices()
    assert np.array_equal(got.row_ptr, S.indptr) and np.array_equal(got.col_idx, S.indices)
    C = sp.csr_matrix((got.val, got.col_idx, got.row_ptr), S.shape)
    assert abs(C - val[0] @ val[1]).sum() == 0


# (K indices, C of n x n, entries per row, the columns of index k): a dot product, tall matrices of few columns, of a few
# popular ones, and aggregates of 4000, 1000 and 200 points
SHAPES = {
    "dot": (1_000_000, 1, 1, "spread"),
    "tall 16": (300_000, 16, 4, "spread"),
    "tall 256": (200_000, 256, 6, "popular"),
    "tall 4096": (200_000, 4096, 6, "popular"),
    "aggregates of 4000": (1_000_000, 250, 1, "aggregates"),
    "aggregates of 1000": (1_000_000, 1000, 1, "aggregates"),
    "aggregates of 200": (1_000_000, 5000, 1, "aggregates"),
}


@pytest.mark.parametrize("shape", SHAPES)
def test_a_small_c_costs_what_a_large_one_does(shape):
    # against as many products of 300000 uniformly drawn columns (one workgroup sorting a bucket, one lane summing a
    # run of equal columns and one atomic per entry of a row: 7 to 550 times as long)
    import torch
    from paper_2606_20855_amd import wingspan as ws
    K, n, r, how = SHAPES[shape]
    rng = np.random.default_rng(3)

    def matrix(n, r, how):
        if how == "aggregates":
            cols = np.arange(K)[:, None] * n // K
        elif how == "popular":
            cols = (n ** rng.random((K, r))).astype(np.int64) - 1
        else:
            cols = rng.integers(0, n, (K, r))
        keys = np.unique(np.arange(K)[:, None] * n + cols)
        rp = np.searchsorted(keys, np.arange(K + 1) * n).astype(np.int32)
        return ws.DeviceCSR.from_host(matgen.CSR(K, n, rp, (keys % n).astype(np.int32), np.ones(len(keys))), "cuda:0")

    took, products = [], []
    for T in (matrix(n, r, how), matrix(300_000, r, "spread")):
        best = float("inf")
        for _ in range(6):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            C = ws.spgemm_outer(T, T)
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, e[0].elapsed_time(e[1]))
        took.append(best)
        products.append(float(C.val.sum()))
    print(f"{shape}: {took[0] * 1e3:.0f} us for {products[0]:.0f} products, spread {took[1] * 1e3:.0f} us for "
          f"{products[1]:.0f}")
    assert took[0] < 5 * took[1]


@pytest.mark.parametrize("m", [1000, 5000])
def test_few_rows_are_spread_over_waves(m):
    # buckets of 144 entries, a wave each, against buckets of 9 (64 rows to a workgroup of four waves: 90 us more)
    import torch
    from paper_2606_20855_amd import wingspan as ws
    took = []
    for r in (3, 12):
        T = ws.DeviceCSR.from_host(matgen.er(m, m, r, 91), "cuda:0")
        best = float("inf")
        for _ in range(20):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            ws.spgemm_outer(T, T)
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, e[0].elapsed_time(e[1]))
        took.append(best)
    print(f"{m} rows: {took[0] * 1e3:.0f} us, {took[1] * 1e3:.0f} us")
    assert took[1] < took[0] + 0.075


@pytest.mark.parametrize("m", [1, 3, 4, 5, 63, 64, 65, 1023, 8191, 8192, 16_385, 65_535, 65_536])
def test_rows_of_a_workgroup(m):
    # rows of 9, 36 and 300 products by turns, the last rows included, at every number of rows per workgroup
    rng = np.random.default_rng(m)
    sizes = [9, 36, 300]
    B = _csr([np.sort(rng.choice(5000, s, replace=False)) for s in sizes for _ in range(40)], 5000, rng, np.float64)
    pick = np.arange(m) % 3 * 40 + rng.integers(0, 40, m)
    A = matgen.CSR(m, B.nrows, np.arange(m + 1, dtype=np.int32), pick.astype(np.int32), np.full(m, 2.0))
    got = _outer(A, B)
    lens = np.diff(B.row_ptr)[pick]
    assert np.array_equal(np.diff(got.row_ptr), lens)
    at = np.repeat(B.row_ptr[pick] - got.row_ptr[:-1], lens) + np.arange(len(got.col_idx))
    assert np.array_equal(got.col_idx, B.col_idx[at]) and np.array_equal(got.val, 2.0 * B.val[at])
