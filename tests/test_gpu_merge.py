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


def pays(f, k, ncols, products):
    """Whether a row of f products from k entries of A is merged rather than hashed (register rows count as merged)."""
    if k > 64:
        return False
    lg = lambda x: max(0, int(x - 1).bit_length())
    places = f + (7 if products else 15) * k
    lm = max(8, lg(places))
    if products:
        l = lg(f + f // 2)
        same = max(9 if f > 128 else 8, l)
        if f > 128 and ncols > 512 << l:
            return lm <= same + 1
        return lm <= same and (lm < 11 or 20 * places <= 27 * f)
    return lm <= max(8, lg(2 * f)) and 4 * places <= 9 * f and (lm < 11 or lm <= lg(f) or 4 * places <= 5 * f)


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
    # (hashed rows, longer ones and rows of more A entries sum with LDS atomics, in any order)
    again, _, _ = run_gpu(A, B)
    count = np.diff(ref.row_ptr)
    merged = np.array([pays(int(f), int(k), ncols, True) for f, k in zip(ref.products, np.diff(A.row_ptr))])
    light = np.repeat(merged & (count < 2048) & (ref.products <= 4096), count)
    assert light.sum() > 1000
    assert np.array_equal(again.val[light], got.val[light])
    import torch
    from paper_2606_20855_amd import wingspan as ws
    dA, dB = ws.DeviceCSR.from_host(A, "cuda:0"), ws.DeviceCSR.from_host(B, "cuda:0")
    S = ws.spgemm_sharded(dA, dB)
    C = ws.sharded_to_csr(S)
    torch.cuda.synchronize()
    assert_matches(C.to_host(), ref, A.val.dtype, what="single pass")


# both sides of every line of the rule: runs too short at each size, the small sizes, the sorted table's products, the
# wide C's extra size, the padding allowed from 2048 places on
@pytest.mark.parametrize("k,L", [(64, 2), (64, 3), (64, 6), (64, 12), (64, 17), (64, 20), (64, 24), (48, 2), (48, 3),
                                 (48, 4), (48, 6), (48, 8), (40, 20), (32, 3), (32, 4), (32, 6), (32, 12), (32, 16),
                                 (16, 8), (16, 9), (16, 12), (16, 64), (12, 6), (12, 10), (8, 9), (8, 12), (8, 15),
                                 (8, 17), (8, 128), (2, 33), (2, 240), (1, 100)])
@pytest.mark.parametrize("ncols", [100_000, 400_000, 1_000_000])
def test_short_runs_are_hashed(k, L, ncols):
    A = matgen.er(50, 600, k, seed=k, dtype=np.float32, dist="open01")
    B = matgen.er(600, ncols, L, seed=L, dtype=np.float32, dist="open01")
    ref = oracle.spgemm(A, B)
    for opts in (None, dict(max_lds_slots=16384)):
        got, sym, num = run_gpu(A, B, opts)
        assert_matches(got, ref, A.val.dtype, what=f"{k} x {L} {opts}")
        # (counted rows of 1024 products are the bitmap kernel's at 100 K columns, of 2048 of either kind the dense tier's)
        if opts is None and k * L < 1024:
            assert num["merged_rows"] == (50 if pays(k * L, k, ncols, True) else 0)
            assert sym["merged_rows"] == (50 if pays(k * L, k, ncols, False) else 0)
    import torch
    from paper_2606_20855_amd import wingspan as ws
    dA, dB = ws.DeviceCSR.from_host(A, "cuda:0"), ws.DeviceCSR.from_host(B, "cuda:0")
    C = ws.sharded_to_csr(ws.spgemm_sharded(dA, dB))
    torch.cuda.synchronize()
    assert_matches(C.to_host(), ref, A.val.dtype, what=f"{k} x {L} single pass")


@pytest.mark.parametrize("k,L", [(64, 2), (40, 2), (64, 4), (48, 12), (16, 32)])
def test_merging_costs_no_more_than_hashing(k, L):
    # kernel times of a hundred thousand rows and more, as the options divide them (merging every row: up to six times)
    import torch
    from paper_2606_20855_amd import wingspan as ws
    m = 16_000_000 // (k * L)
    A = matgen.er(m, 5000, k, seed=1, dtype=np.float64)
    B = matgen.er(5000, 100_000, L, seed=2, dtype=np.float64)
    dA, dB = ws.DeviceCSR.from_host(A, "cuda:0"), ws.DeviceCSR.from_host(B, "cuda:0")
    best = {}
    for _ in range(5):
        for name, opts in (("rule", {}), ("hash", dict(max_lds_slots=16384))):
            ws.spgemm(dA, dB, options=ws.make_options(timing=1, **opts))
            torch.cuda.synchronize()
            for phase in (0, 1):
                t = ws.wingspan_last_stats(phase)["kernel_ms"]["hash"]
                best[name, phase] = min(t, best.get((name, phase), t))
    print({k: f"{1e3 * v:.0f} us" for k, v in best.items()})
    assert all(best["rule", p] < 1.4 * best["hash", p] for p in (0, 1))
