"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle.

Structure (C.row_ptr, C.col_idx) must match bit for bit; values must lie
within tol * sum_k |A[i,k] B[k,j]| with tol 1e-12 (fp64) and 1e-5 (fp32).
Every tier is exercised on small inputs by routing rows to it with options.
"""
import numpy as np
import pytest

import matgen
import oracle
from gpu_util import assert_matches, golden, gpu_row_products, row_ptr_sha256, run_gpu

pytestmark = pytest.mark.gpu


def check(A, B, options=None, what=""):
    got, sym, num = run_gpu(A, B, options)
    ref = oracle.spgemm(A, B)
    assert_matches(got, ref, A.val.dtype, what=what or str(options))
    assert sym["total_products"] == int(ref.products.sum())
    assert num["c_nnz_total"] == ref.nnz
    # the analysis pass's per-row product counts, row by row (the counts the rows are binned by)
    assert np.array_equal(gpu_row_products(A, B), ref.products), f"{what}: per-row product counts differ"
    return got, sym, num, ref


# ---------------------------------------------------------------------------
# degenerate and ragged shapes
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("shape", [(0, 0, 0), (0, 5, 3), (4, 0, 6), (5, 6, 0), (1, 1, 1), (3, 2, 7)])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_degenerate_shapes(shape, dtype):
    m, k, n = shape
    A = matgen.random_sparse(m, k, 0.7, 1, dtype)
    B = matgen.random_sparse(k, n, 0.7, 2, dtype)
    check(A, B, what=f"shape {shape}")


def test_all_rows_empty():
    A = matgen.random_sparse(50, 40, 0.0, 3)
    B = matgen.random_sparse(40, 30, 0.5, 4)
    got, _, num, _ = check(A, B)
    assert got.row_ptr[-1] == 0


def test_b_rows_empty():
    # A has entries but every B row it selects is empty: no products at all
    A = matgen.random_sparse(30, 40, 0.5, 5)
    B = matgen.random_sparse(40, 30, 0.5, 6, empty_rows=1.0)
    check(A, B)


@pytest.mark.parametrize("shape", [(7, 33, 5), (33, 7, 64), (64, 64, 64), (17, 64, 33), (130, 70, 90)])
@pytest.mark.parametrize("density", [0.1, 0.5, 1.0])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_random_small(shape, density, dtype):
    m, k, n = shape
    A = matgen.random_sparse(m, k, density, m * 7 + k, dtype, empty_rows=0.2)
    B = matgen.random_sparse(k, n, density, n * 5 + k, dtype, empty_rows=0.2)
    check(A, B, what=f"{shape} d={density}")


# ---------------------------------------------------------------------------
# every tier, forced with options
# ---------------------------------------------------------------------------

TIER_OPTS = {
    "default": None,
    "tiny_off": dict(tiny_max=-1),
    "tiny16": dict(tiny_max=16),
    "hash_small": dict(tiny_max=-1, max_lds_slots=256, dense_min_nnz=-1),
    "dense_w1024": dict(tiny_max=-1, max_lds_slots=64, window_cols=1024),
    "dense_w4096": dict(tiny_max=-1, max_lds_slots=64, window_cols=4096),
    "dense_w8192": dict(tiny_max=-1, max_lds_slots=64, window_cols=8192),
    "dense_pref": dict(dense_min_nnz=1, window_cols=1024),
    "dense_rank": dict(tiny_max=-1, max_lds_slots=64),
    "dense_rank_pref": dict(dense_min_nnz=1),
    "spill": dict(tiny_max=-1, force_spill=1),
    "spill_tiny": dict(force_spill=1),
    "validate": dict(validate=1),
}


def tier_inputs(kind, dtype):
    if kind == "rmat":
        A = matgen.rmat(11, 16, seed=7, dtype=dtype, dist="pm1" if dtype == np.float64 else "open01")
        return A, A
    if kind == "er":
        return matgen.er_rect(400, 3000, 2500, 20, seed=8, dtype=dtype)
    raise KeyError(kind)


@pytest.mark.parametrize("opts", list(TIER_OPTS), ids=list(TIER_OPTS))
@pytest.mark.parametrize("kind", ["rmat", "er"])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_tiers(opts, kind, dtype):
    A, B = tier_inputs(kind, dtype)
    got, sym, num, ref = check(A, B, TIER_OPTS[opts], what=f"{kind}/{opts}")
    o = TIER_OPTS[opts] or {}
    if o.get("tiny_max") == -1:
        assert sym["rows"]["tiny"] == 0 and num["rows"]["tiny"] == 0
    if o.get("force_spill") and o.get("tiny_max") == -1:
        assert sym["rows"]["hash"] == sym["rows"]["dense"] == 0
        assert num["rows"]["hash"] == num["rows"]["dense"] == 0
        assert num["rows"]["spill"] > 0
    if opts.startswith("dense"):
        assert num["rows"]["dense"] > 0


def test_tier_row_accounting():
    A, B = tier_inputs("rmat", np.float32)
    got, sym, num, ref = check(A, B, dict(max_lds_slots=512, window_cols=1024))
    nonempty = int(np.sum(ref.products > 0))
    assert sum(sym["rows"].values()) == nonempty
    assert sum(num["products"].values()) == int(ref.products.sum())
    assert sum(num["c_nnz"].values()) == ref.nnz
    assert num["rows"]["dense"] > 0 and num["rows"]["hash"] > 0 and num["rows"]["tiny"] > 0


# ---------------------------------------------------------------------------
# identities, closed forms and special matrices
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_identity_and_permutation_bit_exact(dtype):
    A = matgen.random_sparse(300, 300, 0.05, 9, dtype)
    I = matgen.identity(300, dtype)
    for L, R in ((I, A), (A, I)):
        got, _, _ = run_gpu(L, R)
        assert np.array_equal(got.row_ptr, A.row_ptr.astype(np.int64))
        assert np.array_equal(got.col_idx, A.col_idx)
        assert np.array_equal(got.val, A.val)
    P = matgen.permutation(300, 10, dtype)
    got, _, _ = run_gpu(P, A)
    for i in range(300):
        c, v = A.row(P.col_idx[i])
        assert np.array_equal(got.col_idx[got.row_ptr[i]:got.row_ptr[i + 1]], c)
        assert np.array_equal(got.val[got.row_ptr[i]:got.row_ptr[i + 1]], v)


@pytest.mark.parametrize("n,opts,dtype", [(4096, None, np.float64),
                                          (4096, dict(max_lds_slots=64, window_cols=1024), np.float64),
                                          (4096, dict(force_spill=1), np.float64), (12288, None, np.float64),
                                          (12288, None, np.float32), (12288, dict(window_cols=4096), np.float64)])
def test_arrowhead_dense_square(n, opts, dtype):
    # n = 12288: every row has 12288 entries, 8192 of them in the first
    # 8192-column window; with double output that window takes two rank slices
    A = matgen.arrowhead(n, dtype)
    got, _, _ = run_gpu(A, A, opts)
    assert got.row_ptr[-1] == n * n
    rp = got.row_ptr
    assert np.all(np.diff(rp) == n)
    assert np.array_equal(got.col_idx.reshape(n, n), np.tile(np.arange(n, dtype=np.int32), (n, 1)))
    C = got.val.reshape(n, n)
    E = np.ones((n, n))
    E[0, :] = 2
    E[:, 0] = 2
    E[np.arange(n), np.arange(n)] = 2
    E[0, 0] = n
    assert np.array_equal(C, E)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("opts", [None, dict(dense_min_nnz=1)])
def test_dense_rows_across_regions(dtype, opts):
    # rows of ~12K entries spread over 600K columns: several 262144-column
    # regions and several super-windows per row in the rank-indexed kernel
    A = matgen.er(48, 2000, 200, seed=31, dtype=dtype, dist="pm1" if dtype == np.float64 else "open01")
    B = matgen.er(2000, 600_000, 60, seed=32, dtype=dtype, dist="pm1" if dtype == np.float64 else "open01")
    got, sym, num, ref = check(A, B, opts, what="regions")
    assert num["rows"]["dense"] > 0


# every row that fits a hash table takes it: rows of up to 64 A entries would be merged (the caps stay at their
# default)
HASHED = dict(max_lds_slots=16384)


@pytest.mark.parametrize("r", [25, 50, 90])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_hash_rows_rank_emission_windows(r, dtype):
    # hash rows of ~20r entries over 200K columns: tables of 1024, 2048 and
    # 4096 slots write their rows in 4, 2 and 1 bitmap windows (the last one
    # ragged)
    dist = "pm1" if dtype == np.float64 else "open01"
    A = matgen.er(64, 3000, r, seed=70 + r, dtype=dtype, dist=dist)
    B = matgen.er(3000, 200_000, 20, seed=69, dtype=dtype, dist=dist)
    got, sym, num, ref = check(A, B, HASHED, what=f"hash windows r={r}")
    assert num["rows"]["hash"] == 64 and num["merged_rows"] == sym["merged_rows"] == 0


@pytest.mark.parametrize("ncols,r", [(1_000_000, 25), (1_000_000, 50), (1_000_000, 90), (3_000_000, 50),
                                     (20_000, 40)])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_hash_rows_bucket_emission(ncols, r, dtype):
    # hash rows over wide column ranges: tables of 512 to 4096 slots write their rows by column buckets of
    # up to 512 columns, wider buckets fall back to the bitmap or a sort (3 M columns)
    dist = "pm1" if dtype == np.float64 else "open01"
    A = matgen.er(64, 3000, r, seed=80 + r, dtype=dtype, dist=dist)
    B = matgen.er(3000, ncols, 20, seed=79, dtype=dtype, dist=dist)
    got, sym, num, ref = check(A, B, HASHED, what=f"hash buckets n={ncols} r={r}")
    assert num["rows"]["hash"] == 64 and num["merged_rows"] == sym["merged_rows"] == 0


@pytest.mark.parametrize("rows,launches", [(10, (1, 2)), (600, (4, 6))])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_few_hash_rows_share_launches(rows, launches, dtype):
    # rows of 70 A entries whose B rows hold 1 to 23 entries: tables of 2^8 to 2^11 slots (symbolic, the longest row by
    # its bitmap) and 2^7 to 2^12 (numeric). Few rows of a size go along with larger ones, up to eight times its table
    rng = np.random.default_rng(rows)
    sizes, n = [1, 2, 3, 6, 12, 23], 100_000
    cols = [np.sort(rng.choice(n, L, replace=False)) for L in sizes for _ in range(200)]
    B = matgen.CSR(len(cols), n, np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32),
                   np.concatenate(cols).astype(np.int32), None)
    B.val = (1.0 - rng.random(len(B.col_idx))).astype(dtype)
    picks = [200 * g + np.sort(rng.choice(200, 70, replace=False)) for g in range(len(sizes)) for _ in range(rows)]
    A = matgen.CSR(len(picks), B.nrows, (70 * np.arange(len(picks) + 1)).astype(np.int32),
                   np.concatenate(picks).astype(np.int32), None)
    A.val = (1.0 - rng.random(len(A.col_idx))).astype(dtype)
    _, sym, num, _ = check(A, B, None, what="few hash rows")
    assert num["rows"]["hash"] == len(picks) and num["merged_rows"] == 0
    assert (sym["launches"]["hash"], num["launches"]["hash"]) == launches
    _, sym, num, _ = check(A, B, HASHED, what="hash rows by size")
    assert (sym["launches"]["hash"], num["launches"]["hash"]) == (4, 6)
    import torch
    from paper_2606_20855_amd import wingspan as ws
    C = ws.sharded_to_csr(ws.spgemm_sharded(ws.DeviceCSR.from_host(A, "cuda:0"), ws.DeviceCSR.from_host(B, "cuda:0")))
    torch.cuda.synchronize()
    assert_matches(C.to_host(), oracle.spgemm(A, B), dtype, what="single pass")


@pytest.mark.parametrize("r", [8, 20, 60])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_hash_rows_bucket_emission_skewed_columns(r, dtype):
    # B's columns are R-MAT's (heavy-tailed toward low indices), so the rows' low-column buckets hold many
    # entries and take their ranks from per-bucket bitmaps
    dist = "pm1" if dtype == np.float64 else "open01"
    B = matgen.rmat(14, 16, seed=84, dtype=dtype, dist=dist)
    A = matgen.er(200, B.nrows, r, seed=85 + r, dtype=dtype, dist=dist)
    got, sym, num, ref = check(A, B, HASHED, what=f"hash buckets skewed r={r}")
    assert num["rows"]["hash"] > 0 and num["merged_rows"] == sym["merged_rows"] == 0


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_dense_rows_beyond_entry_cache(dtype):
    # 400 A entries per row, more than the 256 whose bounds the rank kernel
    # keeps in LDS, and ~11,600 entries per row over 300K columns: two regions,
    # each taken in one or more rank slices
    dist = "pm1" if dtype == np.float64 else "open01"
    A = matgen.er(32, 3000, 400, seed=61, dtype=dtype, dist=dist)
    B = matgen.er(3000, 300_000, 30, seed=62, dtype=dtype, dist=dist)
    got, sym, num, ref = check(A, B, None, what="long A rows")
    assert num["rows"]["dense"] == 32


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_rank_slices_inside_one_window(dtype):
    # ~8,600 entries per row, ~7,800 of them inside the first 8192-column
    # window: more than the double-output rank accumulator holds, so that
    # window is taken in several rank slices
    dist = "pm1" if dtype == np.float64 else "open01"
    A = matgen.random_sparse(64, 50, 0.9, 41, dtype, dist)
    B = matgen.random_sparse(50, 9000, 0.07, 42, dtype, dist)
    got, sym, num, ref = check(A, B, None, what="rank slices")
    assert num["rows"]["dense"] == 64


def test_laplacian_512_bit_exact():
    A, B = matgen.config("laplace512")
    got, sym, num = run_gpu(A, B)
    ref = oracle.spgemm(A, B)
    assert np.array_equal(got.row_ptr, ref.row_ptr)
    assert np.array_equal(got.col_idx, ref.col_idx)
    assert np.array_equal(got.val, ref.val)        # small integers: exact in any order
    g = golden("laplace512")
    assert got.row_ptr[-1] == g["nnz_c"] == 3_397_636
    assert sym["total_products"] == g["products"] == 6_535_176


def test_er1000():
    A, B = matgen.config("er1000")
    got, sym, num, ref = check(A, B)
    g = golden("er1000")
    assert sym["total_products"] == g["products"] == 100_000
    assert row_ptr_sha256(got.row_ptr) == g["row_ptr_sha256"]


@pytest.mark.slow
def test_er_rect_full():
    A, B = matgen.config("er_rect")
    got, sym, num = run_gpu(A, B)
    g = golden("er_rect")
    assert sym["total_products"] == g["products"] == 64_000_000
    assert row_ptr_sha256(got.row_ptr) == g["row_ptr_sha256"]
    ref = oracle.spgemm(A, B)
    assert_matches(got, ref, A.val.dtype, what="er_rect")


# ---------------------------------------------------------------------------
# API behaviour on the device
# ---------------------------------------------------------------------------

def test_structure_deterministic():
    A = matgen.rmat(12, 16, seed=11, dtype=np.float32)
    first, _, _ = run_gpu(A, A, dict(max_lds_slots=256, window_cols=1024))
    for _ in range(3):
        again, _, _ = run_gpu(A, A, dict(max_lds_slots=256, window_cols=1024))
        assert np.array_equal(first.row_ptr, again.row_ptr)
        assert np.array_equal(first.col_idx, again.col_idx)


def test_numeric_rerun_with_new_values():
    import torch
    from paper_2606_20855_amd import wingspan as ws
    A = matgen.rmat(11, 16, seed=12, dtype=np.float64, dist="pm1")
    dA = ws.DeviceCSR.from_host(A, "cuda:0")
    C = ws.spgemm(dA, dA)
    A2 = matgen.CSR(A.nrows, A.ncols, A.row_ptr, A.col_idx, np.linspace(-1, 1, A.nnz))
    dA2 = ws.DeviceCSR.from_host(A2, "cuda:0")
    wsb, nbytes = ws.allocate_workspace(dA2, dA2)
    h = torch.cuda.current_stream().cuda_stream
    ws.wingspan_spgemm_numeric(dA2.desc(), dA2.desc(), ws.F64, C.row_ptr.data_ptr(), C.col_idx.data_ptr(),
                               C.val.data_ptr(), wsb.data_ptr(), nbytes, h)
    torch.cuda.synchronize()
    assert_matches(C.to_host(), oracle.spgemm(A2, A2), np.float64, what="rerun")


def test_combined_entry_and_capacity():
    import torch
    from paper_2606_20855_amd import wingspan as ws
    A = matgen.rmat(10, 16, seed=13, dtype=np.float32)
    ref = oracle.spgemm(A, A)
    dA = ws.DeviceCSR.from_host(A, "cuda:0")
    wsb, nbytes = ws.allocate_workspace(dA, dA)
    h = torch.cuda.current_stream().cuda_stream
    rp = torch.empty(A.nrows + 1, dtype=torch.int64, device="cuda:0")
    small = ref.nnz - 1
    col = torch.empty(max(small, 1), dtype=torch.int32, device="cuda:0")
    val = torch.empty(max(small, 1), dtype=torch.float32, device="cuda:0")
    with pytest.raises(ws.WingspanError) as e:
        ws.wingspan_spgemm(dA.desc(), dA.desc(), ws.F32, rp.data_ptr(), col.data_ptr(), val.data_ptr(), small,
                           wsb.data_ptr(), nbytes, h)
    assert ws.STATUS[e.value.status] == "WINGSPAN_ERR_INSUFFICIENT_CAPACITY"
    assert np.array_equal(rp.cpu().numpy(), ref.row_ptr)
    col = torch.empty(ref.nnz, dtype=torch.int32, device="cuda:0")
    val = torch.empty(ref.nnz, dtype=torch.float32, device="cuda:0")
    nnz = ws.wingspan_spgemm(dA.desc(), dA.desc(), ws.F32, rp.data_ptr(), col.data_ptr(), val.data_ptr(), ref.nnz,
                             wsb.data_ptr(), nbytes, h)
    torch.cuda.synchronize()
    assert nnz == ref.nnz
    got = ws.HostCSR(A.nrows, A.ncols, rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy())
    assert_matches(got, ref, np.float32, what="combined")


def test_validate_rejects_noncanonical():
    from paper_2606_20855_amd import wingspan as ws
    A = matgen.random_sparse(40, 40, 0.3, 14)
    r = int(np.argmax(np.diff(A.row_ptr) >= 2))
    col = A.col_idx.copy()
    a = A.row_ptr[r]
    col[a], col[a + 1] = col[a + 1], col[a]
    bad = matgen.CSR(A.nrows, A.ncols, A.row_ptr, col, A.val)
    dA = ws.DeviceCSR.from_host(A, "cuda:0")
    dBad = ws.DeviceCSR.from_host(bad, "cuda:0")
    with pytest.raises(ws.WingspanError) as e:
        ws.spgemm(dBad, dA, options=dict(validate=1))
    assert ws.STATUS[e.value.status] == "WINGSPAN_ERR_INVALID_MATRIX"
    with pytest.raises(ws.WingspanError) as e:
        ws.spgemm(dA, dBad, options=dict(validate=1))
    assert ws.STATUS[e.value.status] == "WINGSPAN_ERR_INVALID_MATRIX"


def test_validate_reports_inconsistent_row_ptr():
    import torch
    from paper_2606_20855_amd import wingspan as ws
    A = matgen.rmat(10, 16, seed=15, dtype=np.float64, dist="pm1")
    dA = ws.DeviceCSR.from_host(A, "cuda:0")
    C = ws.spgemm(dA, dA)
    rp = C.row_ptr.clone()
    # shift one row boundary: rows i and i+1 now disagree with the product
    lens = torch.diff(rp)
    i = int(torch.argmax(lens).item())
    rp[i + 1] -= 1
    wsb, nbytes = ws.allocate_workspace(dA, dA)
    h = torch.cuda.current_stream().cuda_stream
    with pytest.raises(ws.WingspanError) as e:
        ws.wingspan_spgemm_numeric(dA.desc(), dA.desc(), ws.F64, rp.data_ptr(), C.col_idx.data_ptr(),
                                   C.val.data_ptr(), wsb.data_ptr(), nbytes, h, dict(validate=1))
    assert ws.STATUS[e.value.status] == "WINGSPAN_ERR_INCONSISTENT"


def test_timing_option_fills_kernel_times():
    A = matgen.rmat(12, 16, seed=16, dtype=np.float32)
    got, sym, num = run_gpu(A, A, dict(timing=1, max_lds_slots=512, window_cols=1024))
    assert num["analysis_ms"] > 0
    assert all(v >= 0 for v in num["kernel_ms"].values())
    assert sum(num["kernel_ms"].values()) > 0
