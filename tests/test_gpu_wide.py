"""GPU tests of products with more than 128 * 8192 columns: the rank kernel and
the symbolic bitmap kernel with wider windows, and the rows merged piece by
piece, against the CPU oracle."""
from __future__ import annotations

import numpy as np
import pytest

import matgen
import oracle
from gpu_util import assert_matches, run_gpu

pytestmark = pytest.mark.gpu


def _pair(ncols, dtype, seed):
    """B: rows of 60, 300 and 3000 columns, half of each clustered (some into one stretch that holds more products
    than a piece or a rank slice takes), the rest spread, the last column among them. A: rows of 2 to 64 entries
    (merged, whole and piece by piece) and of 65 to 400 (the rank kernel)."""
    rng = np.random.default_rng(seed)
    lens = np.array([60] * 400 + [300] * 40 + [3000] * 24)
    at = ncols // 2 + 7
    cols = []
    for n in lens:
        near = at + rng.choice(12_000, size=n // 2, replace=False)
        far = rng.choice(ncols, size=n - n // 2 - 1, replace=False)
        cols.append(np.unique(np.concatenate([near, far, [ncols - 1]])))
    rp = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
    val = (1.0 - rng.random(rp[-1])) * np.where(rng.random(rp[-1]) < 0.5, -1, 1)
    B = matgen.CSR(len(cols), ncols, rp, np.concatenate(cols).astype(np.int32), val.astype(dtype))
    rows = [440 + rng.choice(24, size=k, replace=False) for k in (2, 3, 5, 6, 8, 12, 20, 24)]
    rows += [np.concatenate([400 + rng.choice(40, size=30, replace=False), 440 + rng.choice(24, size=4, replace=False)])]
    rows += [np.concatenate([rng.choice(400, size=60, replace=False), 440 + rng.choice(24, size=4, replace=False)])]
    rows += [np.concatenate([rng.choice(400, size=k, replace=False), 440 + rng.choice(24, size=8, replace=False)])
             for k in (57, 120, 300, 390)]
    rows += [rng.choice(400, size=k, replace=False) for k in (1, 40, 64, 65, 200, 400)] + [np.arange(464), np.arange(0)]
    ap = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    ci = np.concatenate([np.sort(r) for r in rows]).astype(np.int32)
    return matgen.CSR(len(rows), len(cols), ap, ci, (1.0 - rng.random(len(ci))).astype(dtype)), B


# around the first width past 8192-column windows, past the whole-row symbolic bitmap, and past each wider window
@pytest.mark.parametrize("ncols", [1_048_577, 1_179_649, 2_097_152, 2_097_153, 5_000_011, 33_000_000])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_wide(ncols, dtype):
    import torch
    from paper_2606_20855_amd import wingspan as ws
    A, B = _pair(ncols, dtype, ncols % 1000)
    ref = oracle.spgemm(A, B)
    for opts in (None, dict(cache_mib=-1), dict(dense_min_nnz=100), dict(wide_offsets=1, dense_min_nnz=100)):
        got, sym, num = run_gpu(A, B, opts)
        assert_matches(got, ref, A.val.dtype, what=f"{ncols} {opts}")
        assert num["rows"]["dense"] >= 4 and num["rows"]["spill"] == 0
        if opts is None:
            # (the rows of 2 long and of 40 and 64 short B rows fit the places in LDS at every width; the more regions,
            # the longer the rows merged piece by piece)
            assert num["structure_cache_rows"] > 0 and num["merged_rows"] >= (4 if ncols < 4_000_000 else 9)
    dA, dB = ws.DeviceCSR.from_host(A, "cuda:0"), ws.DeviceCSR.from_host(B, "cuda:0")
    C = ws.sharded_to_csr(ws.spgemm_sharded(dA, dB))
    torch.cuda.synchronize()
    assert_matches(C.to_host(), ref, A.val.dtype, what=f"{ncols} single pass")
