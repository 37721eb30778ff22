"""GPU tests of the row analysis: product counts around the tiles of A's entries
(rows that end on, start on and span them), row counts around the binning's
workgroups and the scan's forms, against numpy."""
from __future__ import annotations

import numpy as np
import pytest

import matgen
from gpu_util import gpu_row_products, run_gpu

pytestmark = pytest.mark.gpu


def _a(lens, k, seed):
    """Rows of the given lengths (columns distinct and sorted within a row)."""
    rng = np.random.default_rng(seed)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = np.empty(rp[-1], np.int32)
    for i in np.nonzero(lens)[0]:
        n = int(lens[i])
        ci[rp[i]:rp[i + 1]] = np.sort(rng.choice(k, size=n, replace=False)) if n > 1 else rng.integers(0, k)
    return matgen.CSR(len(lens), k, rp, ci, np.ones(rp[-1]))


@pytest.mark.parametrize("lens", [
    [2048], [2048, 2048], [0, 2047, 1, 0, 2048, 0], [2049], [1, 2047, 2048, 0], [5000, 0, 1192], [100, 9000, 0, 3],
    [0, 0, 0], [1], [4096, 4096, 1],
    # rows of 16 and 17 tiles and more, several in a wave and in one of its lanes' rows that follow no other
    [32767, 1, 34816, 34817, 0, 5, 40000], [1] * 63 + [39999] + [2] * 64 + [35000, 0, 36000]], ids=str)
def test_row_products_around_tiles(lens):
    B = matgen.er(40_000, 50, 1, seed=2)
    keep = np.random.default_rng(3).random(B.nrows) < 0.5   # half of B's rows are empty
    bp = np.concatenate([[0], np.cumsum(keep)]).astype(np.int32)
    B = matgen.CSR(B.nrows, 50, bp, B.col_idx[keep], B.val[keep])
    A = _a(np.array(lens), B.nrows, 4)
    want = np.add.reduceat(np.append(keep[A.col_idx].astype(np.int64), 0), A.row_ptr[:-1]) * (np.diff(A.row_ptr) > 0)
    assert np.array_equal(gpu_row_products(A, B), want)
    got, sym, _ = run_gpu(A, B)
    assert sym["total_products"] == want.sum()
    for i in range(A.nrows):
        cols = np.unique(B.col_idx[bp[A.row(i)[0]][keep[A.row(i)[0]]]])
        assert np.array_equal(got.col_idx[got.row_ptr[i]:got.row_ptr[i + 1]], cols)


@pytest.mark.parametrize("m", [1, 1023, 1024, 1025, 4095, 4096, 4097, 262_143, 262_145, 2_097_152, 2_097_153])
@pytest.mark.parametrize("opts", [None, dict(cache_mib=-1)], ids=["cache", "no cache"])
def test_row_counts(m, opts):
    # rows of 0 to 3 A entries, each selecting one entry of B: C is A with its columns renamed
    rng = np.random.default_rng(m)
    lens = rng.integers(0, 4, m)
    lens[-1] = 2
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    off = np.arange(rp[-1]) - np.repeat(rp[:-1], lens)
    ci = (rng.integers(0, 100, m).repeat(lens) + 100 * off).astype(np.int32)
    A = matgen.CSR(m, 300, rp, ci, np.ones(rp[-1], np.float32))
    B = matgen.CSR(300, 1000, np.arange(301, dtype=np.int32), (3 * np.arange(300)).astype(np.int32),
                   np.full(300, 0.5, np.float32))
    got, sym, num = run_gpu(A, B, opts)
    assert np.array_equal(got.row_ptr, rp) and np.array_equal(got.col_idx, 3 * ci)
    assert np.all(got.val == 0.5)
    assert num["rows"]["tiny"] == int(np.sum(lens > 0)) and num["c_nnz_total"] == rp[-1]


def _rows_of_one_entry_each(rows, per):
    """A of `rows` full rows of `per` entries, B of `per` rows of one entry: every row of A has `per` products."""
    import torch
    from paper_2606_20855_amd import wingspan as ws
    t = dict(device="cuda:0", dtype=torch.int32)
    n = rows * per
    one = torch.ones(1, device="cuda:0").expand(n)   # (values are not read)
    A = ws.DeviceCSR(rows, per, torch.arange(rows + 1, **t) * per, torch.arange(per, **t).repeat(rows), one)
    B = ws.DeviceCSR(per, 64, torch.arange(per + 1, **t), torch.arange(per, **t) % 64, one[:per])
    return A, B


def test_long_rows_cost_what_short_ones_do():
    # a row's products over many tiles of A's entries are added up by a whole wave: one row of 8 M entries takes about
    # as long as 64 rows of 125 K (a lane alone: seven times as long)
    import torch
    from paper_2606_20855_amd import wingspan as ws
    took = []
    for rows, per in ((64, 125_000), (1, 8_000_000)):
        A, B = _rows_of_one_entry_each(rows, per)
        wsb, nbytes = ws.allocate_workspace(A, B)
        out = torch.zeros(rows, dtype=torch.int64, device="cuda:0")
        best = float("inf")
        for _ in range(6):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            for _ in range(5):
                ws.wingspan_spgemm_row_products(A.desc(), B.desc(), out.data_ptr(), wsb.data_ptr(), nbytes,
                                                torch.cuda.current_stream().cuda_stream)
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, e[0].elapsed_time(e[1]) / 5)
        assert torch.all(out == per)
        took.append(best)
    print(f"64 rows {took[0] * 1e3:.0f} us, one row {took[1] * 1e3:.0f} us")
    assert took[1] < 1.8 * took[0]


# run in a process of its own: the library's first call that could take a read-back buffer must be the captured one
CAPTURE = """
import numpy as np, torch, matgen, oracle
from paper_2606_20855_amd import wingspan as ws
A = matgen.rmat(9, 8, seed=5)
want = oracle.row_products(A, A)
d = ws.DeviceCSR.from_host(A, "cuda:0")
rp = torch.empty(A.nrows + 1, dtype=torch.int64, device="cuda:0")
col, val = torch.empty(2 * A.nnz, dtype=torch.int32, device="cuda:0"), torch.empty(2 * A.nnz, device="cuda:0").double()
n = ws.wingspan_elementwise_workspace_size(d.desc(), d.desc())
tmp = torch.empty(n, dtype=torch.uint8, device="cuda:0")
# (loads the library's code; takes no buffer)
ws.wingspan_elementwise_values(ws.OP_ADD, d.desc(), d.desc(), d.dtype_code, rp.data_ptr(), col.data_ptr(),
                               val.data_ptr(), tmp.data_ptr(), n, torch.cuda.current_stream().cuda_stream)
wsb, nbytes = ws.allocate_workspace(d, d)
out = torch.full((A.nrows,), -1, dtype=torch.int64, device="cuda:0")
torch.cuda.synchronize()
g = torch.cuda.CUDAGraph()
with torch.cuda.graph(g):
    ws.wingspan_spgemm_row_products(d.desc(), d.desc(), out.data_ptr(), wsb.data_ptr(), nbytes,
                                    torch.cuda.current_stream().cuda_stream)
for i in range(4):
    out.fill_(-1 - i)
    g.replay()
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), want), i
    assert np.array_equal(ws.row_products(d, d).cpu().numpy(), want)
print("captured")
"""


def test_row_products_can_be_captured_as_a_first_call():
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", CAPTURE], cwd=root, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "captured" in r.stdout, r.stdout + r.stderr
