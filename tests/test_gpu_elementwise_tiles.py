"""GPU tests of the elementwise tiles' codes: rows that start and end at a tile's
boundary or one entry beside it, empty rows there, in front and at the end, and
common coordinates on both sides of a boundary, against the elementwise oracle.
A sum or product of two values formed in double and rounded once has one right
result: equality is exact."""
from __future__ import annotations

import numpy as np
import pytest

import matgen
from oracle import elementwise as ew_oracle

pytestmark = pytest.mark.gpu

TILE = 2048


def _pair(starts, total, kind, dtype, seed):
    """A and B with merged row starts at `starts` (twice: an empty row) and `total` merged entries. A row's first and last
    coordinates are common where it has two entries ("ends"), all are ("equal"), or none is, its first half in A
    ("split"); with "one" B's side is empty in every second row."""
    rng = np.random.default_rng(seed)
    rows_a, rows_b = [], []
    for r, n in enumerate(np.diff(list(starts) + [total])):
        n = int(n)
        if kind == "equal":
            c = np.sort(rng.choice(6000, size=(n + 1) // 2, replace=False))
            a, b = c, c[: n // 2]
        elif kind == "ends" and n >= 4:
            c = np.sort(rng.choice(6000, size=n - 2, replace=False))
            pick = rng.random(n - 2) < 0.5
            pick[0] = pick[-1] = True
            a, b = c[pick], np.concatenate([c[:1], c[~pick], c[-1:]]) if n > 3 else c[:1]
        elif kind == "one" and r % 2:
            a, b = np.sort(rng.choice(6000, size=n, replace=False)), np.zeros(0, dtype=np.int64)
        else:
            c = np.sort(rng.choice(6000, size=n, replace=False))
            a, b = c[: n // 2], c[n // 2:]
        assert len(a) + len(b) == n
        rows_a.append(a)
        rows_b.append(b)

    def csr(rows):
        ptr = np.concatenate([[0], np.cumsum([len(x) for x in rows])]).astype(np.int32)
        return matgen.CSR(len(rows), 6000, ptr, np.concatenate(rows).astype(np.int32),
                          (rng.random(ptr[-1]) - 0.5).astype(dtype))
    return csr(rows_a), csr(rows_b)


STARTS = {
    "at": [0, TILE, 2 * TILE], "beside": [0, TILE - 1, TILE + 1, 2 * TILE + 1],
    "empty": [0, 0, 0, TILE, TILE, TILE, 2 * TILE, 3 * TILE, 3 * TILE],
    "many": [0] * 700 + [7, TILE - 9] + [TILE] * 700 + [TILE + 1],
    "first": [0, 1, 2, 3, 4, 8, 9, 10], "long": [0, 5000],
}


@pytest.mark.parametrize("kind", ["ends", "equal", "split", "one"])
@pytest.mark.parametrize("starts", list(STARTS))
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_tile_boundaries(starts, kind, dtype):
    import torch
    from paper_2606_20855_amd import wingspan as ws
    at = STARTS[starts]
    for total in sorted({max(at[-1], 1), at[-1] + 1, -(-(at[-1] + 1) // TILE) * TILE}):
        A, B = _pair(at, total, kind, dtype, 5 + total)
        dA, dB = ws.DeviceCSR.from_host(A, "cuda:0"), ws.DeviceCSR.from_host(B, "cuda:0")
        for op, ref in (("add", ew_oracle.spadd(A, B)), ("hadamard", ew_oracle.hadamard(A, B))):
            C = ws.elementwise(op, dA, dB)
            torch.cuda.synchronize()
            got = C.to_host()
            assert np.array_equal(np.asarray(got.row_ptr, np.int64), ref.row_ptr), (op, total)
            assert np.array_equal(got.col_idx, ref.col_idx), (op, total)
            assert np.array_equal(got.val, ref.val), (op, total)
