"""GPU tests of SpMSpV's table of range counts, whose rows are as long as the
products x selects: product counts around a chunk's 4096, all of the columns and
few of them, and as many ranges as the table takes, against a plain numpy sum (in
double; 1e-12 of the sum of |products| covers the few terms of a position)."""
from __future__ import annotations

import numpy as np
import pytest

import matgen

pytestmark = pytest.mark.gpu

CHUNK = 4096


@pytest.mark.parametrize("m", [1, 4096, 4097, 100_000, 2048 * 4096])
@pytest.mark.parametrize("products", [1, CHUNK - 1, CHUNK, CHUNK + 1, 2 * CHUNK, 3 * CHUNK + 5])
@pytest.mark.parametrize("rest", [0, 1, 5 * CHUNK])
def test_products_around_chunks(m, products, rest):
    import torch
    from paper_2606_20855_amd import wingspan as ws
    rng = np.random.default_rng(m + products + rest)

    def columns(total):   # columns of A of up to 50 entries (1 where m is 1), `total` in all
        out = []
        while total > 0:
            n = min(total, m, int(rng.integers(1, 51)))
            out.append(np.unique(rng.integers(0, m, n)) if n < m else np.arange(n))
            total -= len(out[-1])
        return out
    taken, left = columns(products), columns(rest)
    cols = taken + left
    order = rng.permutation(len(cols))
    at = [cols[i] for i in order]
    ptr = np.concatenate([[0], np.cumsum([len(c) for c in at])]).astype(np.int32)
    At = matgen.CSR(len(at), m, ptr, np.concatenate(at).astype(np.int32), rng.random(ptr[-1]) - 0.5)
    xi = np.nonzero(order < len(taken))[0].astype(np.int32)
    xv = rng.random(len(xi)) - 0.5
    y_idx, y_val = ws.spmspv(ws.DeviceCSR.from_host(At, "cuda:0"), torch.from_numpy(xi).to("cuda:0"),
                             torch.from_numpy(xv).to("cuda:0"))
    torch.cuda.synchronize()
    rows = np.concatenate([at[j] for j in xi])
    prods = np.concatenate([At.val[ptr[j]:ptr[j + 1]] * v for j, v in zip(xi, xv)])
    assert len(rows) == products
    want = np.unique(rows)
    assert np.array_equal(y_idx.cpu().numpy(), want)
    s, mag = (np.bincount(rows, w, minlength=m)[want] for w in (prods, np.abs(prods)))
    assert (np.abs(y_val.cpu().numpy() - s) <= 1e-12 * mag).all()
