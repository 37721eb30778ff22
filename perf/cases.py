"""The work a user of this framework has it do, as cases that can be timed.

Every operation of the public Python interface is covered with inputs of the
kinds the framework is built for: random matrices with a fixed number of
entries per row, mesh (grid stencil) matrices, power-law (R-MAT) graphs and
products of rectangular matrices, from a thousand rows to a few million, in
float and double. A case is a dict of plain values:

  op       product      C = A B, structure and values, C allocated by the call
           values       C's values again for a known structure (a sequence of
                        products whose patterns stay and whose values change)
           single_pass  C = A B in one pass into a pool, then gathered to CSR
           outer        C = A B by outer products, A given by its columns
           add, hadamard    C = A + B, C = A .* B
           spmspv       y = A x for a sparse x, A given by its columns
  kind     er (about r entries in every row), grid (a 5- or 9-point stencil on
           nx x ny points) or graph (R-MAT on n vertices, ef drawn edges each)
  dtype    f32 or f64

The inputs are made on the GPU. A case's matrices have one pattern, which the
seed moves: their rows and columns are rotated by places that the seed gives (a
squared matrix's alike), so C's entries move too while their number stays. The
values are new with every seed.
"""
import math

import torch

from paper_2606_20855_amd import wingspan as ws

_DTYPE = {"f32": torch.float32, "f64": torch.float64}
_RMAT = (0.57, 0.19, 0.19)   # the quadrant probabilities a, b, c of the repository's graphs


def listed():
    return [
        # the smallest call: launches and the read-backs, not bytes
        {"name": "product_er_1000", "op": "product", "kind": "er", "m": 1000, "k": 1000, "n": 1000, "r": 10,
         "dtype": "f64"},
        # a mesh operator squared (the setup of a multigrid hierarchy)
        {"name": "product_grid_512", "op": "product", "kind": "grid", "nx": 512, "ny": 512, "points": 5,
         "dtype": "f64"},
        # a non-square product of matrices with short rows
        {"name": "product_er_rect", "op": "product", "kind": "er", "m": 1000000, "k": 500000, "n": 1000000, "r": 8,
         "dtype": "f64"},
        # two-hop neighbourhoods of a power-law graph: the framework's headline workload
        {"name": "product_graph_262144", "op": "product", "kind": "graph", "n": 262144, "ef": 16, "dtype": "f32"},
        # the same on a larger, sparser graph of an odd size: C's columns pass what one bitmap region holds
        {"name": "product_graph_1000003", "op": "product", "kind": "graph", "n": 1000003, "ef": 4, "dtype": "f64"},
        # a graph of several million vertices, as web and social graphs have
        {"name": "product_graph_2500000", "op": "product", "kind": "graph", "n": 2500000, "ef": 2, "dtype": "f32"},
        # new edge weights on a known structure
        {"name": "values_graph_131072", "op": "values", "kind": "graph", "n": 131072, "ef": 16, "dtype": "f64"},
        # the single pass with its gather, an odd number of vertices
        {"name": "single_pass_graph_100003", "op": "single_pass", "kind": "graph", "n": 100003, "ef": 16,
         "dtype": "f32"},
        # a mesh operator squared through outer products
        {"name": "outer_grid_512", "op": "outer", "kind": "grid", "nx": 512, "ny": 512, "points": 5, "dtype": "f64"},
        # the sum of two graphs of one degree distribution on different patterns
        {"name": "add_graph_1048576", "op": "add", "kind": "graph", "n": 1048576, "ef": 16, "same": False,
         "dtype": "f64"},
        # elementwise weights on one pattern
        {"name": "hadamard_graph_262144", "op": "hadamard", "kind": "graph", "n": 262144, "ef": 16, "same": True,
         "dtype": "f32"},
        # one step of a frontier through a graph: a tenth of the vertices active
        {"name": "spmspv_graph_1048576", "op": "spmspv", "kind": "graph", "n": 1048576, "ef": 16, "density": 0.1,
         "dtype": "f64"},
    ]


def _log(rng, lo, hi):
    """A whole number in [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _graph_products(n, ef):
    """About the products of an R-MAT graph with itself (repeated edges counted)."""
    return ef * ef * n * 1.27 ** math.log2(n)


def draw(rng):
    op = rng.choice(["product"] * 5 + ["values", "single_pass", "outer", "add", "hadamard", "spmspv"])
    kind = {"outer": ["er", "grid"], "add": ["graph", "er"], "hadamard": ["graph"], "spmspv": ["graph"],
            "values": ["graph", "grid"], "single_pass": ["graph", "er"]}.get(op, ["er", "grid", "graph", "graph"])
    c = {"op": op, "kind": rng.choice(kind), "dtype": rng.choice(["f32", "f64"])}
    if c["kind"] == "er":
        c["r"] = _log(rng, 2, 32)
        # at most 30 M products (one per entry of A and of the row of B it selects) and 16 M entries
        most = min(1000000, 30000000 // (c["r"] * c["r"]))
        c["m"] = _log(rng, 300, most)
        c["k"] = _log(rng, 300, most if op == "outer" else min(1000000, 16000000 // c["r"]))
        c["n"] = c["k"] if op in ("add", "hadamard") else _log(rng, 300, 1000000)
    elif c["kind"] == "grid":
        c["nx"], c["ny"], c["points"] = _log(rng, 20, 600), _log(rng, 20, 600), rng.choice([5, 9])
    else:
        # the products within the listed graphs' (a C of over a million columns within the sparsest one's)
        c["n"] = _log(rng, 1000, 3000000)
        c["ef"] = rng.randint(1, 16)
        if op in ("product", "values", "single_pass"):
            most = _graph_products(262144, 12) if c["n"] <= 1000003 else _graph_products(2500000, 2)
            while c["ef"] > 1 and _graph_products(c["n"], c["ef"]) > most:
                c["ef"] -= 1
        else:
            while c["ef"] > 1 and c["n"] * c["ef"] > 1048576 * 16:
                c["ef"] -= 1
    if op in ("add", "hadamard"):
        c["same"] = rng.random() < 0.5
    if op == "spmspv":
        c["density"] = round(math.exp(rng.uniform(math.log(0.002), math.log(0.3))), 4)
    return c


# ---------------------------------------------------------------------------
# Inputs.
# ---------------------------------------------------------------------------
def _values(g, n, dtype):
    """Graph weights in (0, 1] for float, entries in [-1, 1) for double: the repository's distributions."""
    u = torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    return (1.0 - u).to(torch.float32).clamp_(min=2.0 ** -24) if dtype == torch.float32 else 2.0 * u - 1.0


def _csr(keys, nrows, ncols, val):
    """keys: row * ncols + column of every entry, increasing."""
    rows = torch.div(keys, ncols, rounding_mode="floor")
    rp = torch.zeros(nrows + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.cumsum(torch.bincount(rows, minlength=nrows), 0)
    return ws.DeviceCSR(nrows, ncols, rp.to(torch.int32), (keys - rows * ncols).to(torch.int32), val)


def _rotated(rows, cols, m, n, turn):
    """The sorted keys of entries (rows, cols) of an m x n matrix, rotated by `turn` (down, right); repeated ones
    merged."""
    return torch.unique((rows + turn[0]) % m * n + (cols + turn[1]) % n)


def _er(g, p, m, n, r, turn, dtype):
    """r uniformly drawn columns in every row; repeated ones merged."""
    cols = torch.randint(0, n, (m, r), generator=p, device="cuda", dtype=torch.int64)
    keys = _rotated(torch.arange(m, device="cuda")[:, None], cols, m, n, turn)
    return _csr(keys, m, n, _values(g, keys.numel(), dtype))


def _grid(g, nx, ny, points, dtype):
    """A 5- or 9-point stencil with varying coefficients, Dirichlet boundary, point p = x + nx y."""
    p = torch.arange(nx * ny, device="cuda")
    x, y = p % nx, torch.div(p, nx, rounding_mode="floor")
    keys, diag = [], []
    for dy in (-1, 0, 1):
        for dx in (-1, 0, 1):
            if points == 5 and dx != 0 and dy != 0:
                continue
            ok = (x + dx >= 0) & (x + dx < nx) & (y + dy >= 0) & (y + dy < ny)
            keys.append((p * (nx * ny) + p + dx + nx * dy)[ok])
            diag.append(torch.full_like(keys[-1], dx == 0 and dy == 0, dtype=torch.bool))
    keys, order = torch.sort(torch.cat(keys))
    diag = torch.cat(diag)[order]
    k = 1.0 - torch.rand(keys.numel(), generator=g, device="cuda", dtype=torch.float64)
    return _csr(keys, nx * ny, nx * ny, torch.where(diag, points - 1 + k, -k).to(dtype))


def _graph(g, p, n, ef, turn, dtype):
    """R-MAT: ef * n edges drawn on the next power of two of vertices, folded onto n; repeated ones merged."""
    scale = max(1, math.ceil(math.log2(n)))
    ne = ef * n
    a, b, c = _RMAT
    rows = torch.zeros(ne, dtype=torch.int64, device="cuda")
    cols = torch.zeros(ne, dtype=torch.int64, device="cuda")
    for _ in range(scale):
        u = torch.rand(ne, generator=p, device="cuda")
        rows = 2 * rows + (u >= a + b)
        cols = 2 * cols + (((u >= a) & (u < a + b)) | (u >= a + b + c))
    keys = _rotated(rows, cols, n, n, turn)
    return _csr(keys, n, n, _values(g, keys.numel(), dtype))


def _inputs(case, seed):
    """(A, B) of the case: for outer, A's transpose in A's place; for spmspv, x in B's place."""
    g, p = torch.Generator(device="cuda"), torch.Generator(device="cuda")
    g.manual_seed(seed)
    p.manual_seed(1)
    dt = _DTYPE[case["dtype"]]
    turns = torch.randint(0, 1 << 30, (3,), generator=g, device="cuda").tolist()   # of A's rows, its columns, B's

    def one(m, n, turn):
        if case["kind"] == "er":
            return _er(g, p, m, n, case["r"], turn, dt)
        if case["kind"] == "grid":
            return _grid(g, case["nx"], case["ny"], case["points"], dt)
        return _graph(g, p, case["n"], case["ef"], turn, dt)

    op = case["op"]
    m, k, n = case.get("m"), case.get("k"), case.get("n")
    if op in ("product", "values", "single_pass"):
        if case["kind"] == "er" and not m == k == n:
            return one(m, k, turns[:2]), one(k, n, turns[1:])
        A = one(m, k, (turns[0], turns[0]))
        return A, A
    if op == "outer":
        return one(k, m, (turns[1], turns[0])), one(k, n, turns[1:])
    A = one(m, k, turns[:2])
    if op == "spmspv":
        # a share of the vertices, each with a weight: the same share of the graph, turned with it
        on = torch.rand(A.nrows, generator=p, device="cuda") < case["density"]
        i = torch.nonzero(on.roll(turns[0] % A.nrows)).flatten()
        return A, (i.to(torch.int32), _values(g, i.numel(), dt))
    if case["same"]:
        return A, ws.DeviceCSR(A.nrows, A.ncols, A.row_ptr, A.col_idx, _values(g, A.nnz, dt))
    # A before it was turned, its rows and columns relabelled, turned with A: the same degrees on another pattern
    rows = torch.randperm(A.nrows, generator=p, device="cuda")[(_rows(A) - turns[0]) % A.nrows]
    cols = torch.randperm(A.ncols, generator=p, device="cuda")[(A.col_idx.long() - turns[1]) % A.ncols]
    keys = _rotated(rows, cols, A.nrows, A.ncols, turns[:2])
    return A, _csr(keys, A.nrows, A.ncols, _values(g, keys.numel(), dt))


def _rows(M):
    """The row of every entry."""
    counts = (M.row_ptr[1:] - M.row_ptr[:-1]).long()
    return torch.repeat_interleave(torch.arange(M.nrows, device="cuda"), counts)


def prepare(case, seed):
    A, B = _inputs(case, seed)
    s = {"op": case["op"], "A": A, "B": B}
    if case["op"] in ("product", "values", "single_pass"):
        # a program that multiplies more than once keeps the workspace
        s["workspace"], nbytes = ws.allocate_workspace(A, B)
    if case["op"] == "values":
        # the structure is found once; the arrays of C stay
        s["stream"] = torch.cuda.current_stream().cuda_stream
        s["c_rp"] = torch.empty(A.nrows + 1, dtype=torch.int64, device="cuda")
        nnz = ws.wingspan_spgemm_symbolic(A.desc(), B.desc(), s["c_rp"].data_ptr(), s["workspace"].data_ptr(), nbytes,
                                          s["stream"])
        s["c_col"] = torch.empty(max(nnz, 1), dtype=torch.int32, device="cuda")
        s["c_val"] = torch.empty(max(nnz, 1), dtype=A.val.dtype, device="cuda")
    if case["op"] == "single_pass":
        # a pool that holds C whatever its entries: the product count, which bounds them
        s["pool"] = max(1, _products(A, B))
    return s


def run(s):
    op, A, B = s["op"], s["A"], s["B"]
    if op == "values":
        w = s["workspace"]
        ws.wingspan_spgemm_numeric(A.desc(), B.desc(), A.dtype_code, s["c_rp"].data_ptr(), s["c_col"].data_ptr(),
                                   s["c_val"].data_ptr(), w.data_ptr(), w.numel(), s["stream"])
        return s["c_rp"], s["c_col"], s["c_val"]
    if op == "spmspv":
        return ws.spmspv(A, B[0], B[1])
    if op == "product":
        C = ws.spgemm(A, B, workspace=s["workspace"])
    elif op == "single_pass":
        C = ws.sharded_to_csr(ws.spgemm_sharded(A, B, workspace=s["workspace"], pool_capacity=s["pool"]))
    elif op == "outer":
        C = ws.spgemm_outer(A, B)
    else:
        C = ws.elementwise(op, A, B)
    return C.row_ptr, C.col_idx, C.val


# ---------------------------------------------------------------------------
# What a pass cannot do without, and how exact its results are.
# ---------------------------------------------------------------------------
def _products(A, B):
    lens = (B.row_ptr[1:] - B.row_ptr[:-1]).long()
    return int(lens[A.col_idx.long()].sum())


def _nbytes(*tensors):
    return sum(t.numel() * t.element_size() for t in tensors)


def work(case):
    """Each input read once and each output written once; two operations a product (one a result of the elementwise
    operations). Counted on the inputs of one seed: the random patterns of a case differ little in size."""
    s = prepare(case, 0)
    out = run(s)
    A, B = s["A"], s["B"]
    csr = lambda M: _nbytes(M.row_ptr, M.col_idx, M.val)  # noqa: E731
    written = _nbytes(*out)
    if case["op"] == "values":
        written = _nbytes(out[1], out[2])   # (C.row_ptr is read)
    if case["op"] == "spmspv":
        # the columns x selects, a pair of pointers for each
        idx = B[0].long()
        n = int((A.row_ptr[idx + 1] - A.row_ptr[idx]).sum())
        return {"bytes": n * (4 + A.val.element_size()) + 8 * idx.numel() + _nbytes(*B) + written, "flops": 2 * n}
    # (A and B share what they have in common: a squared matrix, one pattern)
    read = csr(A)
    if B is not A:
        read += _nbytes(B.val) if B.col_idx is A.col_idx else csr(B)
    if case["op"] in ("add", "hadamard"):
        return {"bytes": read + written, "flops": out[1].numel()}
    P = _products(_transpose(A) if case["op"] == "outer" else A, B)
    return {"bytes": read + written + (_nbytes(s["c_rp"]) if case["op"] == "values" else 0), "flops": 2 * P}


def tolerance(case):
    # sums and products of two numbers, rounded once: one result only
    if case["op"] in ("add", "hadamard"):
        return "exact"
    # float results are rounded once from sums in double: another order of the sum moves one here and there by its
    # last bit. Double results differ by the order of the sum, a hub's of thousands of terms of both signs.
    if case["dtype"] == "f32":
        return {"rel": 1e-7, "max": 5e-7}
    return {"rel": 2e-15, "max": 1e-13}


# ---------------------------------------------------------------------------
# The same results in 64 bits, by sorting the products.
# ---------------------------------------------------------------------------
_CHUNK = 1 << 27   # products sorted at a time
_EXACT_MOST = 4000000000   # products of the largest case that takes less than 20 seconds


def _transpose(M):
    keys, order = torch.sort(M.col_idx.long() * M.nrows + _rows(M))
    return _csr(keys, M.ncols, M.nrows, M.val[order])


def _merge(keys, val):
    """The sums of the values of equal keys, in the order of the keys."""
    keys, order = torch.sort(keys)
    val = val[order]
    new = torch.ones(keys.numel(), dtype=torch.bool, device="cuda")
    new[1:] = keys[1:] != keys[:-1]
    at = torch.cumsum(new, 0) - 1
    n = int(at[-1]) + 1 if keys.numel() else 0
    return torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, at, val)


def _product_values(A, B):
    lens = (B.row_ptr[1:] - B.row_ptr[:-1]).long()
    col, start = A.col_idx.long(), B.row_ptr.long()
    per = lens[col]
    before = torch.zeros(A.nnz + 1, dtype=torch.int64, device="cuda")
    before[1:] = torch.cumsum(per, 0)
    rows = _rows(A)
    at = before[A.row_ptr.long()].tolist()   # the products before each row
    rp = A.row_ptr.tolist()
    parts, r0 = [], 0
    while r0 < A.nrows:
        lo, hi = r0 + 1, A.nrows
        while lo < hi:   # the last row end within a chunk of r0's first product
            mid = (lo + hi + 1) // 2
            lo, hi = (mid, hi) if at[mid] - at[r0] <= _CHUNK else (lo, mid - 1)
        e0, e1 = rp[r0], rp[lo]
        e = torch.repeat_interleave(torch.arange(e0, e1, device="cuda"), per[e0:e1])
        b = torch.arange(at[r0], at[lo], device="cuda") - before[e] + start[col[e]]
        keys = (rows[e] - r0) * B.ncols + B.col_idx[b]
        val = A.val[e].double() * B.val[b].double()
        del e, b
        parts.append(_merge(keys, val))
        r0 = lo
    return torch.cat(parts) if parts else torch.zeros(0, dtype=torch.float64, device="cuda")


def exact(case, seed):
    A, B = _inputs(case, seed)
    op = case["op"]
    if op == "spmspv":
        idx = B[0].long()
        n = (A.row_ptr[idx + 1] - A.row_ptr[idx]).long()
        t = torch.repeat_interleave(torch.arange(idx.numel(), device="cuda"), n)
        first = torch.cumsum(n, 0) - n
        b = torch.arange(t.numel(), device="cuda") - first[t] + A.row_ptr[idx[t]].long()
        return None, _merge(A.col_idx[b].long(), A.val[b].double() * B[1][t].double())
    if op in ("add", "hadamard"):
        ka, kb = _rows(A) * A.ncols + A.col_idx.long(), _rows(B) * B.ncols + B.col_idx.long()
        a, b = A.val.double(), B.val.double()
        if op == "add":
            return None, None, _merge(torch.cat([ka, kb]), torch.cat([a, b]))
        at = torch.searchsorted(kb, ka).clamp_(max=max(0, kb.numel() - 1))
        both = kb[at] == ka
        return None, None, a[both] * b[at[both]]
    if op == "outer":
        A = _transpose(A)
    if _products(A, B) > _EXACT_MOST:
        return None
    val = _product_values(A, B)
    # (the arrays of C a program keeps hold one entry at least)
    return None, None, torch.zeros(1, dtype=torch.float64, device="cuda") if op == "values" and not val.numel() else val
