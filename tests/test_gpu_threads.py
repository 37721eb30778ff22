"""GPU tests of calls from several host threads at once, on their own streams and
on shared ones: few threads, and more than there are read-back buffers (a call
past them copies instead). Every result against the first thread's."""
from __future__ import annotations

import threading

import numpy as np
import pytest

import matgen
import oracle
from gpu_util import assert_matches

pytestmark = pytest.mark.gpu


def _calls(ws, torch, dA, dB, x, workspace):
    C = ws.spgemm(dA, dB, workspace=workspace)
    S = ws.sharded_to_csr(ws.spgemm_sharded(dA, dB, workspace=workspace))
    out = [C.row_ptr, C.col_idx, S.row_ptr, S.col_idx, C.val, S.val]
    for op in ("add", "hadamard"):
        E = ws.elementwise(op, dA, dB)
        out += [E.row_ptr, E.col_idx, E.val]
    O = ws.spgemm_outer(dA, dB)
    y = ws.spmspv(dA, *x)
    return out + [O.row_ptr, O.col_idx, O.val, *y]


@pytest.mark.parametrize("threads,rounds", [(2, 20), (80, 4)])
def test_calls_at_once(threads, rounds):
    import torch
    from paper_2606_20855_amd import wingspan as ws
    # whole numbers: sums are exact in any order
    rng = np.random.default_rng(3)
    A, B = matgen.er(700, 700, 9, 1), matgen.er(700, 700, 7, 2)
    A.val[:], B.val[:] = rng.integers(-3, 4, A.nnz), rng.integers(-3, 4, B.nnz)
    dA, dB = ws.DeviceCSR.from_host(A, "cuda:0"), ws.DeviceCSR.from_host(B, "cuda:0")
    x = (torch.arange(0, 700, 7, dtype=torch.int32, device="cuda:0"),
         torch.ones(100, dtype=torch.float64, device="cuda:0"))
    want = _calls(ws, torch, dA, dB, x, ws.allocate_workspace(dA, dB)[0])
    torch.cuda.synchronize()
    ref = oracle.spgemm(A, B)
    assert_matches(ws.HostCSR(700, 700, *(t.cpu().numpy() for t in (want[0], want[1], want[4]))), ref, np.float64)
    spaces = [ws.allocate_workspace(dA, dB)[0] for _ in range(threads)]
    streams = [torch.cuda.Stream() for _ in range(threads)]
    torch.cuda.synchronize()
    start = threading.Barrier(threads)
    bad, done = [], []

    def work(i):
        try:
            with torch.cuda.device(0), torch.cuda.stream(streams[i]):
                start.wait()
                for r in range(rounds):
                    got = _calls(ws, torch, dA, dB, x, spaces[i])
                    streams[i].synchronize()
                    done.append(len(got) == len(want))
                    bad.extend((i, r, k) for k, (a, b) in enumerate(zip(got, want)) if not torch.equal(a, b))
        except Exception as e:   # (a thread's exception does not end the test by itself)
            bad.append((i, repr(e)))

    ts = [threading.Thread(target=work, args=(i,)) for i in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad and done == [True] * (threads * rounds)
