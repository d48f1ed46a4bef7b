"""The one-call neighbour export: it asks for the rows' memory once they are counted, gives the
two-call form's offsets and rows, and ends cleanly when there is no memory for them."""
import ctypes as C

import pytest
import torch

import csph_inputs as ci
import paper_1805_05128_amd as P
from paper_1805_05128_amd import _native as N
from paper_1805_05128_amd import api as A

pytestmark = pytest.mark.gpu
DEV = "cuda"


def two_calls(s, params, ws):
    L, n = N.load(), s.n
    off = torch.empty(n + 1, dtype=torch.int64, device=DEV)
    nnz, st, p = C.c_int64(0), s.c(), params.c()
    call = lambda idx, cap: A._with_ws(
        lambda w, b, nd: L.csph_neighbors(C.byref(st), C.byref(p), A._lp(off), idx, cap,
                                          C.byref(nnz), w, b, nd, A._stream(None)), ws, "two calls")
    call(None, 0)
    idx = torch.empty(max(nnz.value, 1), dtype=torch.int32, device=DEV)
    call(A._ip(idx), idx.shape[0])
    return off, idx[:nnz.value]


@pytest.mark.parametrize("side,spread", [((1, 1, 1), 1.0), ((3, 1, 1), 100.0), ((23, 9, 7), 1.0)])
def test_one_call_equals_two(side, spread):
    print(f"[case] neighbours {side} spread {spread}", flush=True)
    w = ci.jittered_block(*side, seed=3, amp=0.2)
    w.x = w.x * spread  # 100: nobody within reach, no rows at all
    params = P.Params.from_workload(w)
    s = P.state_from_workload(w, params, DEV)
    off, idx = P.csph_neighbors(s, params, ws=P.Workspace(DEV))
    ref_off, ref_idx = two_calls(s, params, P.Workspace(DEV))
    assert torch.equal(off, ref_off) and torch.equal(idx, ref_idx)
    assert idx.numel() == int(off[-1])


def test_no_memory_for_rows(monkeypatch):
    print("[case] neighbours without memory", flush=True)
    w = ci.jittered_block(8, 8, 8, seed=3)
    params = P.Params.from_workload(w)
    s, ws = P.state_from_workload(w, params, DEV), P.Workspace(DEV)
    off, idx = P.csph_neighbors(s, params, ws=ws)
    real = torch.empty

    def refuse(*a, **k):
        if k.get("dtype") == torch.int32:
            raise MemoryError("refused")
        return real(*a, **k)

    monkeypatch.setattr(torch, "empty", refuse)
    with pytest.raises(MemoryError):
        P.csph_neighbors(s, params, ws=ws)
    monkeypatch.undo()
    again = P.csph_neighbors(s, params, ws=ws)
    assert torch.equal(off, again[0]) and torch.equal(idx, again[1])
