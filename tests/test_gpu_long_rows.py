"""Neighbour rows longer than the LDS list: sorted by the whole wave."""
import numpy as np
import pytest
import torch

import csph_inputs as ci
import oracle as O
import paper_1805_05128_amd as P
from helpers import to_np

pytestmark = pytest.mark.gpu
DEV = "cuda"


# around the runs' powers of two; two lengths of rows in one set
@pytest.mark.parametrize("n", [601, 1024, 1025, 1026, 2050, 3000])
def test_rows(n):
    w = ci.random_cloud(n, seed=n, box=1.0)
    w.x[: n // 8] += 2.6  # these and the rest see a part of each other
    params = P.Params.from_workload(w)
    off, idx = P.csph_neighbors(P.state_from_workload(w, params, DEV), params)
    ro, ri = O.neighbors(O.cfg_for(w), w.x, w.y, w.z, None)
    assert np.array_equal(to_np(off), ro) and np.array_equal(to_np(idx), ri)
    assert len(set(np.diff(ro).tolist())) > 2


def _ms(h):
    w = ci.jittered_block(28, 27, 26, seed=3, amp=0.2)
    params = P.Params.from_workload(w, h=h, cell_size=0.0)
    st = P.state_from_workload(w, params, DEV)
    off, _ = P.csph_neighbors(st, params)
    best = np.inf
    for _ in range(5):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        P.csph_neighbors(st, params)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best, int((off[1:] - off[:-1]).max())


def test_long_rows_cost_what_short_rows_do():
    """Rows of up to 1 450 entries (seven times the pairs) against rows that fit the list: sorted
    by one lane they took 85 times as long."""
    short, most = _ms(1.8)
    assert most <= 512
    long, most = _ms(3.5)
    assert most > 1024
    assert long <= 20.0 * short, (short, long)
