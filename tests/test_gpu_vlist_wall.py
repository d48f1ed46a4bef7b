"""Verlet-list steps of one particle, of few and of odd numbers of them, open
and with a piston, equal the direct steps' states (the lists' records are laid out of their own)."""
import numpy as np
import pytest
import torch

import csph_inputs as ci
import paper_1805_05128_amd as P
from helpers import to_np

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("wall", [None, (0.3, 0.2)])
@pytest.mark.parametrize("side", [(1, 1, 1), (3, 3, 3), (8, 8, 8), (17, 11, 13)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_list_steps_equal_direct_steps(precision, side, wall):
    w = ci.jittered_block(*side, seed=4, amp=0.1, v=(0.02, -0.01, 0.03))
    w.vx = w.vx - 0.05 * np.sin(w.z)
    params = P.Params.from_workload(w, precision=precision, cell_size=1.0, wall=wall)
    lists = P.state_from_workload(w, params, DEV)
    sc = P.StepScalars(DEV)
    run = P.VerletRun(lists, params, beta=0.3, n_upd=3)
    got = run.advance(sc, 5, dt_in=0.0)
    st = P.state_from_workload(w, params, DEV)
    sd = P.StepScalars(DEV)
    for _ in range(5):
        st = P.csph_step(st, params, sd)
    a, b = torch.argsort(got["id"]), torch.argsort(st["id"])
    # the order of the additions differs: FP64 rounding, FP32 sums over ~100 partners
    tol = 1e-11 if precision == "fp64" else 2e-5
    for f in P.GRAD_FIELDS:
        x, y = to_np(got[f][a]), to_np(st[f][b])
        assert np.abs(x - y).max() <= tol * max(1.0, np.abs(y).max()), f
    assert float(sc.dt) == pytest.approx(float(sd.dt), rel=10 * tol)
