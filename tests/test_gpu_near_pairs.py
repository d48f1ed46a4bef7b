"""Pairs far closer than any spacing: the direction between them stays a unit vector (it scales
the closing speed in the signal speed, whatever the kernel's weight), down to squared distances at
the smallest normal number, against the CPU oracle."""
import numpy as np
import pytest

import csph_inputs as ci
import oracle as O
import paper_1805_05128_amd as P
from helpers import RATE_FIELDS, field_relerr, rates_np, to_np

pytestmark = pytest.mark.gpu


# squared distances 1e-200 .. 1e-307 in FP64 (smallest normal 2.2e-308), 1e-30 .. 1.2e-38 in FP32
# (1.2e-38); directions along an axis and off the axes
@pytest.mark.parametrize("precision,s", [("fp64", s) for s in (1e-100, 1e-145, 1e-150, 3e-154)] +
                         [("mixed", s) for s in (1e-15, 3e-19, 2e-19, 1.1e-19)])
@pytest.mark.parametrize("e", [(1.0, 0.0, 0.0), (0.6, 0.0, -0.8), (2 / 3, 1 / 3, -2 / 3)])
def test_signal_speed(precision, s, e):
    w = ci.jittered_block(5, 4, 4, seed=2, amp=0.1, v=(0.1, 0.0, -0.1))
    w.x, w.y, w.z = w.x - 2.5, w.y - 2.0, w.z - 2.0
    i, j = 30, 31
    for k, a in enumerate("xyz"):
        p, v = getattr(w, a), getattr(w, "v" + a)
        p[i], p[j] = 0.0, s * e[k]
        v[i], v[j] = 1.5 * e[k], -0.5 * e[k]  # closing at 2
    params = P.Params.from_workload(w, precision=precision)
    out = P.csph_rates(P.state_from_workload(w, params, "cuda"), params)
    ref = O.rates(O.cfg_for(w, search=1), O.state_from(w, O.cfg_for(w)))
    fp64 = precision == "fp64"
    assert ref["signal"][i] > 2.5
    # FP32: a handful of roundings of 6e-8 in the direction, the closing speed and the sum
    assert np.abs(to_np(out["signal"]) / ref["signal"] - 1.0).max() <= (1e-12 if fp64 else 1e-6)
    err = field_relerr(rates_np(out), ref)
    assert max(err[k] for k in RATE_FIELDS) <= (1e-12 if fp64 else 2e-5), err
    assert np.array_equal(to_np(out["nbr_count"]).astype(np.int64), ref["nbr_count"])
