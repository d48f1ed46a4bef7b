"""FP32 walks around periodic images that few lanes of a wave have (the rows' candidates tested by
the whole wave): counts equal the FP64 walk's, rates agree with it within the mixed kernel's
tolerance, for rows with few and with many such lanes, and for sets so dense that the layout or a
particle's list is too short and the lock-step walk takes over."""
import numpy as np
import pytest
import torch

import csph_inputs as ci
import paper_1805_05128_amd as P

pytestmark = pytest.mark.gpu
DEV = "cuda"
RATES = ("drho", "dvx", "dvy", "dvz", "dE")


# spacing 1: ~110 partners, faces of 3 particles a row end; 0.75 and 0.5: past 64 partners of one
# image and past 128 candidates; sides 12 (every particle near a face along it) to 70
@pytest.mark.parametrize("per", [1, 3, 5, 7])
@pytest.mark.parametrize("side,space", [((70, 12, 12), 1.0), ((33, 17, 12), 1.0),
                                        ((30, 16, 16), 0.75), ((30, 16, 16), 0.5),
                                        ((12, 12, 12), 1.0)])
def test_mixed_counts_and_rates(per, side, space):
    _compare(per, side, space, False)


@pytest.mark.parametrize("per", [2, 4, 6])
@pytest.mark.parametrize("side,space", [((12, 70, 12), 1.0), ((16, 30, 16), 0.5)])
def test_with_a_piston(per, side, space):
    _compare(per, side, space, True)


def _compare(per, side, space, wall):
    print(f"[case] few images per={per} side={side} space={space} wall={wall}", flush=True)
    w = ci.jittered_block(*side, seed=sum(side) + per, amp=0.2)
    rng = np.random.default_rng(per)
    for a in ("vx", "vy", "vz"):
        setattr(w, a, rng.normal(0.0, 0.1, w.n))
    box = tuple(s * space for s in side)
    for a, name in enumerate("xyz"):
        q = getattr(w, name) * space
        if (per >> a) & 1:
            q = np.mod(q, box[a])
            q[q >= box[a]] = 0.0
        setattr(w, name, q)
    over = dict(periodic=per, box=((0.0, 0.0, 0.0), box), cell_size=1.0)
    if wall:
        over["wall"] = (0.6, 0.5)
    out = {}
    for prec in ("fp64", "mixed"):
        params = P.Params.from_workload(w, precision=prec, **over)
        out[prec] = P.csph_rates(P.state_from_workload(w, params, DEV), params)
    assert torch.equal(out["fp64"]["nbr_count"], out["mixed"]["nbr_count"])
    vmax = max(float(out["fp64"][k].abs().max()) for k in RATES[1:4])
    for k in RATES:
        den = vmax if k.startswith("dv") else float(out["fp64"][k].abs().max())
        err = float((out["mixed"][k] - out["fp64"][k]).abs().max()) / den
        assert err <= 2e-5, (k, err)
