"""Non-finite data stays with its neighbours in the adjoint: a NaN or an infinity in one particle's
state or cotangent leaves the gradients of every particle outside its support as they are without
it.  Unjittered lattice of spacing 1 and support 3, so that candidates lie exactly on the support
(queued by the FP32 test, turned down by the exact one), with a coincident pair besides."""
import itertools

import numpy as np
import pytest
import torch

import csph_inputs as ci
import paper_1805_05128_amd as P
from helpers import to_np

pytestmark = pytest.mark.gpu
DEV = "cuda"
MODES = {"open": {}, "pair": dict(h_mode="pair"), "periodic": dict(periodic=7),
         "wall": dict(wall=(0.25, 0.4)), "wall_periodic": dict(wall=(0.25, 0.4), periodic=6)}


def _touched(w, bad, wall, periodic, box):
    """The particles within the support of `bad`, of its images and of its mirror images."""
    hit = np.zeros(w.n, bool)
    p = np.stack([w.x, w.y, w.z], 1)
    for k in itertools.product(*[(-1, 0, 1) if (periodic >> a) & 1 else (0,) for a in range(3)]):
        q = p[bad] + np.array(k) * box[1]
        for x in {q[0]} | ({2.0 * wall[0] - q[0]} if wall else set()):
            hit |= (p[:, 0] - x) ** 2 + (p[:, 1] - q[1]) ** 2 + (p[:, 2] - q[2]) ** 2 < 9.0
    hit[bad] = True
    return hit


@pytest.mark.parametrize("where,field,value", [("cotangent", "drho", np.nan),
                                               ("cotangent", "dvy", np.inf),
                                               ("state", "E", np.nan)])
# one lane a particle, and 16
@pytest.mark.parametrize("mode,side", [(m, (14, 13, 12)) for m in MODES] +
                         [(m, (54, 52, 50)) for m in ("open", "periodic")])
def test_others_keep_their_gradients(mode, side, where, field, value):
    print(f"[case] {mode} {side} {where} {field} {value}", flush=True)
    over = dict(MODES[mode])
    box = ((0.0, 0.0, 0.0), tuple(float(s) for s in side))
    if "periodic" in over:
        over["box"] = box
    w = ci.jittered_block(*side, seed=1, amp=0.0, v=(0.1, -0.2, 0.05))
    w.vx = w.vx + 0.1 * np.sin(w.y)
    d = None
    if mode == "pair":
        d = np.full(w.n, 1.5)
    for a in "xyz":  # a coincident pair in the corner, the cell order's first slots
        getattr(w, a)[1] = getattr(w, a)[0]
    params = P.Params.from_workload(w, cell_size=1.0, **over)
    rng = np.random.default_rng(7)
    cot = {k: rng.standard_normal(w.n) for k in ("drho", "dvx", "dvy", "dvz", "dE")}

    def grad(bad):
        st = P.state_from_workload(w, params, DEV)
        if d is not None:
            st.d = torch.as_tensor(d, device=DEV)
        c = {k: torch.as_tensor(v, device=DEV) for k, v in cot.items()}
        if bad is not None:
            (c[field] if where == "cotangent" else st[field])[bad] = value
        return P.csph_rates_vjp(st, params, c, t=0.3)[0]

    clean = grad(None)
    for bad in (0, w.n // 2):
        got = grad(bad)
        keep = ~_touched(w, bad, _wall_at(params, 0.3), over.get("periodic", 0), box)
        assert keep.sum() > w.n // 2
        for f in P.GRAD_FIELDS:
            a, b = to_np(got[f])[keep], to_np(clean[f])[keep]
            # a NaN state's zero impedance takes another instance of the same sums
            assert np.abs(a - b).max() <= 1e-12 * np.abs(b).max(), (bad, f)


def _wall_at(params, t):
    return (params.wall[0] + params.wall[1] * t,) if params.wall else None
