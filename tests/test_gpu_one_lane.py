"""FP64 rates and step VJPs with one lane a particle (more than 131 072 of them), periodic along the
rows, in pair-h mode and across a piston: k exact copies of a set, far apart along its open axis, equal
the set alone, which runs several lanes a particle and is compared with the oracle elsewhere.  Long
rows have a few particles near each periodic face (their images walked by the whole wave); the
crowded layer overflows that walk's lists, and short rows have too many such particles, so the
lock-step walk takes over."""
import copy

import numpy as np
import pytest
import torch

import csph_inputs as ci
import paper_1805_05128_amd as P
from helpers import to_np

pytestmark = pytest.mark.gpu
DEV = "cuda"
RATES = ("drho", "dvx", "dvy", "dvz", "dE")


def _base(side, crowd):
    """A jittered lattice; crowd: and a denser layer at the far end of its first two axes, whose
    images the few particles at the near end meet by the hundred."""
    w = ci.jittered_block(*side, seed=7, amp=0.2)
    rng = np.random.default_rng(1)
    if crowd:
        extra = ci.jittered_block(*side, seed=8, amp=0.2)
        keep = (extra.x > side[0] - 2.0) | (extra.y > side[1] - 2.0)
        more = [keep] * 4
        for f in ("x", "y", "z", "vx", "vy", "vz", "rho", "p", "m", "mat"):
            a = getattr(extra, f)
            setattr(w, f, np.concatenate([getattr(w, f)] + [a[m] for m in more]))
    for a, s in zip("xyz", side):
        q = getattr(w, a) + (rng.uniform(-0.4, 0.4, w.n) if crowd else 0.0)
        # multiples of 2^-30, so that a copy 64 k away has the same offsets to the last bit
        q = np.round(np.mod(q, s) * 2.0 ** 30) / 2.0 ** 30
        q[q >= s] = 0.0
        setattr(w, a, q)
        setattr(w, "v" + a, rng.normal(0.0, 0.1, w.n))
    return w


def _copies(base, k):
    w = copy.copy(base)
    for f in ("x", "y", "z", "vx", "vy", "vz", "rho", "p", "m", "mat"):
        setattr(w, f, np.tile(getattr(base, f), k))
    w.z = w.z + 64.0 * np.repeat(np.arange(k), base.n)
    return w


@pytest.mark.parametrize("periodic,wall", [(3, None), (1, None), (2, None), (2, (0.4, 0.5)),
                                           (0, (0.4, 0.5))])
@pytest.mark.parametrize("pair", [False, True])
@pytest.mark.parametrize("side,crowd,k", [((70, 71, 3), False, 10), ((68, 66, 3), True, 10),
                                          ((24, 17, 12), False, 28)])
def test_copies_equal_one(side, crowd, k, pair, periodic, wall):
    print(f"[case] {side} {crowd} pair={pair} periodic={periodic} wall={wall}", flush=True)
    base = _base(side, crowd)
    assert base.n <= 131072 < k * base.n
    rng = np.random.default_rng(2)
    cot = {f: rng.standard_normal(base.n) for f in P.GRAD_FIELDS}
    d = rng.uniform(1.35, 1.5, base.n)
    box = ((0.0, 0.0, 0.0), tuple(map(float, side)))
    over = dict(periodic=periodic, box=box if periodic else None, wall=wall, reorder=False,
                h_mode="pair" if pair else "fixed", cell_size=1.0)

    def run(w, reps):
        params = P.Params.from_workload(w, **over)
        st = P.state_from_workload(w, params, DEV)
        if pair:
            st.d = torch.as_tensor(np.tile(d, reps), device=DEV)
        out = P.csph_rates(st, params, t=0.1)
        g = {f: torch.as_tensor(np.tile(cot[f], reps), device=DEV) for f in P.GRAD_FIELDS}
        gr, ge = P.csph_step_vjp(st, params, 0.01, g, P.zeros_grad(w.n, DEV), t=0.1)
        out.update({"g" + f: gr[f] for f in P.GRAD_FIELDS})
        return {f: to_np(u).reshape(reps, -1) for f, u in out.items() if torch.is_tensor(u) and
                u.numel() == w.n}, to_np(ge) / reps

    one, ge1 = run(base, 1)
    many, gek = run(_copies(base, k), k)
    assert np.array_equal(many["nbr_count"], np.tile(one["nbr_count"], (k, 1)))
    vmax = max(np.abs(one[f]).max() for f in RATES[1:4])
    for f in RATES + ("signal",) + tuple("g" + f for f in P.GRAD_FIELDS):
        # the same terms added in another order, up to ~1 000 of them
        scale = vmax if f in RATES[1:4] else np.abs(one[f]).max()
        assert np.abs(many[f] - one[f]).max() <= 1e-11 * scale, f
    assert np.allclose(gek, ge1, rtol=1e-10, atol=1e-10 * np.abs(ge1).max())
