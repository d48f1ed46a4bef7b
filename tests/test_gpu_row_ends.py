"""The FP32 walk takes i's own row in two parts around i: neighbour counts where i is the row's
first, last or only particle, or shares its place, equal a brute-force count, for rows of one to
a few chunks of candidates and for a set off the mesh it is given.  The step's totals, summed in
waves, equal exactly rounded sums at the block counts where their tree can go wrong."""
import math

import numpy as np
import pytest
import torch

import csph_inputs as ci
import paper_1805_05128_amd as P

pytestmark = pytest.mark.gpu
DEV = "cuda"


def brute_counts(p, H):
    d = p[:, None, :] - p[None, :, :]
    r2 = (d[..., 0] * d[..., 0] + d[..., 1] * d[..., 1]) + d[..., 2] * d[..., 2]
    return (r2 < H * H).sum(1) - 1


@pytest.mark.parametrize("n", [1, 2, 3, 4, 7, 64, 65, 130])
@pytest.mark.parametrize("step,cell", [(1.0, 1.0), (0.25, 1.0), (0.05, 0.0), (0.0, 1.0)])
def test_counts_along_one_row(n, step, cell):
    print(f"[case] one row n={n} step={step} cell={cell}", flush=True)
    w = ci.jittered_block(n, 1, 1, seed=5, amp=0.0)
    rng = np.random.default_rng(n)
    w.x = 0.5 + step * rng.permutation(n).astype(float)
    params = P.Params.from_workload(w, precision="mixed", cell_size=cell)
    out = P.csph_rates(P.state_from_workload(w, params, DEV), params)
    ref = brute_counts(np.stack([w.x, w.y, w.z], 1), params.kappa * params.h)
    assert np.array_equal(out["nbr_count"].cpu().numpy(), ref)
    for k in ("drho", "dvx", "dvy", "dvz", "dE"):
        assert torch.isfinite(out[k]).all()


@pytest.mark.parametrize("n", [1, 2, 255, 257, 65_537, 196_609, 262_145, 300_007])
def test_totals_are_the_exact_sums(n):
    print(f"[case] totals n={n}", flush=True)
    g = torch.Generator().manual_seed(n)
    u = lambda lo, hi: (lo + (hi - lo) * torch.rand(n, dtype=torch.float64, generator=g)).to(DEV)
    side = int(round(n ** (1 / 3))) + 1
    i = torch.arange(n, dtype=torch.float64, device=DEV)
    pos = dict(x=i % side, y=torch.floor(i / side) % side, z=torch.floor(i / side ** 2))
    f = dict(pos, vx=u(-1, 1), vy=u(-1, 1), vz=u(-1, 1), rho=u(0.9, 1.1), E=u(3.0, 4.0),
             m=u(0.5, 1.5))
    s = P.State(f, torch.zeros(n, dtype=torch.int32, device=DEV), None, None)
    params = P.Params(eos=[(P.EOS_IDEAL, 1.4, 0.0)], precision="mixed", h=1.5, kappa=2.0,
                      cell_size=1.0, cfl=0.1, reorder=False)
    sc = P.StepScalars(DEV)
    out = P.csph_step(s, params, sc)
    m = out["m"].cpu().numpy()
    tot = sc.totals.cpu().numpy().reshape(-1, 2)
    for k, a in enumerate((None, "vx", "vy", "vz", "E")):
        t = m if a is None else m * out[a].cpu().numpy()
        exact = math.fsum(t)
        # double-double sums of n rounded terms: the low parts' own roundings only
        assert abs((tot[k, 0] - exact) + tot[k, 1]) <= 2.0 ** -52 * abs(exact) + \
            n * 2.0 ** -104 * np.abs(t).sum(), (k, tot[k], exact)
