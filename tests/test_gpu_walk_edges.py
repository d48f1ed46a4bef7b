"""Edges of the pair walks: neighbour rows at the limits of the export's LDS lists, FP64 rates
and adjoints at every number of lanes per particle, against the CPU oracle or against the same
set alone."""
import numpy as np
import pytest
import torch

import csph_inputs as ci
import oracle as O
import paper_1805_05128_amd as P
from helpers import RATE_FIELDS, field_relerr, rates_np, to_np

pytestmark = pytest.mark.gpu

DEV = "cuda"
FP64_TOL = 1e-12


def _neighbours(w, **over):
    params = P.Params.from_workload(w, **over)
    off, idx = P.csph_neighbors(P.state_from_workload(w, params, DEV), params)
    cfg = {k: v for k, v in over.items() if k in ("h",)}
    ro, ri = O.neighbors(O.cfg_for(w, **cfg), w.x, w.y, w.z, None)
    assert np.array_equal(to_np(off), ro)
    assert np.array_equal(to_np(idx), ri)
    return ro


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 512, 513, 514])
def test_neighbors_row_lengths(n):
    """Every particle the neighbour of all others: rows of n - 1 entries, around a wave and
    around the longest row ranked in LDS (512)."""
    ro = _neighbours(ci.random_cloud(n, seed=n, box=1.0))
    assert np.diff(ro).tolist() == [n - 1] * n


@pytest.mark.parametrize("cell,box", [(0.62, 6.0), (0.5, 2.4), (0.31, 5.0), (3.0, 3.0), (1.0, 9.0)])
def test_neighbors_row_batches(cell, box):
    """Stencils of 9 to 441 rows (64 at a time), rows of one to hundreds of candidates, more
    candidates than one list holds."""
    _neighbours(ci.random_cloud(2600, seed=3, box=box), cell_size=cell)


def test_neighbors_periodic_small_cells():
    _neighbours(ci.periodic_block(9, 8, 11, seed=6, amp=0.3), cell_size=0.7)


def _copies(base, k):
    """k copies of a set, far apart along x."""
    import copy
    w = copy.copy(base)
    for f in ("x", "y", "z", "vx", "vy", "vz", "rho", "p", "m", "mat"):
        setattr(w, f, np.tile(getattr(base, f), k))
    w.x = w.x + 40.0 * np.repeat(np.arange(k), base.n)
    return w


@pytest.mark.parametrize("cell", [0.0, 1.0])
@pytest.mark.parametrize("side", [(11, 9, 8), (33, 29, 21), (41, 33, 31), (60, 41, 30), (71, 47, 43)])
def test_rates_fp64_lanes_per_particle(side, cell):
    """16, 8, 4, 2 and 1 lanes per particle, candidates dealt out by rows (unit cells) and
    within rows (cells of the support)."""
    w = ci.jittered_block(*side, seed=5, amp=0.2, v=(0.1, -0.2, 0.05))
    w.vx = w.vx + 0.1 * np.sin(w.y)
    params = P.Params.from_workload(w, cell_size=cell)
    out = P.csph_rates(P.state_from_workload(w, params, DEV), params)
    ref = O.rates(O.cfg_for(w, search=1), O.state_from(w, O.cfg_for(w)))
    err = field_relerr(rates_np(out), ref)
    assert max(err[k] for k in RATE_FIELDS) <= FP64_TOL, err
    assert np.array_equal(to_np(out["nbr_count"]).astype(np.int64), ref["nbr_count"])
    assert np.abs(to_np(out["signal"]) / ref["signal"] - 1.0).max() <= FP64_TOL


@pytest.mark.parametrize("wall,periodic", [(False, 0), (True, 0), (False, 6)])
@pytest.mark.parametrize("cell", [0.0, 1.0])
@pytest.mark.parametrize("k", [18, 35, 70, 133])
def test_step_vjp_lanes_per_particle(k, cell, wall, periodic):
    """A step's VJP of k far copies of one set (8, 4, 2 and 1 lanes per particle) equals that of
    the set alone (16 lanes) up to the order of the additions."""
    base = ci.jittered_block(12, 10, 9, seed=8, amp=0.2, v=(-0.3, 0.1, 0.05))
    base.vx = base.vx + 0.1 * np.sin(base.z)
    rng = np.random.default_rng(2)
    cot = {f: rng.standard_normal(base.n) for f in P.GRAD_FIELDS}
    if wall:  # the copies would need a wall each: stack them along y instead
        base.wall = (0.45, 0.4)
    if periodic:
        base.periodic = periodic
        base.box = ((0.0, 0.0, 0.0), (1.0, 10.0, 9.0))
        base.y, base.z = base.y % 10.0, base.z % 9.0

    def grad(w, reps):
        params = P.Params.from_workload(w, cell_size=cell, reorder=False)
        st = P.state_from_workload(w, params, DEV)
        g = {f: torch.as_tensor(np.tile(cot[f], reps), device=DEV) for f in P.GRAD_FIELDS}
        out, ge = P.csph_step_vjp(st, params, 0.05, g, P.zeros_grad(w.n, DEV))
        return {f: to_np(out[f]).reshape(reps, base.n) for f in P.GRAD_FIELDS}, to_np(ge) / reps

    one, ge1 = grad(base, 1)
    many = _copies(base, k)
    if wall:
        many.x = np.tile(base.x, k)
        many.y = many.y + 40.0 * np.repeat(np.arange(k), base.n)
    got, gek = grad(many, k)
    for f in P.GRAD_FIELDS:
        scale = np.abs(one[f]).max()
        # positions 40 k from the origin carry an absolute error of ulp(40 k) = 1e-12, which
        # reaches the gradients through offsets of order one
        assert np.abs(got[f] - one[f]).max() <= 2e-9 * scale, f
    assert np.allclose(gek, ge1, rtol=1e-8, atol=1e-9 * np.abs(ge1).max())


@pytest.mark.parametrize("key_mode", ["linear", "morton"])
@pytest.mark.parametrize("n,box,cell", [(1, 1.0, 0.5), (1023, 5.0, 0.7), (1025, 9.0, 1.0),
                                        (8192, 24.0, 1.0), (16384, 20.0, 0.85),
                                        (16384, 25.0, 1.0), (16385, 20.0, 1.0),
                                        (5000, 1.9, 1.0), (300, 24.9, 1.0)])
def test_bin_sizes(n, box, cell, key_mode):
    """Binning at the limits of its one-workgroup form (16 384 particles, fewer than 16 384 keys,
    64 particles a key) equals the stable sort by key."""
    w = ci.random_cloud(n, seed=n, box=box)
    params = P.Params.from_workload(w, cell_size=cell, key_mode=key_mode)
    x, y, z = (torch.as_tensor(a, device=DEV) for a in (w.x, w.y, w.z))
    g = P.csph_grid_build(x, y, z, params)
    key, perm, start = P.csph_bin(x, y, z, g)
    key, perm, start = to_np(key), to_np(perm), to_np(start)
    c = [np.clip(np.floor((a - g.origin[k]) * g.inv_cell), 0, g.dims[k] - 1).astype(np.int64)
         for k, a in enumerate((w.x, w.y, w.z))]
    if key_mode == "linear":
        ref = (c[2] * g.dims[1] + c[1]) * g.dims[0] + c[0]
    else:
        ref = sum(((c[a] >> b) & 1) << (3 * b + a) for a in range(3) for b in range(10))
    assert np.array_equal(key, ref)
    assert np.array_equal(perm, np.argsort(ref, kind="stable"))
    assert np.array_equal(start, np.searchsorted(np.sort(ref), np.arange(g.nkey + 1)))


@pytest.mark.parametrize("in_place", [True, False])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_step_kept_order_equals_renumbered(precision, in_place):
    """A step that keeps the caller's order writes what the renumbering step writes, bit for bit,
    at the particles' places, with materials, ids and counts; other arrays stay whole."""
    w = ci.random_cloud(3000, seed=9, box=14.0, n_mat=2)
    w.wall = (0.0, 0.2)
    over = dict(precision=precision, cell_size=1.0)
    pr = P.Params.from_workload(w, **over)
    pk = P.Params.from_workload(w, reorder=False, **over)
    st = P.state_from_workload(w, pr, DEV)
    counts = [torch.empty(w.n, dtype=torch.int32, device=DEV) for _ in range(2)]
    scal = [P.StepScalars(DEV, t0=0.1) for _ in range(2)]
    a = P.csph_step(st, pr, scal[0], nbr_count=counts[0])
    kept = st if in_place else st.like()
    b = P.csph_step(st, pk, scal[1], s_out=kept, nbr_count=counts[1])
    order = a["id"]
    assert torch.equal(torch.sort(order).values, torch.arange(w.n, device=DEV))
    for f in P.GRAD_FIELDS + ("m", "mat", "id"):
        assert torch.equal(a[f], b[f][order]), f
    assert torch.equal(counts[0], counts[1][order])
    assert torch.equal(scal[0].dt, scal[1].dt) and torch.equal(scal[0].totals, scal[1].totals)
