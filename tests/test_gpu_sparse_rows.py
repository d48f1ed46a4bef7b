"""The neighbour export of large sparse sets (a lane a particle, dense spots by the whole wave)
equals that of the same set on coarse cells (a wave a particle throughout)."""
import numpy as np
import pytest
import torch

import csph_inputs as ci
import paper_1805_05128_amd as P

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _set(n, clusters, order, side=240.0):
    """A thin cloud with clusters of the given sizes, each within a third of the support."""
    w = ci.random_cloud(n, seed=n, box=side)
    rng = np.random.default_rng(3)
    k = 0
    for c in clusters:
        at = rng.uniform(3.0, side - 3.0, 3)
        if c > 400:
            at = np.full(3, 1.5)  # at the corner: periodic images of a dense spot
        for a, q in zip("xyz", at):
            getattr(w, a)[k:k + c] = q + rng.uniform(-0.5, 0.5, c)
        k += c
    o = rng.permutation(n) if order == "shuffled" else np.arange(n)
    for a in ("x", "y", "z"):
        setattr(w, a, np.ascontiguousarray(getattr(w, a)[o]))
    return w


# neighbours of a lane's own list (16) and one more, candidates of a lane's walk (96) and one more
@pytest.mark.parametrize("n", [1 << 17, 131135, 200003])
@pytest.mark.parametrize("mode", ["open", "pair", "periodic", "pair_periodic"])
@pytest.mark.parametrize("order", ["clustered", "shuffled"])
def test_equal_on_coarse_cells(n, mode, order):
    w = _set(n, [16, 17, 18, 17, 60, 95, 96, 97, 98, 130, 700] + 300 * [17, 2, 5], order)
    over = {}
    if "pair" in mode:
        over["h_mode"] = "pair"
    if "periodic" in mode:
        over.update(periodic=7, box=((0.0, 0.0, 0.0), (240.0, 240.0, 240.0)))
    out = []
    for cell in (0.0, 1.6, 24.0):  # the support; a reach of 2; coarse: the wave a particle
        params = P.Params.from_workload(w, cell_size=cell, **over)
        st = P.state_from_workload(w, params, DEV)
        if "pair" in mode:
            st.d = torch.as_tensor(np.random.default_rng(1).uniform(1.2, 1.5, n), device=DEV)
        out.append(P.csph_neighbors(st, params))
    assert int((out[2][0][1:] - out[2][0][:-1]).max()) >= 699
    for off, idx in out[:2]:
        assert torch.equal(off, out[2][0]) and torch.equal(idx, out[2][1])


def test_thin_sets_cost_less_than_dense_ones():
    def ms(side):
        w = ci.random_cloud(1000000, seed=1, box=side)
        params = P.Params.from_workload(w, cell_size=0.0)
        st = P.state_from_workload(w, params, DEV)
        ws = P.Workspace(DEV)
        P.csph_neighbors(st, params, ws=ws)
        best = np.inf
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            P.csph_neighbors(st, params, ws=ws)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    # a wave a particle took 1.38 ms for 0.3 neighbours each, 1.47 ms for 11
    thin, dense = ms(700.0), ms(215.0)
    assert thin <= 0.75 * dense, (thin, dense)
