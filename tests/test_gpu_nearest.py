"""Generators near a wave: the pruned ownership scan equals the full one (FP64 argmin in the same
operations, ties to the smaller index) for particles in cell order and shuffled, far from the
origin, tied, tiny, huge and not finite, at the edges of its generator ranges; the statistics of
owners that are not the nearest generator equal the oracle's; the generator move with more
triplets than a wave has lanes equals the oracle's."""
import numpy as np
import pytest
import torch

from oracle import balance as B
import paper_1805_05128_amd as P

pytestmark = pytest.mark.gpu
DEV = "cuda"


def dev(a, dt=np.float64):
    return torch.as_tensor(np.ascontiguousarray(a, dt), device=DEV)


def full_scan(p, g):
    best, bd = np.zeros(len(p), np.int64), np.full(len(p), np.inf)
    with np.errstate(all="ignore"):
        for k in range(len(g)):
            d = p - g[k]
            d2 = (d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1]) + d[:, 2] * d[:, 2]
            closer = d2 < bd
            bd[closer], best[closer] = d2[closer], k
    return best


def particles(kind, n, rng):
    i = np.arange(n)
    p = np.stack([i % 37, (i // 37) % 11, i // 407], 1) + 0.5  # rows along x, as in cell order
    if kind == "shuffled":
        p = p[rng.permutation(n)] + rng.uniform(-0.4, 0.4, (n, 3))
    elif kind == "far":
        p = p + rng.uniform(-0.4, 0.4, (n, 3)) + np.array([1e7, -3e6, 5e8])
    elif kind == "tiny":
        p = p * 1e-25
    elif kind == "huge":
        p = p * 1e25
    elif kind == "odd":
        p = p + rng.uniform(-0.4, 0.4, (n, 3))
        p[::97, 0] = np.nan
        p[5::131, 1] = np.inf
        p[7::173, 2] = -1e200
    return p


@pytest.mark.parametrize("K", [1, 11, 12, 64, 65, 1024])
@pytest.mark.parametrize("kind", ["rows", "shuffled", "far", "tiny", "huge", "odd"])
def test_owner_equals_full_scan(kind, K):
    n = 12345
    print(f"[case] nearest {kind} K={K}", flush=True)
    rng = np.random.default_rng(K)
    p = particles(kind, n, rng)
    fin = p[np.isfinite(p).all(1) & (np.abs(p).max(1) < 1e150)]
    g = fin[rng.integers(0, len(fin), K)]  # on lattice points: ties between generators
    if K > 2:
        g[K // 2] = g[0]  # and a duplicate
    cnt = rng.integers(0, 200, n)
    owner, part, pairs = P.voronoi_assign(dev(p[:, 0]), dev(p[:, 1]), dev(p[:, 2]), dev(g),
                                          dev(cnt, np.int32))
    ref = full_scan(p, g)
    assert np.array_equal(owner.cpu().numpy(), ref)
    assert np.array_equal(part.cpu().numpy(), np.bincount(ref, minlength=K))
    assert np.array_equal(pairs.cpu().numpy(),
                          np.bincount(ref, weights=cnt, minlength=K).astype(np.int64))


@pytest.mark.parametrize("K", [2, 12, 65])
@pytest.mark.parametrize("kind", ["rows", "shuffled", "far"])
def test_stats_of_any_owner(kind, K):
    n = 5003
    print(f"[case] stats {kind} K={K}", flush=True)
    rng = np.random.default_rng(100 + K)
    p = particles(kind, n, rng)
    g = p[rng.integers(0, n, K)] + rng.uniform(-0.3, 0.3, (K, 3))
    owner = full_scan(p, g).astype(np.int32)
    owner[::13] = rng.integers(-1, K + 1, len(owner[::13]))
    cnt = rng.integers(0, 200, n)
    ref = B.stats(p[:, 0], p[:, 1], p[:, 2], owner, g, 2.0, cnt)
    got = P.csph_balance_stats(dev(p[:, 0]), dev(p[:, 1]), dev(p[:, 2]), dev(owner, np.int32),
                               dev(g), 2.0, nbr_count=dev(cnt, np.int32))
    assert np.array_equal(got["particles"].cpu().numpy(), ref["particles"])
    assert np.array_equal(got["pairs"].cpu().numpy(), ref["pairs"])
    assert np.array_equal(P.adjacency_matrix(got["adjacency"], K).numpy(), ref["adjacency"])
    c = got["centre"].cpu().numpy()
    assert np.all(np.abs(c - ref["centre"]) <= 1e-9 + 1e-13 * np.abs(ref["centre"]))


@pytest.mark.parametrize("K", [1, 2, 33, 65])
def test_move_all_touching(K):
    print(f"[case] move K={K}", flush=True)
    rng = np.random.default_rng(K)
    g = rng.uniform(0.0, 40.0, (K, 3))
    loads = rng.integers(1, 1000, K)
    centre = g + rng.uniform(-1.0, 1.0, (K, 3))
    adj = ~np.eye(K, dtype=bool)
    bits = np.zeros((K, (K + 31) // 32), np.uint32)
    for k, l in zip(*np.nonzero(adj)):
        bits[k, l >> 5] |= np.uint32(1 << (l & 31))
    ref, ref_ms = B.move(g, loads, centre, adj, B.BalanceParams(sigma=0.5, theta=0.25, gamma=1.0,
                                                                dsh=3.0, load="particles"))
    stats = dict(particles=dev(loads, np.int64), pairs=None, centre=dev(centre),
                 adjacency=torch.as_tensor(bits.view(np.int32), device=DEV))
    new, ms = P.csph_balance_move(dev(g), stats, P.BalanceParams(sigma=0.5, theta=0.25, gamma=1.0,
                                                                 dsh=3.0, load="particles"))
    # the rotations' axes are cross products of nearly parallel vectors for some triplets: the
    # existing move test's 1e-12 of the coordinates' scale, times the K^2/2 triplets of a sum
    assert np.abs(new.cpu().numpy() - ref).max() <= 1e-12 * 40.0 * max(1, K * K // 2)
    assert abs(float(ms.item()) - ref_ms) <= 1e-11 * max(ref_ms, 1.0) * max(1, K * K // 2)
