"""Queries over many grains against brute force in FP64: the grain map where
the lists of grains per tile end, overflow or are empty."""
import numpy as np
import pytest

from paper_2504_12858_amd import binding as B
from paper_2504_12858_amd import workloads as W
from tests.gpu_helpers import require_gpu

pytestmark = pytest.mark.gpu

LAM = 5e-6


def _rotations(q):
    w, x, y, z = (q / np.linalg.norm(q, axis=1, keepdims=True)).T
    return np.stack([np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)], 1),
                     np.stack([2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)], 1),
                     np.stack([2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1)], 1)


@pytest.mark.parametrize("n_grains,r,n,periodic", [
    (1, 3, (1, 1, 1), 0), (7, 4, (17, 5, 9), 0), (300, 2, (33, 16, 70), 0),
    (1500, 1, (24, 17, 37), 0), (60, 3, (20, 31, 18), 7)])
def test_grain_map_matches_brute_force(n_grains, r, n, periodic):
    """Octahedral balls of L1 radius r crowded into a 0.2 mm cube; the map
    grid reaches past the box.  Voxels within FP32 rounding of a site
    boundary or of a tie between two grains (3e-4 of a lattice step: several
    ulps of 0.2 mm) are left out."""
    require_gpu()
    L = 2e-4
    g = W.rng(100 + n_grains)
    c = L * (0.05 + 0.9 * g.random((n_grains, 3)))
    q = W.shoemake_quaternions(g, n_grains)
    p = B.make_params((0, 0, 0), (L, L, L), LAM, LAM, LAM, W.KIN_A, W.KIN_B, cap_particles=1 << 16,
                      cap_stopped=1 << 16, cap_grains=2048, cap_claim_bricks=1 << 16,
                      periodic=periodic)
    ctx = B.Context(p)
    ctx.init_grains(c, q, np.full(n_grains, r, np.int32))
    lo = np.array([-0.1 * L] * 3) if not periodic else np.zeros(3)
    sp = (1.2 if not periodic else 1.0) * L / np.array(n)
    got = ctx.grain_map(n, lo, sp).ravel()
    ctx.close()
    k, j, i = np.meshgrid(*(np.arange(m) for m in n[::-1]), indexing="ij")
    y = lo + (np.stack([i, j, k], -1).reshape(-1, 3) + 0.5) * sp
    best, bd = np.zeros(len(y), int), np.full(len(y), np.inf)
    unsure = np.zeros(len(y), bool)
    shifts = [np.zeros(3)] if not periodic else \
        [L * np.array([a, b, d]) for d in (-1, 0, 1) for b in (-1, 0, 1) for a in (-1, 0, 1)]
    R = _rotations(q)
    tol = 3e-4
    for m in range(n_grains):
        for s in shifts:
            l = (y + s - c[m]) @ R[m] / LAM
            S = np.rint(l)
            near = np.abs(l).sum(1) < r + 2
            unsure |= near & (np.abs(np.abs(l - S) - 0.5).min(1) < tol)
            hit = near & (np.abs(S).sum(1) <= r)
            d = np.where(hit, np.linalg.norm(l - S, axis=1), np.inf)
            unsure |= hit & np.isfinite(bd) & (np.abs(d - np.where(np.isfinite(bd), bd, 0)) < tol) & \
                (best != m + 1)
            win = d < bd
            best[win], bd[win] = m + 1, d[win]
    assert unsure.mean() < 0.02 + 1e-5 * n_grains
    assert (best > 0).any() or n_grains == 1
    np.testing.assert_array_equal(got[~unsure], best[~unsure])


@pytest.mark.parametrize("off,n,part,r", [(-1.0, (37, 18, 23), 1.2, 3), (8.0, (37, 18, 23), 1.2, 1),
                                          (64.0, (64, 64, 64), 0.3, 0), (64.0, (64, 64, 64), 0.3, 1)])
def test_grain_map_far_from_the_origin(off, n, part, r):
    """Boxes so far from the origin (up to 1.3e7 site spacings) that positions
    are rounded by as much as the distance between sites: every voxel equals
    the rule in the FP32 arithmetic of the map, tried for every grain."""
    require_gpu()
    L, n_grains = 2e-4, 40
    f4, f8 = np.float32, np.float64
    g = W.rng(7)
    c = off + L * (0.05 + 0.9 * g.random((n_grains, 3)))
    p = B.make_params((off,) * 3, (off + L,) * 3, LAM, LAM, LAM, W.KIN_A, W.KIN_B, cap_particles=1 << 16,
                      cap_stopped=1 << 16, cap_grains=64, cap_claim_bricks=1 << 12)
    ctx = B.Context(p)
    ctx.init_grains(c, W.shoemake_quaternions(g, n_grains), np.full(n_grains, r, np.int32))
    sp = part * L / np.array(n)
    lo = np.full(3, off + 0.5 * L * (1 - part))
    got = ctx.grain_map(n, lo, sp).ravel()
    rows = ctx.grains()
    ctx.close()

    def fma(a, b, x):  # the product is exact in FP64
        return (a.astype(f8) * b.astype(f8) + x.astype(f8)).astype(f4)
    k, j, i = np.meshgrid(*(np.arange(m) for m in n[::-1]), indexing="ij")
    ijk = np.stack([i, j, k], -1).reshape(-1, 3).astype(f4)
    y = lo.astype(f4) + (ijk + f4(0.5)) * sp.astype(f4)
    best, bd = np.zeros(len(y), int), np.full(len(y), np.inf, f4)
    for m, G in enumerate(rows):
        d = y - G[:3]
        s = np.empty_like(y)
        for a in range(3):
            s[:, a] = np.rint(fma(G[10 + a], d[:, 2], fma(G[7 + a], d[:, 1], G[4 + a] * d[:, 0])) *
                              (f4(1) / f4(LAM)))
        x = np.stack([fma(G[13 + 3 * a], s[:, 0], fma(G[14 + 3 * a], s[:, 1],
                                                     fma(G[15 + 3 * a], s[:, 2], G[a]))) for a in range(3)], 1)
        e = y - x
        d2 = (e[:, 0] * e[:, 0] + e[:, 1] * e[:, 1]) + e[:, 2] * e[:, 2]
        win = (np.abs(s).sum(1) <= r) & (d2 < bd)
        best[win], bd[win] = m + 1, d2[win]
    assert (best > 0).any()
    np.testing.assert_array_equal(got, best)


@pytest.mark.parametrize("n_grains,r,n,periodic", [
    (300, 2, (1, 70, 33), 0), (300, 2, (2, 17, 64), 0), (300, 2, (3, 65, 16), 0), (300, 2, (8, 33, 40), 0),
    (300, 2, (9, 33, 40), 0), (1500, 1, (1, 40, 37), 0), (60, 3, (2, 31, 38), 7), (60, 3, (5, 31, 18), 7)])
def test_thin_grain_map_matches_brute_force(n_grains, r, n, periodic):
    """Grids of few voxels along x, whose tiles extend along y and z instead."""
    test_grain_map_matches_brute_force(n_grains, r, n, periodic)
