"""The tabulated pair sum over blocks (each pair once, the j's going round the
wave) at the edges of blocks and superblocks, over table and mesh sizes,
densities and particles on faces: against the plain
sum of the minimum-image Newtonian terms and the plan's own interpolated
correction at every pair's separation, in FP64. The two form the same terms,
so only rounding of sums of n terms is left: 1e-12 in norm."""
import numpy as np
import pytest

from paper_1510_07621_amd import ics

from _gpu import dev, host, plan, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,E", [(16, 8), (32, 64), (64, 16)])
@pytest.mark.parametrize("kind,n", [("uniform", 63), ("uniform", 65), ("uniform", 513),
                                    ("uniform", 1100), ("clustered", 901), ("faces", 130)])
def test_block_sum_equals_the_plain_sum(grid, E, kind, n):
    require_gpu()
    box = 2.0
    rng = np.random.default_rng(n + grid)
    pos = ics.uniform(n, box, seed=n)
    if kind == "clustered":      # one crowded column, one crowded cell, the rest spread
        pos[:2, :300] = (np.array([3.0, grid - 1.0])[:, None] + rng.random((2, 300))) * box / grid
        pos[:, 300:500] = (np.array([9.0, 0.0, 5.0])[:, None] + rng.random((3, 200))) * box / grid
    if kind == "faces":          # on cell faces, half the box apart, next to the box's faces
        pos[:, :64] = rng.integers(0, grid, (3, 64)) * (box / grid)
        pos[:, 64:80] = np.mod(pos[:, :16] + box / 2, box)
        pos[:, 80:90] = np.nextafter(box, 0)
    m = rng.uniform(0.5, 1.5, n) / n
    eps = 1e-3 * box
    d = pos[:, :, None] - pos[:, None, :]
    d -= box * np.rint(d / box)
    with plan(grid, n, "fp64", box=box, softening=eps, ewald_gridsize=E) as P:
        got = host(P.pp_ewald_force(dev(pos), dev(m)))
        c = host(P.ewald_correction(dev(d.reshape(3, -1)))).reshape(3, n, n)
    r2 = (d * d).sum(0)
    pair = np.where(r2 > 0, d / np.where(r2 > 0, r2 + eps * eps, 1.0) ** 1.5 + c, 0.0)
    want = -m * (pair * m).sum(2)
    # (a separation of exactly half the box may take either sign)
    ok = (np.abs(np.abs(d) - box / 2) > 1e-12 * box).all(axis=(0, 2))
    assert ok.sum() >= n // 4
    err = np.linalg.norm((got - want)[:, ok]) / np.linalg.norm(want[:, ok])
    assert err <= 1e-12, err


@pytest.mark.parametrize("n", [65536, 65537])
def test_both_sides_of_the_block_sums_line(n):
    """Up to 65536 particles by blocks, above from both sides: sampled
    particles against the plain sum, to n rounding errors of the terms."""
    require_gpu()
    pos = ics.uniform(n, 1.0, seed=n)
    m = np.random.default_rng(n).uniform(0.5, 1.5, n) / n
    eps = 1e-3
    tg = np.array([0, 1, 511, 512, 40000, n - 2, n - 1])
    d = pos[:, tg, None] - pos[:, None, :]
    d -= np.rint(d)
    with plan(32, n, "fp64", softening=eps, ewald_gridsize=16) as P:
        got = host(P.pp_ewald_force(dev(pos), dev(m)))[:, tg]
        c = host(P.ewald_correction(dev(np.ascontiguousarray(d.reshape(3, -1))))).reshape(d.shape)
    r2 = (d * d).sum(0)
    pair = np.where(r2 > 0, d / np.where(r2 > 0, r2 + eps * eps, 1.0) ** 1.5 + c, 0.0) * m
    size = m[tg] * np.sqrt((pair * pair).sum(0)).sum(1)
    err = np.sqrt(((got + m[tg] * pair.sum(2)) ** 2).sum(0))
    assert (err <= n * 2.0 ** -53 * size).all(), err / size


@pytest.mark.parametrize("n", [1, 3, 65, 700])
def test_particles_next_to_the_origin(n):
    """Without softening, a particle next to the origin but not on it: the
    places past the last particle, which the blocks fill with no mass at the
    origin, add nothing to it (its weight with them would overflow)."""
    require_gpu()
    pos = ics.uniform(n, 1.0, seed=n)
    pos[:, 0] = (1e-120, 0.0, 1e-130)
    m = np.random.default_rng(n).uniform(0.5, 1.5, n) / n
    d = pos[:, :, None] - pos[:, None, :]
    d -= np.rint(d)
    with plan(16, n, "fp64", softening=0.0, ewald_gridsize=16) as P:
        got = host(P.pp_ewald_force(dev(pos), dev(m)))
        c = host(P.ewald_correction(dev(d.reshape(3, -1)))).reshape(3, n, n)
    r2 = (d * d).sum(0)
    pair = np.where(r2 > 0, d / np.where(r2 > 0, r2, 1.0) ** 1.5 + c, 0.0)
    want = -m * (pair * m).sum(2)
    assert np.isfinite(got).all(), got[:, ~np.isfinite(got).all(axis=0)]
    assert np.linalg.norm(got - want) <= 1e-12 * np.linalg.norm(want)
