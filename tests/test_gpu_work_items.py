"""How the short-range sum is cut into work items: small sets share an item's
stencil among several waves (8, 4 or 2 of them by the particle number) and
take smaller chunks of i-particles; plans with pair_partials > 0 evaluate
pairs of dense groups once only above a particle number. Both sides of every
line are compared with the oracle, held to the bars of the short-range sum
(FP64 1e-12, FP32 1e-5 RMS; the adjoint 1e-9 and 1e-4).
"""
import numpy as np
import pytest

from oracle import adjoint, metrics
from oracle import pp as o_pp
from paper_1510_07621_amd import ics

from _gpu import dev, host, plan, require_gpu, sample_targets

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


# (n, grid): one particle more or less than a chunk, and both sides of the
# lines at 8192, 24576, 65536 and 393216 particles (with at least 16 a group)
@pytest.mark.parametrize("n,grid", [(15, 16), (17, 16), (1024, 16), (8191, 16), (8193, 16), (24577, 16),
                                    (65536, 32), (65537, 32), (393217, 64)])
@pytest.mark.parametrize("precision,tol,vjp_tol", [("fp64", 1e-12, 1e-9), ("fp32", 1e-5, 1e-4)])
def test_cut_items_match_the_oracle(n, grid, precision, tol, vjp_tol):
    rng = np.random.default_rng(n)
    dense = ((np.array([5, 9, 15])[:, None] + rng.random((3, min(300, n // 3)))) / grid)
    pos = np.concatenate([dense, ics.uniform(n - dense.shape[1], seed=n)], axis=1)
    m = rng.uniform(0.5, 1.5, n) / n
    lam = rng.normal(size=(3, n))
    r_s = 1.25 / grid
    eps = 0.03 / n ** (1 / 3)
    tg = np.unique(np.concatenate([np.arange(min(8, n)), sample_targets(pos, 160)]))
    ref = o_pp.pp_accel(pos, m, 1.0, r_s, 4.5 * r_s, eps, targets=tg, method="kdtree") * m[tg]
    ref_v = adjoint.pp_vjp(pos, m, 1.0, r_s, 4.5 * r_s, eps, lam, targets=tg)
    with plan(grid, n, precision, softening=eps, adjoint=True) as P:
        F = host(P.pp_force(dev(pos), dev(m)))[:, tg]
        g = host(P.pp_force_vjp(dev(pos), dev(m), dev(lam)))[:, tg]
    assert metrics.force_errors(F, ref)["rms"] <= tol
    assert metrics.force_errors(g, ref_v)["rms"] <= vjp_tol


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32", 1e-5)])
@pytest.mark.parametrize("kind,n,grid", [("force", 3200001, 128), ("vjp", 400001, 64),
                                         ("vjp", 2700001, 128)])
def test_one_sided_above_its_line(precision, tol, kind, n, grid):
    """Above the line the one-sided sum, with enough partials and with too few
    (the call then falls back on the device), equals the two-sided sum: dense
    cells of several chunks, one across the z face, over a uniform
    background, per-particle masses."""
    rng = np.random.default_rng(91)
    cells = [([5, 9, grid - 1], 300), ([5, 9, 0], 700), ([6, 10, grid - 3], 500)]
    dense = np.concatenate([(np.array(c)[:, None] + rng.random((3, k))) / grid for c, k in cells],
                           axis=1)
    pos = np.concatenate([dense, ics.uniform(n - dense.shape[1], seed=92)], axis=1)
    m = rng.uniform(0.5, 1.5, n) / n
    x, md = dev(pos), dev(m)
    lam = dev(rng.normal(size=(3, n)))
    out = []
    for partials in (0, 80, 1):
        with plan(grid, n, precision, softening=0.02 / grid, adjoint=kind == "vjp",
                  pair_partials=partials) as P:
            out.append(host(P.pp_force(x, md) if kind == "force" else P.pp_force_vjp(x, md, lam)))
    for got in out[1:]:
        assert metrics.force_errors(got, out[0])["global"] <= (1 if kind == "force" else 10) * tol


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32", 1e-5)])
def test_noalloc_follows_its_parameters(precision, tol):
    """pp_force_noalloc keeps the tables of the last parameters: calls that
    change the cutoff, the grid, the softening or the particle number and
    come back equal the plan's force each time, also with a stencil of
    thousands of rows (several launches to hand it over)."""
    from paper_1510_07621_amd import binding
    calls = [(5000, dict(grid_n=32)), (5000, dict(grid_n=32, cutoff_rs=6.0)),
             (3001, dict(grid_n=64, rs_cells=4.0, cutoff_rs=6.0)), (5000, dict(grid_n=32)),
             (5000, dict(grid_n=32, softening=0.3 / 32)), (301, dict(grid_n=32, softening=0.3 / 32))]
    for n, kw in calls:
        prm = binding.Params(precision=precision, **kw)
        x = dev(ics.uniform(n, seed=n))
        got = host(binding.pp_force_noalloc(prm, x, 1.0 / n))
        with binding.Plan(prm, n) as P:
            want = host(P.pp_force(x, 1.0 / n))
        assert metrics.force_errors(got, want)["global"] <= tol
