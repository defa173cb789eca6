"""The mesh deposit at the edges of its split: cells of up to 16 particles are
summed by one thread, fuller ones by a wave, and bricks meet at node planes
(4 x 4 x 16 nodes in FP32, 4 x 4 x 8 in FP64 and for cotangents). The mesh
force and its adjoint against the oracle, held to the bars of the mesh path
(FP64 1e-10 and 1e-9, FP32 1e-4)."""
import numpy as np
import pytest

from oracle import adjoint, metrics
from oracle import p3m as o_p3m
from paper_1510_07621_amd import ics

from _gpu import dev, host, plan, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,tol,vjp_tol", [("fp64", 1e-10, 1e-9), ("fp32", 1e-4, 1e-4)])
@pytest.mark.parametrize("grid", [16, 32])
@pytest.mark.parametrize("crowd", [1, 16, 17, 63, 65, 700])
def test_crowded_cells_on_brick_faces(grid, crowd, precision, tol, vjp_tol):
    require_gpu()
    rng = np.random.default_rng(crowd)
    cells = [(0, 0, 0), (grid - 1,) * 3, (3, 4, 15), (4, 3, 7), (4, 3, 8), (8, 8, grid - 1)]
    pos = np.concatenate([(np.array(c)[:, None] + rng.random((3, crowd))) / grid for c in cells] +
                         [ics.uniform(301, seed=crowd)], axis=1)
    n = pos.shape[1]
    m = rng.uniform(0.5, 1.5, n) / n
    lam = rng.normal(size=(3, n))
    ref = o_p3m.pm_force(pos, m, 1.0, grid)
    ref_v = adjoint.pm_vjp(pos, m, 1.0, grid, 1.25 / grid, lam)
    with plan(grid, n, precision, adjoint=True) as P:
        F = host(P.pm_force(dev(pos), dev(m)))
        g = host(P.pm_force_vjp(dev(pos), dev(m), dev(lam)))
    assert metrics.force_errors(F, ref)["rms"] <= tol
    assert metrics.force_errors(g, ref_v)["rms"] <= vjp_tol
