"""The mesh transforms on both sides of the line between plane passes and
separate z and y passes: planes of every grid up to 64^3 and of 128^3 in FP32,
separate passes of 128^3 in FP64. The mesh force against the oracle, held to the
bars of the mesh path (FP64 1e-10, FP32 1e-4), and the power spectrum to those
of its own (1e-10 and 1e-3 in every shell)."""
import numpy as np
import pytest

from oracle import metrics, powerspec
from oracle import p3m as o_p3m
from paper_1510_07621_amd import ics

from _gpu import dev, host, plan, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,tol,ptol", [("fp64", 1e-10, 1e-10), ("fp32", 1e-4, 1e-3)])
@pytest.mark.parametrize("grid", [16, 32, 64, 128])
def test_planes(grid, precision, tol, ptol):
    require_gpu()
    n, nbins = 3001, grid // 2
    pos = ics.uniform(n, seed=grid)
    m = np.random.default_rng(grid).uniform(0.5, 1.5, n) / n
    with plan(grid, n, precision) as P:
        F = host(P.pm_force(dev(pos), dev(m)))
        _, power, modes, _ = P.power_spectrum(dev(pos), dev(m), nbins=nbins, r_tophat=0.1)
    assert metrics.force_errors(F, o_p3m.pm_force(pos, m, 1.0, grid))["rms"] <= tol
    _, ref, rmodes, _ = powerspec.power_spectrum(pos, m, 1.0, grid, nbins, r_tophat=0.1)
    np.testing.assert_array_equal(host(modes), rmodes)
    np.testing.assert_allclose(host(power)[rmodes > 0], ref[rmodes > 0], rtol=ptol)
