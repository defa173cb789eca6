"""The one-sided pair sum at small sizes, where the library by itself sums
every pair from both sides: plans whose line is moved to zero particles
evaluate pairs of dense groups once. Sets that mix dense and sparse groups,
ragged chunks, a group across the box face, particles of one mass and of
their own, and both tables (a softening wide against a bin takes the one over
r), against the oracle at the bars of the short-range sum (FP32 force 1e-5
RMS, its maximum 100 times that, adjoint 1e-4; FP64 adjoint 1e-9).

The number of partials a call needs is counted here on the host, so that a
plan's capacity is known to be enough, or too small (the call then sums from
both sides on the device).
"""
import functools

import numpy as np
import pytest
import torch

from oracle import adjoint, metrics
from oracle import pm as o_pm
from oracle import pp as o_pp
from paper_1510_07621_amd import ics

from _gpu import dev, host, require_gpu, sample_targets

pytestmark = pytest.mark.gpu

GRID, BOX = 16, 2.7
H = BOX / GRID
R_S = 1.25 * H
R_C = 4.5 * R_S
DENSE = 32          # a group of more particles is dense
CHUNK = 64          # i-particles of a work item
SPARE = 65536       # partials a plan holds besides those per particle


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def partials_needed(pos, grid, box, n_max, radius_cells):
    """(partials of a one-sided call, dense groups, groups): each item (a
    chunk of a dense group) leaves one for every particle of its group after
    the chunk and one for every particle of the stencil's segments that lie
    in dense groups at positive offsets."""
    from paper_1510_07621_amd import binding
    G = binding.group_edge(n_max, grid)
    c = np.minimum((pos / (box / grid)).astype(np.int64), grid - 1)
    count = np.bincount((c[0] * grid + c[1]) * grid + c[2], minlength=grid ** 3).reshape((grid,) * 3)
    nd = grid // G
    groups = count.reshape(nd, G, nd, G, nd, G).sum(axis=(1, 3, 5))
    dense = groups > DENSE
    first = np.arange(0, grid, G)
    entries = np.zeros_like(groups)
    for dx, dy, lo, hi, sign in binding.segment_rows(G, radius_cells):
        if sign <= 0:
            continue
        col = count[(first + dx) % grid][:, (first + dy) % grid]
        part = sum(col[:, :, (first + z) % grid] for z in range(lo, hi + 1))
        entries += part * np.roll(dense, (-(dx // G), -(dy // G), -(lo // G)), axis=(0, 1, 2))
    k = -(-groups // CHUNK)
    need = np.where(dense, k * entries + (k - 1) * groups - CHUNK // 2 * k * (k - 1), 0)
    return int(need.sum()), int(dense.sum()), groups.size


def one_sided_plan(n, precision, **kw):
    from paper_1510_07621_amd import binding
    return binding.Plan(binding.Params(grid_n=GRID, box=BOX, precision=precision, **kw), n,
                        one_sided_above=0)


def the_set(full, seed):
    """Dense cells in neighbouring groups, one group across the z face, over a
    sparse background with some dense groups; `full`: a crowded cell more,
    whose partials alone pass the spare ones."""
    rng = np.random.default_rng(seed)
    cells = [([5, 9, 15], 300), ([5, 9, 0], 650), ([6, 10, 13], 500), ([2, 3, 4], 33)]
    if full:
        cells.append(([11, 2, 7], 4000))
    dense = np.concatenate([(np.array(c)[:, None] + rng.random((3, k))) * H for c, k in cells], axis=1)
    pos = np.concatenate([dense, ics.uniform(1701, BOX, seed=seed + 1)], axis=1)
    pos = pos[:, rng.permutation(pos.shape[1])]
    n = pos.shape[1]
    return pos, rng.uniform(0.5, 1.5, n) / n, rng.normal(size=(3, n))


def check_capacity(pos, partials):
    """With 80 partials a particle the call's fit, with 1 they do not."""
    n = pos.shape[1]
    need, ndense, ngroup = partials_needed(pos, GRID, BOX, n, R_C / H)
    assert 0 < ndense < ngroup                      # dense and sparse groups
    assert (need <= partials * n + SPARE) == (partials == 80), (need, n)


def ran_one_sided(P, calls):
    count, ms = P.stage_times()
    return count == calls and ms["react"] > 0


@functools.lru_cache(maxsize=None)
def force_refs(full, soft):
    """(targets, short-range force, with one mass, mesh force) of the set."""
    pos, m, _ = the_set(full, 23)
    n, eps = pos.shape[1], soft * H
    tg = sample_targets(pos, 1200)
    ref = o_pp.pp_accel(pos, m, BOX, R_S, R_C, eps, targets=tg) * m[tg]
    ref_s = o_pp.pp_accel(pos, 1.0 / n, BOX, R_S, R_C, eps, targets=tg) / n
    return tg, ref, ref_s, o_pm.pm_accel(pos, m, BOX, GRID, R_S, targets=tg) * m[tg]


@functools.lru_cache(maxsize=None)
def adjoint_refs(full, soft):
    pos, m, lam = the_set(full, 83)
    n, eps = pos.shape[1], soft * H
    tg = sample_targets(pos, 1200)
    ref = adjoint.pp_vjp(pos, m, BOX, R_S, R_C, eps, lam, targets=tg)
    ref_s = adjoint.pp_vjp(pos, 1.0 / n, BOX, R_S, R_C, eps, lam, targets=tg)
    return tg, ref, ref_s, adjoint.pm_vjp(pos, m, BOX, GRID, R_S, lam)[:, tg]


@pytest.mark.parametrize("soft", [0.0, 0.02, 0.6])
@pytest.mark.parametrize("partials", [80, 1])
def test_force(partials, soft):
    pos, m, _ = the_set(partials == 1, 23)
    n = pos.shape[1]
    check_capacity(pos, partials)
    tg, ref, ref_s, ref_pm = force_refs(partials == 1, soft)
    x, md = dev(pos), dev(m)
    with one_sided_plan(n, "fp32", softening=soft * H, pair_partials=partials) as P:
        P.set_timing(6)
        F = host(P.pp_force(x, md))[:, tg]
        Fs = host(P.pp_force(x, 1.0 / n))[:, tg]
        F32 = host(P.pp_force(x, md, fp32_out=True))[:, tg]
        full = [host(P.force(x, md))[:, tg]]
        for out32 in (False, True):
            Fc, order = P.force_cell_order(x, md, fp32_out=out32)
            back = np.empty((3, n))
            back[:, order.cpu().numpy().astype(np.int64)] = host(Fc)
            full.append(back[:, tg])
        assert ran_one_sided(P, 6)
    for got, want in ((F, ref), (Fs, ref_s), (F32, ref)):
        e = metrics.force_errors(got, want)
        assert e["rms"] <= 1e-5 and e["max"] <= 1e-3, e
    for got in full:
        assert metrics.force_errors(got, ref + ref_pm)["rms"] <= 1e-4


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-9), ("fp32", 1e-4)])
@pytest.mark.parametrize("soft", [0.02, 0.6])
@pytest.mark.parametrize("partials", [80, 1])
def test_adjoint(precision, tol, partials, soft):
    pos, m, lam = the_set(partials == 1, 83)
    n = pos.shape[1]
    check_capacity(pos, partials)
    tg, ref, ref_s, ref_pm = adjoint_refs(partials == 1, soft)
    x, md, l = dev(pos), dev(m), dev(lam)
    with one_sided_plan(n, precision, softening=soft * H, adjoint=True,
                        pair_partials=partials) as P:
        P.set_timing(3)
        got = host(P.pp_force_vjp(x, md, l))[:, tg]
        got_s = host(P.pp_force_vjp(x, 1.0 / n, l))[:, tg]
        full = host(P.force_vjp(x, md, l))[:, tg]
        assert ran_one_sided(P, 3)
    assert metrics.force_errors(got, ref)["rms"] <= tol
    assert metrics.force_errors(got_s, ref_s)["rms"] <= tol
    assert metrics.force_errors(full, ref + ref_pm)["rms"] <= tol


@pytest.mark.parametrize("n,edge,partials", [(32001, 2, 260), (100001, 1, 300)])
def test_smaller_groups(n, edge, partials):
    """Groups of 2^3 and of single cells, in crowded sets, beside a group of
    several chunks: force and adjoint."""
    from paper_1510_07621_amd import binding
    rng = np.random.default_rng(n)
    crowd = (np.array([15, 0, 7])[:, None] + rng.random((3, 333))) * H
    pos = np.concatenate([crowd, ics.uniform(n - 333, BOX, seed=n)], axis=1)
    m = rng.uniform(0.5, 1.5, n) / n
    lam = rng.normal(size=(3, n))
    assert binding.group_edge(n, GRID) == edge
    need, ndense, ngroup = partials_needed(pos, GRID, BOX, n, R_C / H)
    assert 0 < ndense and need <= partials * n + SPARE, (need, n)
    eps = 0.02 * H
    tg = np.concatenate([np.arange(60), sample_targets(pos, 300)])
    ref = o_pp.pp_accel(pos, m, BOX, R_S, R_C, eps, targets=tg) * m[tg]
    ref_v = adjoint.pp_vjp(pos, m, BOX, R_S, R_C, eps, lam, targets=tg)
    for precision, tol, vjp_tol in (("fp32", 1e-5, 1e-4), ("fp64", 1e-12, 1e-9)):
        with one_sided_plan(n, precision, softening=eps, adjoint=True,
                            pair_partials=partials) as P:
            P.set_timing(2)
            F = host(P.pp_force(dev(pos), dev(m)))[:, tg]
            g = host(P.pp_force_vjp(dev(pos), dev(m), dev(lam)))[:, tg]
            assert ran_one_sided(P, 2)
        assert metrics.force_errors(F, ref)["rms"] <= tol
        assert metrics.force_errors(g, ref_v)["rms"] <= vjp_tol


@pytest.mark.parametrize("precision,adj,n,holds", [
    ("fp32", False, 3 << 20, False), ("fp32", False, (3 << 20) + 1, True),
    ("fp64", False, (3 << 20) + 1, False), ("fp32", True, 5 << 19, False),
    ("fp64", True, 5 << 19, False), ("fp64", True, (5 << 19) + 1, True)])
def test_partials_are_held_only_where_a_call_takes_them(precision, adj, n, holds):
    """A plan none of whose calls is one-sided takes no memory for partials."""
    from paper_1510_07621_amd import binding

    def taken(partials):
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        with binding.Plan(binding.Params(grid_n=128, precision=precision, adjoint=adj,
                                         pair_partials=partials), n):
            return before - torch.cuda.mem_get_info()[0]

    taken(0)                                # (what the runtime keeps of its own)
    extra = taken(80) - taken(0)
    size = 80 * n * 3 * (4 if precision == "fp32" else 8)
    assert extra >= size if holds else extra < size // 50


@pytest.mark.parametrize("kind,tol", [("force", 1e-5), ("vjp", 1e-4)])
@pytest.mark.parametrize("grid,n,partials,one_sided", [
    (64, 3 << 19, 140, False), (64, (3 << 19) + 1, 140, True), (64, (3 << 19) + 1, 60, False),
    (128, (3 << 19) + 1, 140, False), (32, (3 << 19) + 1, 300, True)])
def test_crowded_sets_are_one_sided_from_fewer_particles(grid, n, partials, one_sided, kind, tol):
    """Both sides of the crowded sets' line, by particles, by particles a cell
    and by partials: the route, and the result against the two-sided sum's."""
    from paper_1510_07621_amd import binding
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + grid)
    x = torch.rand((3, n), generator=gen, dtype=torch.float64, device="cuda")
    lam = torch.randn((3, n), generator=gen, dtype=torch.float64, device="cuda")
    prm = dict(grid_n=grid, precision="fp32", softening=0.02 / grid, adjoint=kind == "vjp",
               rs_cells=1.0, cutoff_rs=4.5 if grid > 32 else 3.0)
    out = []
    for pp in (0, partials):
        with binding.Plan(binding.Params(pair_partials=pp, **prm), n) as P:
            P.set_timing(1)
            out.append(P.pp_force(x, 1.0 / n) if kind == "force" else P.pp_force_vjp(x, 1.0 / n, lam))
            assert (P.stage_times()[1]["react"] > 0) == (pp > 0 and one_sided)
    assert ((out[1] - out[0]).norm() <= tol * out[0].norm()).item()
