"""Host-side checks of the C ABI (no GPU needed, nothing computed on a device).

The library must load, export every function its headers declare, reject
bad arguments before touching the GPU, and build the neighbour stencil the
pair sum relies on.
"""
import ctypes
import itertools
import math
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1510_07621_amd", "libp3m.so")

pytestmark = pytest.mark.skipif(not os.path.exists(LIB),
                                reason="libp3m.so not built (run __graft_entry__.build())")


def _declared_functions():
    names = set()
    for h in ("p3m.h", "p3m_host.h"):
        text = open(os.path.join(ROOT, "include", h)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        for m in re.finditer(r"^\s*(?:const\s+)?[A-Za-z_][\w ]*?[\s\*]+(\w+)\s*\(", text, re.M):
            names.add(m.group(1))
    return names


@pytest.fixture(scope="module")
def b():
    from paper_1510_07621_amd import binding
    return binding


def test_every_declared_function_is_exported(b):
    names = _declared_functions()
    assert {"p3m_force", "pm_force", "pp_force", "p3m_kick", "p3m_drift",
            "p3m_plan_create", "p3m_plan_destroy", "p3m_strerror",
            "p3m_stencil_rows"} <= names
    lib = ctypes.CDLL(LIB)
    for n in sorted(names):
        assert hasattr(lib, n), f"{n} declared but not exported"


def _create(b, n_max=16, **kw):
    p = b.Params(**{"grid_n": 32, **kw}).to_c()
    h = ctypes.c_void_p()
    st = b._lib.p3m_plan_create(ctypes.byref(p), n_max, None, ctypes.byref(h))
    return st, h


@pytest.mark.parametrize("kw,expect", [
    (dict(grid_n=100), -1), (dict(grid_n=8), -1), (dict(grid_n=1024), -1),
    (dict(precision="fp32", fd_order=3), -1), (dict(deconv_power=1), -1),
    (dict(box=0.0), -1), (dict(box=float("nan")), -1), (dict(rs_cells=-1.0), -1),
    (dict(cutoff_rs=0.0), -1), (dict(softening=-1e-3), -1), (dict(G=float("inf")), -1),
    (dict(grid_n=16, rs_cells=2.0, cutoff_rs=4.0), -4),       # r_c = box/2
    (dict(grid_n=16, rs_cells=1.25, cutoff_rs=8.0), -4),
])
def test_plan_create_rejects_bad_parameters(b, kw, expect):
    prec = kw.pop("precision", "fp32")
    st, h = _create(b, precision=prec, **kw)
    assert st == expect and not h.value


def test_plan_create_rejects_bad_sizes_and_nulls(b):
    assert _create(b, n_max=-1)[0] == -1
    assert _create(b, n_max=2 ** 31)[0] == -1
    h = ctypes.c_void_p()
    assert b._lib.p3m_plan_create(None, 4, None, ctypes.byref(h)) == -1
    p = b.Params(grid_n=32).to_c()
    assert b._lib.p3m_plan_create(ctypes.byref(p), 4, None, None) == -1
    bad = b.Params(grid_n=32, precision="fp32").to_c()
    bad.precision = 7
    assert b._lib.p3m_plan_create(ctypes.byref(bad), 4, None, ctypes.byref(h)) == -1
    for E in (6, 7, 514, -2):
        bad = b.Params(grid_n=32, ewald_gridsize=E).to_c()
        assert b._lib.p3m_plan_create(ctypes.byref(bad), 4, None, ctypes.byref(h)) == -1
    bad = b.Params(grid_n=32, adjoint=True).to_c()
    assert bad.adjoint == 1
    bad.adjoint = 2
    assert b._lib.p3m_plan_create(ctypes.byref(bad), 4, None, ctypes.byref(h)) == -1


def test_plan_create_one_sided_rejects_what_plan_create_does(b):
    p, h = b.Params(grid_n=32, pair_partials=80).to_c(), ctypes.c_void_p()
    make = b._lib.p3m_plan_create_one_sided
    assert make(ctypes.byref(p), 4, -2, None, ctypes.byref(h)) == -1
    assert make(None, 4, 0, None, ctypes.byref(h)) == -1
    assert make(ctypes.byref(p), 4, 0, None, None) == -1
    assert make(ctypes.byref(p), -1, 0, None, ctypes.byref(h)) == -1
    p.grid_n = 100
    assert make(ctypes.byref(p), 4, 0, None, ctypes.byref(h)) == -1
    assert not h.value


def test_calls_on_null_plan_and_bad_arguments(b):
    L = b._lib
    for fn in (L.p3m_force, L.pm_force, L.pp_force):
        assert fn(None, 10, 1, None, 1.0, 2, 0) == -1
    assert L.p3m_pair_count(None, 1, 1, 1) == -1
    assert L.p3m_plan_destroy(None) == 0
    assert L.p3m_plan_set_stream(None, None) == -1
    assert L.p3m_set_timing(None, 1) == -1
    assert L.p3m_kick(-1, 1, 1, 0, 1.0, None) == -1
    assert L.p3m_kick(0, None, None, 0, 1.0, None) == 0       # empty: no-op
    assert L.p3m_kick(5, None, 1, 0, 1.0, None) == -1
    assert L.p3m_kick(5, 1, 1, 0, float("nan"), None) == -1
    assert L.p3m_drift(-1, 1, 1, None, 1.0, 1.0, 1.0, None) == -1
    assert L.p3m_drift(0, None, None, None, 1.0, 1.0, 1.0, None) == 0
    assert L.p3m_drift(5, 1, 1, None, 1.0, 1.0, 0.0, None) == -1     # box <= 0
    assert L.p3m_drift(5, 1, 1, None, 0.0, 1.0, 1.0, None) == -1     # zero scalar mass
    assert L.p3m_power_spectrum(None, 10, 1, None, 1.0, 8, 0.0, 2, 3, 4, None) == -1
    assert L.pp_ewald_force(None, 10, 1, None, 1.0, 2, 0) == -1
    assert L.p3m_ewald_correction(None, 10, 1, 2) == -1
    for fn in (L.p3m_force_vjp, L.pm_force_vjp, L.pp_force_vjp):
        assert fn(None, 10, 1, None, 1.0, 2, 3) == -1
    assert L.p3m_force_cell_order(None, 10, 1, None, 1.0, 2, 0, 3) == -1
    # kick and reorder: order, pos, mom, force, ids, mass, c, outputs ...
    KR = L.p3m_kick_reorder
    big = 1 << 20                                    # (addresses only, never touched)
    assert KR(-1, 1, 2, 3, 4, 0, None, None, 1.0, 5, 6, None, None, None) == -1
    assert KR(0, None, None, None, None, 0, None, None, 1.0, None, None, None, None,
              None) == 0                                              # empty: no-op
    assert KR(5, None, 2, 3, 4, 0, None, None, 1.0, 5, 6, None, None, None) == -1  # no order
    assert KR(5, 1, 2, 3, 4, 0, None, None, float("nan"), 5, 6, None, None, None) == -1
    assert KR(5, 1, 2, 3, 4, 0, 7, None, 1.0, 5, 6, None, None, None) == -1  # ids w/o ids_out
    assert KR(5, 1, 2, 3, 4, 0, None, 8, 1.0, 5, 6, None, None, None) == -1  # mass w/o out
    assert KR(5, big, 2 * big, 3 * big, 4 * big, 0, None, None, 1.0, 2 * big, 6 * big, None,
              None, None) == -1                                      # pos_out over pos
    assert KR(5, big, 2 * big, 3 * big, 4 * big, 0, None, None, 1.0, 5 * big, 5 * big + 8,
              None, None, None) == -1                                # outputs overlap
    assert L.p3m_drift_vjp(-1, 1, 2, None, 1.0, 1.0, None) == -1
    assert L.p3m_drift_vjp(0, None, None, None, 1.0, 1.0, None) == 0    # empty: no-op
    assert L.p3m_drift_vjp(5, None, 2, None, 1.0, 1.0, None) == -1
    assert L.p3m_drift_vjp(5, 1, 4096, None, 0.0, 1.0, None) == -1     # zero scalar mass
    assert L.p3m_drift_vjp(5, 4096, 4096, None, 1.0, 1.0, None) == -1  # in place on itself
    assert L.p3m_drift_vjp(5, 4096, 8192, None, 1.0, float("inf"), None) == -1
    st = b._lib.p3m_stencil_rows(0, 5.0, None, 0)
    assert st == -1


def test_noalloc_argument_errors_before_any_device_call(b):
    """pp_force_noalloc rejects bad arguments and sizes beyond its fixed
    workspace before it touches the device (these paths run without a GPU)."""
    L = b._lib
    p = b.Params(grid_n=32, softening=1e-3).to_c()
    assert L.pp_force_noalloc(None, 10, 1, None, 1.0, 2, 0, None) == -1
    assert L.pp_force_noalloc(ctypes.byref(p), -1, 1, None, 1.0, 2, 0, None) == -1
    assert L.pp_force_noalloc(ctypes.byref(p), 65537, 1, None, 1.0, 2, 0, None) == -5
    assert L.pp_force_noalloc(ctypes.byref(p), 0, None, None, 1.0, None, 0, None) == 0
    assert L.pp_force_noalloc(ctypes.byref(p), 10, None, None, 1.0, 2, 0, None) == -1
    assert L.pp_force_noalloc(ctypes.byref(p), 10, 1, None, float("nan"), 2, 0, None) == -1
    # force overlapping pos
    assert L.pp_force_noalloc(ctypes.byref(p), 10, 4096, None, 1.0, 4096 + 80, 0, None) == -1
    big = b.Params(grid_n=128).to_c()
    assert L.pp_force_noalloc(ctypes.byref(big), 10, 1, None, 1.0, 4096, 0, None) == -5
    bad = b.Params(grid_n=24).to_c()
    assert L.pp_force_noalloc(ctypes.byref(bad), 10, 1, None, 1.0, 4096, 0, None) == -1
    far = b.Params(grid_n=16, rs_cells=2.0, cutoff_rs=4.0).to_c()     # r_c = box / 2
    assert L.pp_force_noalloc(ctypes.byref(far), 10, 1, None, 1.0, 4096, 0, None) == -4
    assert "fixed workspace" in b.strerror(-5)


def test_strerror(b):
    assert b.strerror(0) == "success"
    assert "invalid" in b.strerror(-1)
    assert "memory" in b.strerror(-2)
    assert "HIP" in b.strerror(-3)
    assert "half the box" in b.strerror(-4)
    assert b.strerror(12345) == "unknown status"


def _gap(d, g):
    return -d - 1 if d < 0 else (d - g if d >= g else 0)


@pytest.mark.parametrize("g,R", [(1, 5.625), (2, 5.625), (4, 5.625), (2, 2.5), (2, 7.99),
                                 (1, 0.3), (4, 1.0)])
def test_stencil_rows_cover_exactly_the_cells_within_reach(b, g, R):
    """A cell is in the stencil iff its box comes closer than R cells to the
    g^3 group box; rows are z-runs with no overlaps."""
    rows = b.stencil_rows(g, R)
    got = set()
    for dx, dy, lo, hi in rows:
        assert lo <= hi
        for dz in range(lo, hi + 1):
            assert (dx, dy, dz) not in got
            got.add((dx, dy, dz))
    reach = math.ceil(R) + 2
    want = set()
    for dx, dy, dz in itertools.product(range(-reach, g + reach), repeat=3):
        # the library keeps a 1e-9 cell margin so FP rounding cannot drop a pair
        if _gap(dx, g) ** 2 + _gap(dy, g) ** 2 + _gap(dz, g) ** 2 < (R + 1e-9) ** 2:
            want.add((dx, dy, dz))
    assert got == want


def test_stencil_contains_every_partner_cell_of_random_pairs(b):
    """Monte Carlo: for i in the group and j within r_c, j's cell is visited."""
    import numpy as np
    rng = np.random.default_rng(0)
    g, R = 2, 5.625
    cells = {(dx, dy, dz) for dx, dy, lo, hi in b.stencil_rows(g, R) for dz in range(lo, hi + 1)}
    xi = rng.random((20000, 3)) * g
    d = rng.normal(size=(20000, 3))
    d *= (rng.random(20000) ** (1 / 3) * R / np.linalg.norm(d, axis=1))[:, None]
    xj = xi + d
    for c in np.floor(xj).astype(int):
        assert tuple(c) in cells


@pytest.mark.parametrize("g,R", [(1, 5.625), (2, 5.625), (4, 5.625), (4, 10.0), (2, 1.0)])
def test_segments_cut_the_stencil_at_groups_and_sign_each_pair_once(b, g, R):
    """The segments partition the full stencil's cells, each lies in one
    group and carries the lexicographic sign of that group's offset; of two
    different groups that hold a pair of cells closer than R cells, exactly
    one sees the other at a positive offset (so a pair between two groups is
    evaluated once); the group itself has sign 0. Checked for all cell
    pairs with the first cell in the group at the origin."""
    full = b.stencil_rows(g, R)
    segs = b.segment_rows(g, R)
    fcells = {(dx, dy, dz) for dx, dy, lo, hi in full for dz in range(lo, hi + 1)}
    sign = {}
    for dx, dy, lo, hi, sg in segs:
        assert lo <= hi and lo // g == hi // g                 # inside one group
        o = (dx // g, dy // g, lo // g)
        want = 0 if o == (0, 0, 0) else (1 if o > (0, 0, 0) else -1)
        assert sg == want
        for dz in range(lo, hi + 1):
            assert (dx, dy, dz) not in sign
            sign[(dx, dy, dz)] = sg
    assert set(sign) == fcells
    # order: the full stencil's row order, pieces by increasing z
    key = {(dx, dy): k for k, (dx, dy, lo, hi) in enumerate(full)}
    order = [(key[(dx, dy)], lo) for dx, dy, lo, hi, sg in segs]
    assert order == sorted(order)
    for ci in itertools.product(range(g), repeat=3):   # i's cell inside the group at 0
        for cj in fcells:
            d = tuple(cj[a] - ci[a] for a in range(3))
            if sum(_gap(x, 1) ** 2 for x in d) >= (R + 1e-9) ** 2:
                continue                               # no pair of points closer than R
            o = tuple(cj[a] // g for a in range(3))     # j's group offset
            if o == (0, 0, 0):
                assert sign[cj] == 0
                continue
            back = tuple(ci[a] - g * o[a] for a in range(3))   # i's cell seen from j's group
            assert back in sign
            assert (sign[cj] > 0) != (sign[back] > 0), (ci, cj)
            assert sign[cj] == -sign[back]


def test_group_edge(b):
    assert b.group_edge(128 ** 3, 128) == 4        # one particle per cell -> 64 per group
    assert b.group_edge(16 ** 3, 128) == 4         # sparse: largest group
    assert b.group_edge(8 * 64 ** 3, 64) == 2      # eight per cell -> 64 per group
    assert b.group_edge(64 * 32 ** 3, 32) == 1     # dense
    assert b.group_edge(0, 64) == 1
    assert b.group_edge(10 ** 9, 16) == 1


def _split_f(u):
    from scipy.special import erfc
    import numpy as np
    return erfc(u) + 2.0 / np.sqrt(np.pi) * u * np.exp(-u * u)


@pytest.mark.parametrize("cutoff_rs,soft_rs", [(4.5, 0.0), (4.5, 0.024), (3.0, 0.024),
                                               (6.0, 0.01), (4.5, 0.08)])
def test_adjoint_weight_from_piece_derivatives(b, cutoff_rs, soft_rs):
    """The force adjoint's second pair weight w2 = g'(r)/r, g = f / rho^3,
    takes f'(r)/r = (df/drho)/rho from the derivative of the split-factor
    piece when the table variable is the softened distance. Against the
    closed form f'(r) = -r^2 e^{-u^2} / (2 sqrt(pi) r_s^3): FP32 pieces within
    1e-5 of w2 for cutoffs up to 4.5 r_s (2e-4 at 6), FP64 pieces within
    1e-11 (1e-10 at 6); the FP64 leading exact pieces are excluded (the
    kernel evaluates those from the closed form)."""
    import numpy as np
    r = np.linspace(1e-4, cutoff_rs, 200001)[:-1]           # units of r_s
    u = 0.5 * r
    exact_d = -r * np.exp(-u * u) / (2.0 * np.sqrt(np.pi))
    for prec in ("fp32", "fp64"):
        if prec == "fp32":
            tab, (v, v0, v1) = b.split_table(cutoff_rs, soft_rs)
            exact_bins = 0
        else:
            tab, (v, v0, v1, exact_bins) = b.split_table64(cutoff_rs, soft_rs)
        if v != 1:
            continue
        B = tab.shape[1] - 1
        s = B / (v1 - v0)
        rho = np.sqrt(r * r + soft_rs * soft_rs)
        x = (rho - v0) * s
        k = np.minimum(x.astype(np.int64), B)
        t = x - k
        f = tab[-1][k].astype(np.float64)
        ft = np.zeros_like(t)
        for l in range(tab.shape[0] - 2, -1, -1):
            ft = ft * t + f
            f = f * t + tab[l][k]
        w2 = s * ft / rho / rho ** 3 - 3.0 * f / rho ** 5
        w2x = exact_d / rho ** 3 - 3.0 * _split_f(u) / rho ** 5
        keep = k >= exact_bins
        rel = np.abs(w2 / w2x - 1.0)[keep]
        if prec == "fp32":
            assert rel.max() < (1e-5 if cutoff_rs <= 4.5 else 2e-4)
        else:
            assert rel.max() < (1e-11 if cutoff_rs <= 4.5 else 1e-10)


@pytest.mark.parametrize("cutoff_rs,soft_rs,var", [
    (4.5, 0.0, 1),          # no softening: the softened distance is r itself
    (4.5, 0.024, 1),        # 0.03 mean spacing at r_s = 1.25 cells
    (3.0, 0.024, 1),
    (6.0, 0.01, 1),
    (4.5, 0.08, 0),         # eps wide against a bin: the kink forces r
    (4.5, 0.8, 0),
])
def test_split_table_matches_erfc_split(b, cutoff_rs, soft_rs, var):
    """The FP32 pair sum's table of f(u) = erfc(u) + (2u/sqrt(pi)) exp(-u^2),
    u = r / (2 r_s), looked up the way the kernel does (FP32 bin coordinate,
    bin = floor, entry B past the cutoff), agrees with SciPy's erfc to FP32
    rounding over all of 0 <= r < r_c."""
    import numpy as np
    tab, (v, v0, v1) = b.split_table(cutoff_rs, soft_rs)
    B = tab.shape[1] - 1
    assert tab.shape == (4, B + 1) and tab.dtype == np.float32
    assert v == var
    r = np.linspace(0.0, cutoff_rs, 400001)[:-1]            # units of r_s
    rho = np.sqrt(r * r + soft_rs * soft_rs) if v == 1 else r
    if v == 1:
        assert soft_rs * (1 - 2e-6) <= v0 <= soft_rs
        assert v1 == pytest.approx(np.hypot(cutoff_rs, soft_rs), rel=1e-15)
    else:
        assert (v0, v1) == (0.0, cutoff_rs)
    x = ((rho - v0) * (B / (v1 - v0))).astype(np.float32)
    assert x.min() >= 0 and x.max() < B + 1
    k = x.astype(np.int64)
    t = x - k.astype(np.float32)
    c = [tab[l][k] for l in range(4)]
    f32 = c[0] + t * (c[1] + t * (c[2] + t * c[3]))
    assert np.max(np.abs(f32 - _split_f(0.5 * r))) < 2.5e-7
    assert tab[0][B] == np.float32(_split_f(0.5 * cutoff_rs))
    assert np.all(tab[1:, B] == 0)
    # neighbouring pieces meet: the end of bin k is the start of bin k + 1
    ends = tab[0][:B] + tab[1][:B] + tab[2][:B] + tab[3][:B]
    assert np.max(np.abs(ends - tab[0][1:])) < 2e-7


@pytest.mark.parametrize("cutoff_rs,soft_rs,var", [
    (4.5, 0.0, 1), (4.5, 0.024, 1), (3.0, 0.024, 1), (6.0, 0.01, 1),
    (4.5, 0.24, 1), (4.5, 0.8, 0)])
def test_split_table64_matches_erfc_split(b, cutoff_rs, soft_rs, var):
    """The FP64 table, looked up as the kernel does (bins below `exact` by the
    exact formula), agrees with SciPy's erfc-based f over all of [0, r_c):
    3e-15 for cutoffs up to 4.5 r_s, 3e-14 at 6 (degree-6 pieces); the exact
    bins are few and lie next to r = 0."""
    import numpy as np
    tab, (v, v0, v1, exact) = b.split_table64(cutoff_rs, soft_rs)
    B = tab.shape[1] - 1
    assert tab.shape == (7, B + 1) and v == var and 0 <= exact <= 8
    r = np.linspace(0.0, cutoff_rs, 300001)[:-1]            # units of r_s
    vv = np.sqrt(r * r + soft_rs * soft_rs) if v == 1 else r
    x = (vv - v0) * (B / (v1 - v0))
    assert x.min() >= 0
    k = np.minimum(x.astype(np.int64), B)
    t = x - k
    f = tab[6][k]
    for l in range(5, -1, -1):
        f = f * t + tab[l][k]
    f = np.where(k < exact, _split_f(0.5 * r), f)
    assert np.max(np.abs(f - _split_f(0.5 * r))) < (3e-15 if cutoff_rs <= 4.5 else 3e-14)
    if soft_rs == 0.0:
        assert exact == 0                     # no kink: the table covers everything
    assert tab[0][B] == pytest.approx(_split_f(0.5 * cutoff_rs), rel=1e-15)
    assert np.all(tab[1:, B] == 0)
    assert b._lib.p3m_split_table64(0.0, 0.0, None, 0, None) == -1
    assert b._lib.p3m_split_table64(4.5, -1.0, None, 0, None) == -1
    assert b._lib.p3m_split_table64(4.5, 0.0, None, 3, None) == -1


def test_split_table_rejects_bad_arguments(b):
    f = b._lib.p3m_split_table
    assert f(0.0, 0.0, None, 0, None) == -1
    assert f(float("nan"), 0.0, None, 0, None) == -1
    assert f(4.5, -0.1, None, 0, None) == -1
    assert f(4.5, float("inf"), None, 0, None) == -1
    assert f(4.5, 0.0, None, 8, None) == -1
    assert f(4.5, 0.0, None, 0, None) > 0
