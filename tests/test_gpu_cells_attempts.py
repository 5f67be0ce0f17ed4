"""Points of mvpb_solve_cells that the Krylov route has to hand on (a block of 16
vectors cannot hold as many copies of one value): a homogeneous cell without lateral
contraction, whose shear waves (3, 1) and pressure waves (2, 1) have one frequency,
sixteen-fold at Gamma, against the folded free dispersion."""
import ctypes

import numpy as np
import pytest

from oracle.compare import band_error
from synth import random_iso_props

pytestmark = pytest.mark.gpu

TOL64 = 1e-9
E0, RHO0 = 70e9, 2700.0
M, NB = 8, 60          # 2N = 578; the sixteen lie at bands 43 .. 58
QS = np.array([[0.0, 0.0], [0.13, 0.21], [0.0, 0.0]])


@pytest.fixture(scope="module")
def ctx():
    from paper_1310_6380_amd import mvpb
    c = mvpb.Context(0)
    yield c
    c.close()


def _even(ctx, scale=1.0):
    return ctx.cell(np.zeros((8, 8), np.int32), np.array([[E0 * scale, 0.0, RHO0]]))


def _folded(Q, scale=1.0):
    g = np.arange(-M, M + 1)
    n = np.stack(np.meshgrid(g, g, indexing="ij"), axis=-1).reshape(-1, 2)
    K = 2.0 * np.pi * np.linalg.norm(Q[:, None] + n[None], axis=2)
    c2 = E0 * scale / (2.0 * RHO0)
    return np.sort(np.concatenate([np.sqrt(c2) * K, np.sqrt(2.0 * c2) * K], axis=1), axis=1)[:, :NB]


def _solve_cells(ctx, cells, Ms, Qs, nb):
    """(status, outputs) of the call itself."""
    from paper_1310_6380_amd import mvpb
    n = len(cells)
    Qs = [np.ascontiguousarray(q) for q in Qs]
    out = [np.full((len(q), nb), np.nan) for q in Qs]
    ms = (ctypes.c_int * n)(*Ms)
    rc = mvpb.load().mvpb_solve_cells(
        ctx.h, n, (ctypes.c_void_p * n)(*[c.h for c in cells]), ms, ms, 0, (ctypes.c_int * n)(*map(len, Qs)),
        (ctypes.POINTER(ctypes.c_double) * n)(*[q.ctypes.data_as(ctypes.POINTER(ctypes.c_double)) for q in Qs]), nb,
        (ctypes.c_void_p * n)(*[o.ctypes.data for o in out]), 0)
    return rc, out


def test_points_stand_beside_a_cell_that_does_not_factor(ctx):
    """The other cells' results are meaningful when one cell's matrices are not
    positive definite, those of points that need another attempt too."""
    from paper_1310_6380_amd import mvpb
    phase = np.zeros((16, 16), np.int32)
    phase[1:] = 1
    void = ctx.cell(phase, np.array([[E0, 0.3, RHO0], [E0, 0.3, 1e-30]]))   # a strip of mass: singular to rounding
    rc, out = _solve_cells(ctx, [_even(ctx), void], [M, M], [QS, QS[1:2]], NB)
    print("status", rc, flush=True)
    assert rc == mvpb.E_NOT_PD
    assert band_error(out[0], _folded(QS)) <= TOL64


def test_every_cap_above_an_accepted_one_is_accepted():
    """60 points of 2N = 242, 4 bands, under caps from the least that a single item of
    the reduction fits to well above one of the Krylov route."""
    from paper_1310_6380_amd import mvpb
    rng = np.random.default_rng(5)
    phase, props = rng.integers(0, 3, (16, 16)).astype(np.int32), random_iso_props(3, rng)
    Q = rng.uniform(0.05, 0.5, (60, 2))

    def accepted(cap):
        c = mvpb.Context(0, workspace_cap=cap)
        try:
            rc, out = _solve_cells(c, [c.cell(phase, props)], [5], [Q], 4)
            assert rc in (mvpb.OK, mvpb.E_NOMEM)
            assert rc != mvpb.OK or np.all(np.isfinite(out[0]))
            return rc == mvpb.OK
        finally:
            c.close()

    lo, hi = 1 << 20, 64 << 20
    assert accepted(hi) and not accepted(lo)
    while hi - lo > 4096:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if accepted(mid) else (mid, hi)
    refused = [cap for cap in range(hi, hi + (5 << 19), 40 << 10) if not accepted(cap)]
    print("least cap", hi, "refused above it", refused, flush=True)
    assert not refused


def test_calls_of_one_shape_and_other_routes(ctx):
    """Cells of one shape whose materials ask for more steps, in other places of the
    call: its launch sequence is that of the chunks, not of the shape alone."""
    x, y = np.meshgrid((np.arange(16) + 0.5) / 16 - 0.5, (np.arange(16) + 0.5) / 16 - 0.5, indexing="ij")
    phase = (x * x + y * y < 0.09).astype(np.int32)
    plain = np.array([[1e9, 0.35, 1200.0], [5e9, 0.33, 1500.0]])
    heavy = np.array([[1e9, 0.35, 1200.0], [1e11, 0.33, 120000.0]])
    Q = np.random.default_rng(3).uniform(0.05, 0.5, (7, 2))
    ref = {}
    for name, props in (("plain", plain), ("heavy", heavy)):
        plan = ctx.cell(phase, props).plan(6)
        ref[name] = plan.solve(Q, 5)
        plan.close()
    for names in (("plain", "plain", "heavy"), ("plain", "heavy", "heavy"), ("heavy", "plain", "plain"),
                  ("plain", "plain", "plain"), ("plain", "heavy", "heavy")):
        cells = [ctx.cell(phase, plain if n == "plain" else heavy) for n in names]
        for name, om in zip(names, ctx.solve_cells(cells, [6] * 3, [Q] * 3, 5)):
            print(names, name, band_error(om, ref[name]), flush=True)
            assert band_error(om, ref[name]) <= 1e-10
