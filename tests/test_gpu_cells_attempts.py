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


def _launches(ctx, call):
    ctx.profile(True)
    out = call()
    n = {k: n for k, (_, n) in ctx.profile_read().items()}
    ctx.profile(False)
    return out, n


@pytest.mark.parametrize("cap", [0, 256 << 20])   # 256 MB: the plans and two points at a time
def test_points_handed_on_are_solved_together(ctx, cap):
    """Points of three cells that need the reduction: one longer attempt and one
    reduction for all of them (for the chunks of them that a cap allows), from the
    coefficients at hand; the launches of the captured graph are not counted."""
    from paper_1310_6380_amd import mvpb
    own = mvpb.Context(0, workspace_cap=cap)
    try:
        scales = (1.0, 2.0, 0.5)
        cells = [_even(own, s) for s in scales]
        (rc, out), n = _launches(own, lambda: _solve_cells(own, cells, [M] * 3, [QS] * 3, NB))
        print("cap", cap, "status", rc, {k: v for k, v in n.items() if v}, flush=True)
        assert rc == mvpb.OK
        for s, om in zip(scales, out):
            assert band_error(om, _folded(QS, s)) <= TOL64
        assert n["potrf_trtri"] == 0 and n["zgemm"] == 0 and n["hb2st"] > 0
        if not cap:
            assert n["krylov_factor"] == 1 and n["form_operator"] == 2
        buf = mvpb.DeviceBuffer(out[0].nbytes * 3)
        args = [(ctypes.c_void_p * 3)(*[c.h for c in cells]), (ctypes.c_int * 3)(*[M] * 3), (ctypes.c_int * 3)(*[3] * 3),
                (ctypes.POINTER(ctypes.c_double) * 3)(*[QS.ctypes.data_as(ctypes.POINTER(ctypes.c_double))] * 3),
                (ctypes.c_void_p * 3)(*[buf.value + i * out[0].nbytes for i in range(3)])]
        assert mvpb.load().mvpb_solve_cells(own.h, 3, args[0], args[1], args[1], 0, args[2], args[3], NB, args[4],
                                            mvpb.F_DEVICE_PTRS) == mvpb.OK
        assert np.array_equal(buf.to_numpy(np.float64, (3,) + out[0].shape), np.stack(out))
    finally:
        own.close()


def test_no_reduction_at_large_contrast(ctx):
    """Cells of stiffness ratios 1e-5 .. 1e5 in one call: no point is handed on to the
    reduction (8 bands take the steps that just reach the bar: one longer attempt)."""
    x, y = np.meshgrid((np.arange(24) + 0.5) / 24 - 0.5, (np.arange(24) + 0.5) / 24 - 0.5, indexing="ij")
    phase = (x * x + y * y < 0.09).astype(np.int32)
    ratios = [1e-5, 1e-4, 1e-3, 1e3, 1e4, 1e5]
    props = [np.array([[1e9, 0.35, 1200.0], [1e9 * r, 0.33, 2400.0]]) for r in ratios]
    Ms = [8, 6, 7, 8, 6, 7]
    Q = np.array([[0.0, 0.0], [0.02, 0.01], [0.31, 0.12], [0.5, 0.5]])
    cells = [ctx.cell(phase, p) for p in props]
    (rc, out), n = _launches(ctx, lambda: _solve_cells(ctx, cells, Ms, [Q] * 6, 8))
    print({k: v for k, v in n.items() if v}, flush=True)
    assert rc == 0 and n["krylov_factor"] <= 1 and n["he2hb_panel"] == 0, n
    for c, m, om in zip(cells, Ms, out):
        plan = c.plan(m)
        assert band_error(om, plan.solve(Q, 8)) <= 1e-10
        plan.close()
