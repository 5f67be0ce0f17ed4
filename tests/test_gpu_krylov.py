"""The shift-invert block Krylov route of FP64 solves, at the sizes where its
tiles end: orders just around multiples of the factorisation's block (64), of
the products' rows (16) and of the orthogonalisation's chunk (128), one block
and many, few and many bands.  Frequencies against the oracle to the bar of
every FP64 path (1e-9), degenerate spectra against the folded free dispersion,
where more copies of one eigenvalue than the block holds (16) have to come from
the reduction, and modes by their residual in the Galerkin equations."""
import numpy as np
import pytest

from oracle import mixed_oracle as mo
from oracle.compare import band_error
from synth import random_iso_props

pytestmark = pytest.mark.gpu

TOL64 = 1e-9
OBLIQUE = np.array([[1.0, 0.0], [0.5, np.sqrt(3.0) / 2.0]])


@pytest.fixture(scope="module")
def ctx():
    from paper_1310_6380_amd import mvpb
    c = mvpb.Context(0)
    yield c
    c.close()


def _cell(seed, n=24, phases=4):
    rng = np.random.default_rng(seed)
    return rng.integers(0, phases, (n, n)).astype(np.int32), random_iso_props(phases, rng)


# (M1, M2, bands): 2N = 198 (3 blocks and 6), 162 and 198 at the most steps that the route takes, 242,
# 310 = 2 x 128 + 54, 378, 510 = 512 - 2, 518 = 512 + 6, 578, 650
@pytest.mark.parametrize("M1,M2,nb", [(4, 5, 1), (4, 4, 5), (4, 5, 11), (5, 5, 4), (2, 15, 3), (4, 10, 9), (7, 8, 6),
                                      (3, 18, 20), (8, 8, 24), (6, 12, 33)])
def test_krylov_bands_match_oracle(ctx, M1, M2, nb):
    phase, props = _cell(M1 * 31 + M2)
    Q = np.array([[0.0, 0.0], [0.31, 0.12], [0.5, 0.5]])
    print("krylov", M1, M2, nb, flush=True)
    om = ctx.cell(phase, props, OBLIQUE).plan(M1, M2).solve(Q, nb)
    ref, _ = mo.bands(phase, props, OBLIQUE, M1, M2, Q, nb)
    err = band_error(om, ref)
    print("  error", err, flush=True)
    assert np.all(np.isfinite(om)) and err <= TOL64


def test_krylov_same_by_every_entry(ctx):
    """One operator through solve (host and device output), solve_batch and
    solve_cells, and without waiting (the reduction): one result."""
    from paper_1310_6380_amd import mvpb
    phase, props = _cell(5)
    M, nb = 6, 5
    Q = np.array([[0.05, 0.21], [0.44, 0.1], [0.5, 0.5], [0.3, 0.3]])
    cell = ctx.cell(phase, props)
    plan = cell.plan(M)
    om = plan.solve(Q, nb)
    buf = mvpb.DeviceBuffer(om.nbytes)
    plan.solve_device(Q, nb, buf.value)
    assert np.array_equal(buf.to_numpy(np.float64, om.shape), om)
    assert np.array_equal(ctx.solve_batch([plan], [Q], nb)[0], om)
    assert band_error(ctx.solve_cells([cell], [M], [Q], nb)[0], om) <= 1e-10
    plan.solve_device(Q, nb, buf.value, mvpb.F_DEVICE_PTRS | mvpb.F_ASYNC)
    mvpb.device_synchronize()
    assert band_error(buf.to_numpy(np.float64, om.shape), om) <= 1e-10


def _folded(c, T, n, q, nb):
    """Sorted c |2 pi T (q + n)| over the plane waves n and the wave speeds c."""
    K = np.linalg.norm(2.0 * np.pi * (np.asarray(q)[None, :] + n) @ T.T, axis=1)
    return np.sort(np.concatenate([s * K for s in c]))[:nb]


def test_krylov_degenerate_planar(ctx):
    """Homogeneous cell: eightfold frequencies at Gamma."""
    E, nu, rho = 70e9, 0.33, 2700.0
    lam, mu = mo.lame(E, nu)
    c = (np.sqrt((lam + 2 * mu) / rho), np.sqrt(mu / rho))
    M, nb = 8, 20
    n = mo.plane_wave_indices(M, M)
    Q = np.array([[0.0, 0.0], [0.5, 0.5], [0.25, 0.0]])
    om = ctx.cell(np.zeros((8, 8), np.int32), np.array([[E, nu, rho]])).plan(M).solve(Q, nb)
    ref = np.stack([_folded(c, np.eye(2), n, q, nb) for q in Q])
    assert band_error(om, ref) <= TOL64


def test_krylov_more_copies_than_block(ctx):
    """Homogeneous cube at Gamma: 24 equal shear frequencies of the twelve
    waves (1, 1, 0), which no Krylov space of 16 vectors holds."""
    E, nu, rho = 3.5e9, 0.35, 1180.0
    mu, lam = E / (2 * (1 + nu)), E * nu / ((1 + nu) * (1 - 2 * nu))
    ct, cl = np.sqrt(mu / rho), np.sqrt((lam + 2 * mu) / rho)
    M, nb = 3, 40
    g = np.arange(-M, M + 1)
    n = np.stack(np.meshgrid(g, g, g, indexing="ij"), axis=-1).reshape(-1, 3)
    Q = np.array([[0.0, 0.0, 0.0], [0.13, 0.21, 0.34]])
    om = ctx.cell_voxels(np.zeros((6, 6, 6), np.int32), np.array([[E, nu, rho]])).plan(M).solve(Q, nb)
    ref = np.stack([_folded((ct, ct, cl), np.eye(3), n, q, nb) for q in Q])
    assert band_error(om, ref) <= TOL64


def test_krylov_modes(ctx):
    """Modes: H Phi^-1 H* U = lambda Omega U and U^H Omega U = 1."""
    phase, props = _cell(11)
    M, nb = 7, 9
    Q = np.array([[0.21, 0.35], [0.02, -0.4]])
    om, U = ctx.cell(phase, props).plan(M).solve(Q, nb, vectors=True)
    I = mo.subdomain_integral_tables(phase, props.shape[0], np.eye(2), M, M)
    for t, q in enumerate(Q):
        m = mo.assemble(I, props, np.eye(2), M, M, q)
        V = U[t].T
        A = m["H"] @ np.linalg.solve(m["Phi"], m["Hs"] @ V)
        B = m["Omega"] @ V
        # the residual in the norm of the low part of the spectrum
        res = np.linalg.norm(np.linalg.solve(m["Omega"], A - B * om[t] ** 2)) / \
            np.linalg.norm(np.linalg.solve(m["Omega"], B * om[t] ** 2))
        orth = np.abs(V.conj().T @ B - np.eye(nb)).max()
        print("  residual", res, "orthonormality", orth, flush=True)
        assert res <= 1e-7 and orth <= 1e-10


# (M1, M2, bands): 2N = 510 (8 blocks) and 578 = 9 x 64 + 2, one part; 650 = 10 x 64 + 10 in 2 of 5; 1250 = 19 x 64 + 34
# in 3 of 7, 7 and 6; all of them in one call with orders that the small and the general reduction take
def test_krylov_parts_mixed_with_other_routes(ctx):
    """The inverse factor in its parts, orders of one to three parts in one
    batch with orders that other routes take: as each plan alone."""
    Ms, nb = [(12, 12), (6, 12), (8, 8), (7, 8), (3, 3), (4, 4), (3, 18)], 5
    phase, props = _cell(77)
    cell = ctx.cell(phase, props, OBLIQUE)
    Q = np.random.default_rng(7).uniform(0.02, 0.5, (4, 2))
    print("parts", Ms, nb, flush=True)
    plans = [cell.plan(*M) for M in Ms]
    for M, plan, om in zip(Ms, plans, ctx.solve_batch(plans, [Q] * len(plans), nb)):
        assert np.array_equal(om, plan.solve(Q, nb)), M
        ref, _ = mo.bands(phase, props, OBLIQUE, *M, Q[:1], nb)
        print("  error", M, band_error(om[:1], ref), flush=True)
        assert band_error(om[:1], ref) <= TOL64


def _launches(ctx, call):
    """(what call returns, {kernel family: its launches})."""
    ctx.profile(True)
    out = call()
    n = {k: n for k, (_, n) in ctx.profile_read().items()}
    ctx.profile(False)
    return out, n


def _contrast_cell(geom, E, rho):
    """A 24 x 24 cell of soft (0) and hard (1) phases whose moduli and densities
    are in the ratios E and rho; coated: rubber-coated lead cylinders in epoxy."""
    x, y = np.meshgrid((np.arange(24) + 0.5) / 24 - 0.5, (np.arange(24) + 0.5) / 24 - 0.5, indexing="ij")
    r = np.hypot(x, y)
    if geom == "coated":
        phase = np.where(r < 0.27, 0, np.where(r < 0.36, 1, 2))
        return phase.astype(np.int32), np.array([[40.8e9, 0.37, 11600.0], [E, 0.47, 1300.0], [4.35e9, 0.37, 1180.0]])
    inside = r < 0.3 if geom == "circle" else (np.minimum(abs(x), abs(y)) < 0.12) & (np.maximum(abs(x), abs(y)) < 0.4)
    return inside.astype(np.int32), np.array([[1e9, 0.35, 1200.0], [1e9 * E, 0.33, 1200.0 * rho]])


CONTRASTS = [("circle", 1e3, 1.0), ("circle", 1e4, 1.0), ("circle", 1e5, 1.0), ("circle", 1e-3, 1.0), ("circle", 1e-4, 1.0),
             ("circle", 1e-5, 1.0), ("cross", 1e4, 8.0), ("cross", 1e-4, 0.5), ("circle", 10.0, 16.0), ("coated", 1e5, 0.0),
             ("coated", 1e7, 0.0)]


# 2N = 338 and 578 with the bands of small and of ordinary calls, 450 with modes (more steps, a lower bar), and the
# benchmark's 882 with 18 bands
@pytest.mark.parametrize("geom,E,rho,M,nb,modes",
                         [(*c, *s) for s in [(6, 4, False), (8, 10, False), (7, 4, True)] for c in CONTRASTS] +
                         [(*c, 10, 18, False) for c in CONTRASTS[1::4]])
def test_krylov_stands_at_large_contrast(ctx, geom, E, rho, M, nb, modes):
    """Cells of large stiffness ratio, as locally resonant crystals have it: the
    frequencies of the first attempt stand, and no point needs the reduction for its
    modes.  Two solvers that are backward stable to n eps of the largest eigenvalue
    differ by that, beside the bar of every FP64 path."""
    phase, props = _contrast_cell(geom, E, rho)
    Q = np.array([[0.0, 0.0], [0.02, 0.01], [0.31, 0.12], [0.5, 0.5]])
    plan = ctx.cell(phase, props).plan(M)
    print("contrast", geom, E, rho, M, nb, modes, flush=True)
    out, n = _launches(ctx, lambda: plan.solve(Q, nb, vectors=modes))
    om = out[0] if modes else out
    assert n["krylov_factor"] <= 1 + modes and n["krylov_factor"] > 0 and n["he2hb_panel"] == 0, n
    tabs = mo.subdomain_integral_tables(phase, props.shape[0], np.eye(2), M, M)
    m = mo.assemble(tabs, props, np.eye(2), M, M, Q[2])
    order = m["Omega"].shape[0]
    lam = mo.solve_k(m, order)[1]
    err = np.abs(om[2] ** 2 - lam[:nb])
    bar = 2.0 * TOL64 * lam[:nb] + order * np.finfo(np.float64).eps * lam[-1]
    print("  worst error over its bar", (err / bar).max(), flush=True)
    assert np.all(err <= bar)


# ratios below, at and above the benchmark's inclusion cells', few and more bands
@pytest.mark.parametrize("M,nb", [(7, 4), (8, 10)])
@pytest.mark.parametrize("E", [20.0, 100.0, 0.01])
def test_krylov_modes_to_rounding(ctx, E, M, nb):
    """Modes as a dense solve gives them: |C y - lambda y| within rounding of the
    largest eigenvalue, 4 sqrt(n) eps lambda_max, for C and y of the reduced problem."""
    phase, props = _contrast_cell("circle", E, 2.0)
    Q = np.array([[0.21, 0.35], [0.02, -0.4]])
    om, U = ctx.cell(phase, props).plan(M).solve(Q, nb, vectors=True)
    tabs = mo.subdomain_integral_tables(phase, 2, np.eye(2), M, M)
    for t, q in enumerate(Q):
        m = mo.assemble(tabs, props, np.eye(2), M, M, q)
        L = np.linalg.cholesky(0.5 * (m["Omega"] + m["Omega"].conj().T))
        C = np.linalg.solve(L, np.linalg.solve(L, mo.reduced_operator(m)).conj().T)
        y = L.conj().T @ U[t].T
        res = np.linalg.norm(C @ y - y * om[t] ** 2, axis=0)
        bar = 4.0 * np.sqrt(len(C)) * np.finfo(np.float64).eps * np.linalg.eigvalsh(C)[-1]
        print("modes", E, M, nb, "residual over its bar", (res / bar).max(), flush=True)
        assert np.all(res <= bar)


def test_krylov_shapes_are_its_own(tmp_path):
    """The autotuner's entry holds a shape for the reduction and one for the Krylov
    route; a plan that takes only the reduction leaves the other in the file, and a
    context that loads the file gives the same bands by both."""
    import json

    from paper_1310_6380_amd import mvpb
    phase, props = _cell(21)
    Q, nb, path = np.array([[0.31, 0.12], [0.5, 0.5], [0.2, 0.4]]), 6, str(tmp_path / "tuning.json")

    def entry():
        with open(path) as fh:
            lines = [json.loads(l.strip().rstrip(",")) for l in fh if '"device"' in l]
        assert len(lines) == 1
        return lines[0]

    def bands(load):
        c = mvpb.Context(0)
        try:
            if load:
                assert c.load_tuning(path) == 1
            plan = c.cell(phase, props).plan(7)
            if not load:
                plan.autotune(Q, nb, path)
            om = plan.solve(Q, nb)
            buf = mvpb.DeviceBuffer(om.nbytes)
            plan.solve_device(Q, nb, buf.value, mvpb.F_DEVICE_PTRS | mvpb.F_ASYNC)
            mvpb.device_synchronize()
            if not load:
                first = entry()
                assert first["krylov_group"] in (0, 1, 2, 4, 8) and first["parts"] in (1, 2, 3, 4)
                c.cell(phase, props).plan(7, None, mvpb.PREC_SF_FP32 | mvpb.PREC_EIG_FP32_RR64).autotune(Q, nb, path)
                assert (entry()["krylov_group"], entry()["krylov_wg"]) == (first["krylov_group"], first["krylov_wg"])
            return om, buf.to_numpy(np.float64, om.shape)
        finally:
            c.close()

    for a, b in zip(bands(False), bands(True)):
        assert np.array_equal(a, b)


# the orders of the edge cases above, planar and spatial
@pytest.mark.parametrize("M1,M2,nb,modes", [(4, 5, 1, False), (4, 5, 11, False), (2, 15, 3, True), (7, 8, 6, True), (3, 18, 20, False),
                                            (6, 12, 33, False), (12, 12, 5, False)])
def test_krylov_is_the_route_taken(ctx, M1, M2, nb, modes):
    """The bands above come from the route under test: one attempt, no reduction."""
    phase, props = _cell(M1 * 31 + M2)
    Q = np.array([[0.0, 0.0], [0.31, 0.12], [0.5, 0.5]])
    plan = ctx.cell(phase, props, OBLIQUE).plan(M1, M2)
    _, n = _launches(ctx, lambda: plan.solve(Q, nb, vectors=modes))
    assert n["krylov_factor"] == 1 and n["he2hb_panel"] == 0 and n["small_tridiag"] == 0, n


@pytest.mark.parametrize("spatial", [False, True])
def test_krylov_hands_points_on(ctx, spatial):
    """Sixteen equal frequencies (shear waves (3, 1) and pressure waves (2, 1) of a cell
    without lateral contraction) and the homogeneous cube's twenty-four, with modes: at
    Gamma a longer attempt, then the reduction; the other points keep what they have."""
    if spatial:
        E, nu, rho, M, nb = 3.5e9, 0.35, 1180.0, 3, 40
        plan = ctx.cell_voxels(np.zeros((6, 6, 6), np.int32), np.array([[E, nu, rho]])).plan(M)
        Q = np.array([[0.13, 0.21, 0.34], [0.0, 0.0, 0.0], [0.4, 0.1, 0.2]])
        g = np.arange(-M, M + 1)
        waves = np.stack(np.meshgrid(g, g, g, indexing="ij"), axis=-1).reshape(-1, 3)
    else:
        E, nu, rho, M, nb = 70e9, 0.0, 2700.0, 9, 60
        plan = ctx.cell(np.zeros((8, 8), np.int32), np.array([[E, nu, rho]])).plan(M)
        Q = np.array([[0.13, 0.21], [0.0, 0.0], [0.4, 0.1]])
        waves = mo.plane_wave_indices(M, M)
    lam, mu = mo.lame(E, nu)
    ct, cl = np.sqrt(mu / rho), np.sqrt((lam + 2 * mu) / rho)
    out, n = _launches(ctx, lambda: plan.solve(Q, nb, vectors=spatial))
    om = out[0] if spatial else out
    assert n["krylov_factor"] == 2 and n["he2hb_panel"] > 0, n
    ref = np.stack([_folded((ct, ct, cl) if spatial else (ct, cl), np.eye(Q.shape[1]), waves, q, nb) for q in Q])
    assert band_error(om, ref) <= TOL64
    alone = plan.solve(Q[[0, 2]], nb, vectors=spatial)
    assert np.array_equal(alone[0] if spatial else alone, om[[0, 2]])
    if spatial:
        assert np.array_equal(alone[1], out[1][[0, 2]])
        U = out[1][1].T
        assert np.abs(rho * (U.conj().T @ U) - np.eye(nb)).max() <= 1e-10


def test_krylov_polygon_cells(ctx):
    """Polygon cells take the route (their medium comes from the polygons' areas), and
    cells of phases next to incompressible are accepted as before."""
    from synth import hex_steel_epoxy
    c = hex_steel_epoxy(32)
    Q = np.array([[0.31, 0.12], [0.5, 0.25]])
    plan = ctx.cell_polygons(c.polygons, c.poly_phase, c.props, c.lattice).plan(6)
    om, n = _launches(ctx, lambda: plan.solve(Q, 6))
    assert n["krylov_factor"] == 1 and n["he2hb_panel"] == 0, n
    I = mo.polygon_integral_tables(c.polygons, c.poly_phase, c.n_phases, c.lattice, 6, 6)
    ref, _ = mo.bands(None, c.props, c.lattice, 6, 6, Q, 6, I_p=I)
    assert band_error(om, ref) <= TOL64
    props = np.array(c.props, dtype=np.float64)
    props[:, 1] = 0.5 - 2e-13
    assert np.all(np.isfinite(ctx.cell_polygons(c.polygons, c.poly_phase, props, c.lattice).plan(2).solve(Q, 4)))
