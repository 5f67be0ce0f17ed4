"""The one-workgroup reduction of small operators (orders up to 128), at the
edges of its two sizes (64 and 128 rows) and of its groups of four columns, one
band and every band, against the oracle; the modes by their residual."""
import numpy as np
import pytest

from oracle import mixed3d_oracle as m3
from oracle import mixed_oracle as mo
from oracle.compare import band_error
from synth import random_iso_props

pytestmark = pytest.mark.gpu

TOL64 = 1e-9


@pytest.fixture(scope="module")
def ctx():
    from paper_1310_6380_amd import mvpb
    c = mvpb.Context(0)
    yield c
    c.close()


# 2N = 2, 18, 50, 54 = 64 - 10, 66 = 64 + 2, 98, 126 = 128 - 2, 130 = 128 + 2 (the two-stage reduction)
@pytest.mark.parametrize("M1,M2,nb", [(0, 0, 2), (1, 1, 18), (2, 2, 3), (1, 4, 20), (1, 5, 66), (3, 3, 6), (3, 4, 1),
                                      (3, 4, 126), (2, 6, 9)])
def test_small_bands_match_oracle(ctx, M1, M2, nb):
    rng = np.random.default_rng(10 * M1 + M2)
    phase, props = rng.integers(0, 3, (16, 18)).astype(np.int32), random_iso_props(3, rng)
    Q = np.array([[0.0, 0.0], [0.31, 0.12], [0.5, 0.5]])
    om = ctx.cell(phase, props).plan(M1, M2).solve(Q, nb)
    ref, _ = mo.bands(phase, props, np.eye(2), M1, M2, Q, nb)
    err = band_error(om, ref)
    print("small", M1, M2, nb, err, flush=True)
    assert err <= TOL64


def test_small_voxel_cell(ctx):
    rng = np.random.default_rng(3)
    phase, props = rng.integers(0, 2, (5, 4, 6)).astype(np.int32), random_iso_props(2, rng)
    Q = np.array([[0.1, 0.2, 0.3], [0.5, 0.0, 0.0]])
    om = ctx.cell_voxels(phase, props).plan(1).solve(Q, 10)
    ref, _ = m3.bands3(phase, props, np.eye(3), 1, 1, 1, Q, 10)
    assert band_error(om, ref) <= TOL64


@pytest.mark.parametrize("M", [2, 3])
def test_small_modes(ctx, M):
    rng = np.random.default_rng(7 + M)
    phase, props = rng.integers(0, 3, (12, 12)).astype(np.int32), random_iso_props(3, rng)
    Q, nb = np.array([[0.21, 0.35], [0.02, -0.4]]), 7
    om, U = ctx.cell(phase, props).plan(M).solve(Q, nb, vectors=True)
    I = mo.subdomain_integral_tables(phase, 3, np.eye(2), M, M)
    for t, q in enumerate(Q):
        m = mo.assemble(I, props, np.eye(2), M, M, q)
        V = U[t].T
        B = m["Omega"] @ V
        R = np.linalg.solve(m["Omega"], m["H"] @ np.linalg.solve(m["Phi"], m["Hs"] @ V)) - V * om[t] ** 2
        assert np.linalg.norm(R) <= 1e-9 * np.linalg.norm(V * om[t] ** 2)
        assert np.abs(V.conj().T @ B - np.eye(nb)).max() <= 1e-10
