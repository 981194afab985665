"""Far-field coefficients at the edges of their kernels against the oracle: the
direct sums with waves that span several level-1 cells or wrap over lattice rows,
lists with no far or no near lens, every number of terms and the FP32 form; the
level-1 series at every split of its slices over threads.

Tolerances: a_0 is a sum of at most 400 terms, each right to a few ulps, in FP64
on both sides, so it agrees to 400 x 2^-53 < 1e-13 of the sum of the terms'
sizes; the re-expanded series multiplies that by at most 1 / (1 - rho)^4 < 20
(rho <= 0.38).  1e-11 of the terms' sizes covers both.  a_1.. are rounded to FP32
(2^-24).  The FP32 form's terms carry a few FP32 ulps each: 1e-5."""
import numpy as np
import pytest

import paper_2308_14278_amd.lensmap as lm
from tests.helpers import oracle_geom

pytestmark = pytest.mark.gpu


def _geometry(nx, ny, kx, ky, halo, terms, far_order=0, precision=lm.LM_PREC_MIXED):
    g = lm.lm_geometry_derive(4.0, 4.0, 32, 32, 0.5, 0.2, 0.01, protect=0.0, ray_nx=nx,
                              ray_ny=ny, coarse=64)
    g.l1_kx, g.l1_ky, g.near_halo, g.taylor_terms = kx, ky, halo, terms
    g.far_order, g.precision = far_order, precision
    return g


def _check(g, lenses, oracle_lib, tol=1e-11):
    m = lm.Map(g, 0.5, 0.2, 0.01, lenses)
    orc = oracle_lib.Oracle(oracle_geom(g), 0.5, 0.2, 0.01, *lenses)
    x, y, mass = lenses
    ncx, ncy = -(-g.ray_nx // g.coarse), -(-g.ray_ny // g.coarse)
    for cj in range(ncy):
        for ci in range(ncx):
            got = lm.lm_read_coeffs(m.h, ci, cj, g.taylor_terms)
            ref = orc.coeffs(ci, cj)
            z = complex(g.ray_x0 + (ci + 0.5) * g.coarse * g.ray_dx,
                        g.ray_y0 + (cj + 0.5) * g.coarse * g.ray_dy)
            far = ~orc.near_mask(ci, cj)
            r = np.abs(x[far] + 1j * y[far] - z)
            for n in range(g.taylor_terms):
                size = float((mass[far] / r ** (n + 1)).sum())
                lim = tol * size + (2.0 ** -24 * abs(ref[n]) if n else 0.0)
                assert abs(got[n] - ref[n]) <= lim, (ci, cj, n, got[n], ref[n], size)
    m.close()


def _lenses(g, n, spread, seed):
    rng = np.random.default_rng(seed)
    hx, hy = spread * g.ray_nx * g.ray_dx / 2, spread * g.ray_ny * g.ray_dy / 2
    return rng.uniform(-hx, hx, n), rng.uniform(-hy, hy, n), rng.uniform(0.1, 1.0, n)


@pytest.mark.parametrize("nx,ny,kx,ky,halo,terms,n,spread", [
    (1280, 200, 3, 2, 1, 4, 400, 2.0),    # a wave over many level-1 cells, partial rows
    (130, 1300, 2, 5, 1, 4, 397, 2.0),    # waves that wrap over 22 rows
    (64, 64, 1, 1, 0, 1, 5, 3.0),         # one cell, no halo
    (700, 330, 4, 3, 2, 7, 259, 1.5),
    (700, 330, 40, 30, 1, 3, 100, 3.0),   # one level-1 cell: the rest is far
    (700, 330, 40, 30, 3, 2, 60, 1.0),    # every lens near
    (300, 260, 2, 2, 1, 5, 3, 1.0), (300, 260, 2, 2, 1, 6, 0, 1.0)])
def test_direct_coefficients(nx, ny, kx, ky, halo, terms, n, spread, oracle_lib):
    g = _geometry(nx, ny, kx, ky, halo, terms)
    _check(g, _lenses(g, n, spread, nx + n), oracle_lib)


def test_direct_coefficients_fp32(oracle_lib):
    g = _geometry(700, 330, 3, 2, 1, 4, precision=lm.LM_PREC_FP32)
    _check(g, _lenses(g, 300, 2.0, 8), oracle_lib, tol=1e-5)


@pytest.mark.parametrize("far_order,halo", [
    (5, 60), (8, 12), (9, 12), (16, 3), (17, 3), (24, 1), (31, 1), (33, 1), (40, 1), (41, 1),
    (48, 1), (49, 1), (56, 1), (57, 1), (64, 1)])
def test_series_coefficients(far_order, halo, oracle_lib):
    # square level-1 cells of 5 x 5: rho = sqrt(8) / (5 halo + 2.5)
    g = _geometry(1280, 1280, 5, 5, halo, 4, far_order)
    g.ray_dy = g.ray_dx
    g.ray_y0 = -g.ray_dy * g.ray_ny / 2
    _check(g, _lenses(g, 300, 6.0 + 8 * halo, far_order), oracle_lib)
