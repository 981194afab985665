"""Every near-sum form of the interpolated scheme at 4, 8 and 16 rays per lane, on
near lists of zero lenses to several table blocks and ragged rectangles, linear
and fold: the batched counts are those of the rays traced one by one, exactly."""
import numpy as np
import pytest

import paper_2308_14278_amd.lensmap as lm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [lm.LM_PREC_MIXED, lm.LM_PREC_MIXED_CENTRED,
                                       lm.LM_PREC_MIXED_FP64, lm.LM_PREC_FP32])
@pytest.mark.parametrize("n,terms", [(0, 4), (1, 4), (17, 1), (40, 4), (300, 4), (700, 7)])
@pytest.mark.parametrize("fold", [False, True])
def test_lanes(precision, n, terms, fold):
    rng = np.random.default_rng(n + terms)
    if fold:
        g = lm.lm_geometry_derive_fold(6.0, 4.0, 61, 47, 0.83, 2e-2, 0.01, margin=0.5,
                                       n_rays=1.2e5, coarse=64)
    else:
        g = lm.lm_geometry_derive(6.0, 4.0, 61, 47, 0.5, 0.2, 0.01, protect=0.3, ray_nx=411,
                                  ray_ny=301, coarse=64)
    g.precision, g.taylor_terms = precision, terms
    g.l1_kx = g.l1_ky = 2
    hx, hy = g.ray_nx * g.ray_dx / 2, g.ray_ny * g.ray_dy / 2
    lenses = (rng.uniform(-hx, hx, n), rng.uniform(-hy, hy, n), rng.uniform(0.1, 1.0, n) / 50)
    if fold:
        m = lm.Map(g, kappa_star=0.01, lenses=lenses, fold=(0.83, 2e-2, -1.5e-2))
    else:
        m = lm.Map(g, 0.5, 0.2, 0.01, lenses)
    i0, j0, ni, nj = 61, 3, min(301, g.ray_nx - 61), min(203, g.ray_ny - 3)
    jj, ii = np.mgrid[j0:j0 + nj, i0:i0 + ni]
    p, q = m.trace(ii.ravel(), jj.ravel())
    want = np.zeros((g.src_ny, g.src_nx), dtype=np.uint64)
    np.add.at(want, (q[p >= 0], p[p >= 0]), 1)
    m.shoot(i0, j0, ni, nj)
    c, n_out, _ = m.counts()
    np.testing.assert_array_equal(c, want)
    assert n_out == int((p < 0).sum())
    for nr in (4, 8, 16):
        m.reset()
        b = lm.lm_batch_create([m.h])
        lm.lm_batch_set_rect(b, 0, i0, j0, ni, nj)
        lm.lm_batch_set_params(b, nr, 1, 0, 0)
        lm.lm_batch_shoot(b)
        np.testing.assert_array_equal(m.counts()[0], want)
        lm.lm_batch_destroy(b)
    m.close()
