"""The direct sum at the edges of its blocks (256 lenses), steps (8 columns) and
units, per map and batched at 4, 8 and 16 rays per lane: the counts are those of
the rays traced one by one, exactly, and of the FP64 oracle within the FP32
bin-mismatch bar."""
import numpy as np
import pytest

import paper_2308_14278_amd.lensmap as lm
from tests.helpers import mismatch_fraction, oracle_geom

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [0, 1, 2, 255, 256, 257, 512, 513])
@pytest.mark.parametrize("rect", [(0, 0, 150, 131), (1, 3, 77, 64), (63, 65, 2, 1)])
def test_direct_blocks(n, rect, oracle_lib):
    rng = np.random.default_rng(100 + n)
    lenses = (rng.uniform(-12, 12, n), rng.uniform(-6, 6, n), rng.uniform(0.1, 1.0, n) / 20)
    g = lm.lm_geometry_derive(10.0, 10.0, 61, 53, 0.45, 0.25, 0.01, protect=0.0, ray_nx=150,
                              ray_ny=131, scheme=lm.LM_SCHEME_DIRECT, coarse=64)
    m = lm.Map(g, 0.45, 0.25, 0.01, lenses)
    i0, j0, ni, nj = rect
    jj, ii = np.mgrid[j0:j0 + nj, i0:i0 + ni]
    p, q = m.trace(ii.ravel(), jj.ravel())
    want = np.zeros((g.src_ny, g.src_nx), dtype=np.uint64)
    np.add.at(want, (q[p >= 0], p[p >= 0]), 1)
    ref, _ = oracle_lib.Oracle(oracle_geom(g), 0.45, 0.25, 0.01, *lenses).shoot(i0, j0, ni, nj)
    # rays whose FP32 image crosses a pixel edge: a few ulps of ~512 near sums,
    # |error| < 1e-5 pixels, so below one of 1e4 rays is expected to differ
    assert mismatch_fraction(want, ref, ni * nj) <= 2.0 / (ni * nj)
    m.shoot(i0, j0, ni, nj)
    c, n_out, n_shot = m.counts()
    np.testing.assert_array_equal(c, want)
    assert n_out == int((p < 0).sum()) and n_shot == ni * nj
    for nr in (4, 8, 16):
        m.reset()
        b = lm.lm_batch_create([m.h])
        lm.lm_batch_set_rect(b, 0, i0, j0, ni, nj)
        lm.lm_batch_set_params(b, nr, 1, 0, 0)
        lm.lm_batch_shoot(b)
        np.testing.assert_array_equal(m.counts()[0], want)
        lm.lm_batch_destroy(b)
    m.close()
