"""Magnifications of small maps at the edges of what the runtime's copy reads (2049 to
8192 entries): bit-equal to the counts times the factor, converted in 64 bits."""
import numpy as np
import pytest

import paper_2308_14278_amd.lensmap as lm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(2048, 1), (2049, 1), (64, 64), (3, 1501), (8192, 1), (8193, 1)])
def test_small_magnification_maps(nx, ny):
    import torch
    rng = np.random.default_rng(nx + ny)
    c = rng.integers(0, 2 ** 64, nx * ny, dtype=np.uint64) >> rng.integers(
        0, 64, nx * ny, dtype=np.uint64)
    buf = torch.from_numpy(c.view(np.int64)).cuda()
    torch.cuda.synchronize()
    g = lm.lm_geometry_derive(10.0, 10.0, nx, ny, 0.45, 0.5, 0.01, protect=0.0, ray_nx=64,
                              ray_ny=64, scheme=lm.LM_SCHEME_DIRECT, coarse=64)
    m = lm.Map(g, 0.45, 0.5, 0.01)
    lm.lm_bind_counts(m.h, buf.data_ptr())
    for _ in range(2):
        mu = lm.lm_read_mu(m.h, g)
        want = c.reshape(ny, nx).astype(np.float64) * m.mu_factor()
        assert np.array_equal(mu.view(np.int64), want.view(np.int64))
    m.close()
