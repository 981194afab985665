"""Light-curve calls on lists of every length: rows and bins passed by value (up
to 64 rows, 511 bins) and through device memory, bins without columns and edges
outside the map, and traces of more rays than one staging block holds; against
the oracle's plain implementations, exactly."""
import numpy as np
import pytest

import paper_2308_14278_amd.lensmap as lm
from oracle.peak_stats import peak_stats
from oracle.peaks import find_peaks

pytestmark = pytest.mark.gpu


def _map(counts):
    import torch
    ny, nx = counts.shape
    g = lm.lm_geometry_derive(1.0, 1.0, nx, ny, 0.4, 0.1, 0.0, protect=0.0, ray_nx=64,
                              ray_ny=64, scheme=lm.LM_SCHEME_DIRECT, coarse=64)
    mp = lm.Map(g, 0.4, 0.1, 0.0, ([], [], []))
    buf = torch.from_numpy(np.ascontiguousarray(counts, dtype=np.int64)).cuda()
    torch.cuda.synchronize()
    lm.lm_bind_counts(mp.h, buf.data_ptr())
    return mp, g, buf


def _counts(ny, nx):
    rng = np.random.default_rng(ny * 1000 + nx)
    c = rng.poisson(200, size=(ny, nx)).astype(np.int64)
    for _ in range(ny * nx // 40):  # ridges over three rows: true peaks
        i, j = int(rng.integers(1, ny - 1)), int(rng.integers(1, nx - 1))
        c[i - 1:i + 2, j] += 400
    return c


@pytest.mark.parametrize("nx,n_tracks,bins", [
    (3, 1, 1), (255, 2, 3), (256, 63, 511), (257, 64, 510), (300, 65, 512), (130, 200, 700)])
def test_lists(nx, n_tracks, bins):
    ny = 40
    c = _counts(ny, nx)
    mp, g, buf = _map(c)
    tracks = [(7 * t) % ny for t in range(n_tracks)]
    flags = lm.lm_find_peaks(mp.h, g, tracks)
    want = np.array(find_peaks(c.tolist(), tracks, 5), dtype=np.uint8)
    np.testing.assert_array_equal(flags, want)
    x0, x1 = g.src_x0, g.src_x0 + g.src_nx * g.src_dx
    for lo, hi in ((x0, x1), (x0 - 1.0, x1 + 1.0), (x0 + 0.3, x0 + 0.7), (x1 + 1.0, x1 + 2.0)):
        edges = np.linspace(lo, hi, bins + 1)
        ref = peak_stats(c.tolist(), tracks, edges.tolist(), g.src_x0, g.src_dx)
        calls = [lm.lm_peak_stats] + ([lm.lm_peak_stats_noalloc] if bins <= 4096 else [])
        for f in calls:
            for a, b in zip(f(mp.h, tracks, edges), ref):
                np.testing.assert_array_equal(a, np.array(b, dtype=np.uint64))
    mp.close()


def test_flags_in_several_blocks():
    """More flags than the staging holds at a time: 45 rows of 2^19 pixels."""
    rng = np.random.default_rng(3)
    row = rng.poisson(200, size=1 << 19).astype(np.int64)
    row[::97] += 500
    c = np.stack([np.roll(row, r % 2) for r in range(45)])
    mp, g, buf = _map(c)
    tracks = list(range(44, -1, -1))
    flags = lm.lm_find_peaks(mp.h, g, tracks)
    one = np.stack([lm.lm_find_peaks(mp.h, g, [t])[0] for t in tracks])
    np.testing.assert_array_equal(flags, one)
    assert int((flags & 1).sum()) > 0
    mp.close()


def test_trace_in_several_blocks():
    """More rays than one staging block holds (16 MiB at 24 and 32 bytes a ray):
    equal to the same rays traced in parts."""
    rng = np.random.default_rng(5)
    g = lm.lm_geometry_derive(10.0, 10.0, 64, 64, 0.45, 0.5, 0.01, protect=0.0, ray_nx=2000,
                              ray_ny=1500, scheme=lm.LM_SCHEME_DIRECT, coarse=64)
    mp = lm.Map(g, 0.45, 0.5, 0.01, (rng.uniform(-9, 9, 3), rng.uniform(-9, 9, 3), np.ones(3)))
    n = 1_500_001
    i, j = rng.integers(0, 2000, n), rng.integers(0, 1500, n)
    p, q = mp.trace(i, j)
    b = mp.trace_beta(i, j)
    for s in (slice(0, 400_000), slice(400_000, 900_000), slice(1_400_000, n)):
        ps, qs = mp.trace(i[s], j[s])
        np.testing.assert_array_equal(p[s], ps)
        np.testing.assert_array_equal(q[s], qs)
        np.testing.assert_array_equal(b[s], mp.trace_beta(i[s], j[s]))
    ok = p >= 0
    u, v = (b[:, 0] - g.src_x0) / g.src_dx, (b[:, 1] - g.src_y0) / g.src_dy
    # the pixel is the floor of the coordinate: 64 pixels, rounding within 1e-9
    assert np.all((u[ok] > p[ok] - 1e-9) & (u[ok] < p[ok] + 1 + 1e-9))
    assert np.all((v[ok] > q[ok] - 1e-9) & (v[ok] < q[ok] + 1 + 1e-9))
    mp.close()
