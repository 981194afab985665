"""Peak statistics at the edges of their launches: bins on both sides of what the
last workgroup hands over itself (1024) and of the columns of the map, rows on both
sides of what is passed by value (64) and of one row per workgroup row, exactly as
the oracle counts them, twice (the histograms are left zero)."""
import numpy as np
import pytest

import paper_2308_14278_amd.lensmap as lm
from oracle.peak_stats import peak_stats
from tests.test_gpu_curve_lists import _counts, _map

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,n_tracks,bins", [
    (3, 1, 1024), (3, 65, 1025), (257, 600, 256), (257, 64, 257), (700, 300, 1024),
    (700, 65, 1025), (1025, 70, 1023), (64, 10, 20000), (300, 3, 65536), (5000, 40, 4096)])
def test_hand_off(nx, n_tracks, bins):
    ny = 40
    c = _counts(ny, nx)
    mp, g, buf = _map(c)
    tracks = [(7 * t) % ny for t in range(n_tracks)]
    x0, x1 = g.src_x0, g.src_x0 + g.src_nx * g.src_dx
    for lo, hi in ((x0 - 0.1, x1), (x0 + 0.3, x0 + 0.7)):
        edges = np.linspace(lo, hi, bins + 1)
        ref = peak_stats(c.tolist(), tracks, edges.tolist(), g.src_x0, g.src_dx)
        for f in [lm.lm_peak_stats] * 2 + ([lm.lm_peak_stats_noalloc] * 2 if bins <= 4096 else []):
            for a, b in zip(f(mp.h, tracks, edges), ref):
                np.testing.assert_array_equal(a, np.array(b, dtype=np.uint64))
    mp.close()


def test_flags_and_statistics_of_more_rows_than_the_scratch_takes():
    """2^20 + 5 rows of an 8-pixel map: their list goes up by a plain copy."""
    c = _counts(40, 8)
    mp, g, buf = _map(c)
    n = (1 << 20) + 5
    tracks = (np.arange(n) * 7 % 40).astype(np.int32)
    edges = np.linspace(g.src_x0, g.src_x0 + 8 * g.src_dx, 4)
    flags = lm.lm_find_peaks(mp.h, g, tracks)
    rows = np.stack([lm.lm_find_peaks(mp.h, g, [t])[0] for t in range(40)])
    np.testing.assert_array_equal(flags, rows[tracks])
    one = [lm.lm_peak_stats(mp.h, [t], edges) for t in range(40)]
    times = np.bincount(tracks, minlength=40).astype(np.uint64)
    for q, v in enumerate(lm.lm_peak_stats(mp.h, tracks, edges)):
        want = sum(times[t] * one[t][q] for t in range(40))
        np.testing.assert_array_equal(v, want)
    mp.close()
