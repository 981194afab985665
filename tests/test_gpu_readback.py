"""Read-back of counts, windows, magnifications and sums at the edges of its
staging: one lane, its chunks of 2^17 entries, several lanes; exact integers and
bit-equal magnifications against the caller's own buffer."""
import numpy as np
import pytest

import paper_2308_14278_amd.lensmap as lm

pytestmark = pytest.mark.gpu

CHUNK = 1 << 17


def _geometry(nx, ny):
    g = lm.lm_geometry_derive(10.0, 10.0, nx, ny, 0.45, 0.5, 0.01, protect=0.0, ray_nx=64,
                              ray_ny=64, scheme=lm.LM_SCHEME_DIRECT, coarse=64)
    return g


@pytest.mark.parametrize("nx,ny,offset", [
    (1, 1, 0), (3, 5, 1), (CHUNK - 1, 1, 0), (CHUNK, 1, 1), (CHUNK + 1, 1, 0),
    (1, 2 * CHUNK + 3, 0), (509, 521, 1), (4 * CHUNK - 1, 1, 0), (2003, 1999, 0),
    (37, 16 * CHUNK // 37 + 11, 1)])
def test_read_back(nx, ny, offset):
    import torch
    rng = np.random.default_rng(nx * 7 + ny)
    # counts over the whole range of 64 bits, small ones and zeros among them
    c = rng.integers(0, 2 ** 64, nx * ny, dtype=np.uint64) >> rng.integers(
        0, 64, nx * ny, dtype=np.uint64)
    c[:: 5] = 0
    buf = torch.zeros(nx * ny + 1, dtype=torch.int64, device="cuda")
    buf[offset:offset + nx * ny] = torch.from_numpy(c.view(np.int64)).cuda()
    torch.cuda.synchronize()
    g = _geometry(nx, ny)
    m = lm.Map(g, 0.45, 0.5, 0.01)
    lm.lm_bind_counts(m.h, buf.data_ptr() + 8 * offset)
    c = c.reshape(ny, nx)
    got, n_out, n_shot = m.counts()
    assert np.array_equal(got, c) and n_out == 0 and n_shot == 0
    assert lm.lm_read_counts(m.h, g, with_counts=False)[1:] == (0, 0)
    mu = lm.lm_read_mu(m.h, g)
    assert np.array_equal(mu.view(np.int64), (c.astype(np.float64) * m.mu_factor()).view(np.int64))
    assert lm.lm_sum_counts(m.h) == int(c.sum(dtype=np.uint64))
    for _ in range(4):
        p, q = int(rng.integers(0, nx)), int(rng.integers(0, ny))
        np_, nq = int(rng.integers(1, nx - p + 1)), int(rng.integers(1, ny - q + 1))
        win = lm.lm_read_counts_region(m.h, p, q, np_, nq)
        assert np.array_equal(win, c[q:q + nq, p:p + np_])
    m.close()


def test_read_back_from_two_threads():
    """Two maps read at the same time from two threads, while a third is made
    and destroyed: every read has a staging set of its own."""
    import threading

    import torch
    maps, want = [], []
    for k in range(2):
        g = _geometry(1500, 1400 + k)
        b = torch.arange(g.src_nx * g.src_ny, dtype=torch.int64, device="cuda") * (k + 3)
        m = lm.Map(g, 0.45, 0.5, 0.01)
        lm.lm_bind_counts(m.h, b.data_ptr())
        maps.append((m, g, b))
        want.append(b.cpu().numpy().view(np.uint64).reshape(g.src_ny, g.src_nx))
    torch.cuda.synchronize()
    bad = []

    def read(k):
        for _ in range(10):
            if not np.array_equal(maps[k][0].counts()[0], want[k]):
                bad.append(k)

    th = [threading.Thread(target=read, args=(k,)) for k in range(2)]
    for t in th:
        t.start()
    for _ in range(5):
        lm.Map(_geometry(8, 8), 0.45, 0.5, 0.01).close()
    for t in th:
        t.join()
    assert not bad
    for m, _, _ in maps:
        m.close()
