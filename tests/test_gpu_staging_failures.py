"""Calls whose staging cannot be had: with pinned memory refused, and with streams or
events refused beyond the first, every call returns what it returns otherwise.

Each setting runs in a process of its own, where a small library in front of the HIP
runtime refuses those calls; lens uploads of more than the pinned block (16 MiB) go
plainly in every one."""
import os
import subprocess
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

FRONT = r"""
#include <cstddef>
typedef int (*malloc_t)(void**, size_t, unsigned);
typedef int (*create_t)(void**, unsigned);
static malloc_t real_malloc;
static create_t real_stream, real_event;
static int pinned_left, streams_left, events_left;
extern "C" void front_set(void* m, void* s, void* e, int pinned, int streams, int events)
{
    real_malloc = (malloc_t)m;
    real_stream = (create_t)s;
    real_event = (create_t)e;
    pinned_left = pinned;
    streams_left = streams;
    events_left = events;
}
extern "C" int front_refused;
int front_refused = 0;
extern "C" int hipHostMalloc(void** p, size_t n, unsigned f)
{
    return pinned_left-- > 0 ? real_malloc(p, n, f) : (++front_refused, 2);  // out of memory
}
extern "C" int hipStreamCreateWithFlags(void** s, unsigned f)
{
    return streams_left-- > 0 ? real_stream(s, f) : (++front_refused, 2);
}
extern "C" int hipEventCreateWithFlags(void** e, unsigned f)
{
    return events_left-- > 0 ? real_event(e, f) : (++front_refused, 2);
}
"""

CHILD = r"""
import ctypes, sys
sys.path.insert(0, sys.argv[1])
front = ctypes.CDLL(sys.argv[2], mode=ctypes.RTLD_GLOBAL)
import numpy as np
import paper_2308_14278_amd.lensmap as lm
lm.load()
path = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l)
hip = ctypes.CDLL(path)
f = lambda n: ctypes.cast(getattr(hip, n), ctypes.c_void_p)
front.front_set(f("hipHostMalloc"), f("hipStreamCreateWithFlags"), f("hipEventCreateWithFlags"),
                *[ctypes.c_int(int(v)) for v in sys.argv[4:7]])
rng = np.random.default_rng(11)
out = {}
def lenses(n, m):
    return rng.uniform(-9, 9, n), rng.uniform(-9, 9, n), np.full(n, m)
g = lm.lm_geometry_derive(10.0, 10.0, 1300, 900, 0.45, 0.5, 0.01, protect=0.0, ray_nx=3000,
                          ray_ny=2500, scheme=lm.LM_SCHEME_DIRECT, coarse=64)
m = lm.Map(g, 0.45, 0.5, 0.01, lenses(40, 0.01))
m.shoot(stream=0)
c, n_out, n_shot = m.counts()
out.update(counts=c, n=np.array([n_out, n_shot, lm.lm_sum_counts(m.h)]), mu=lm.lm_read_mu(m.h, g))
out["n_only"] = np.array(lm.lm_read_counts(m.h, g, with_counts=False)[1:])
for k, w in enumerate([(0, 0, 1300, 1), (7, 5, 1, 800), (3, 2, 1290, 890), (1299, 899, 1, 1)]):
    out["window%d" % k] = lm.lm_read_counts_region(m.h, *w)
few, many = list(range(1, 880, 300)), [(13 * t) % 900 for t in range(70)]
for k, tr in enumerate((few, many)):
    out["flags%d" % k] = lm.lm_find_peaks(m.h, g, tr)
    for bins in (5, 600, 2000):
        e = np.linspace(g.src_x0, g.src_x0 + 1300 * g.src_dx, bins + 1)
        for q, v in enumerate(lm.lm_peak_stats(m.h, tr, e) + lm.lm_peak_stats(m.h, tr, e)):
            out["stats%d_%d_%d" % (k, bins, q)] = v
for n in (5, 800000):
    i, j = rng.integers(0, 3000, n), rng.integers(0, 2500, n)
    out["p%d" % n], out["q%d" % n] = m.trace(i, j)
    out["b%d" % n] = m.trace_beta(i, j)
m.close()
gi = lm.lm_geometry_derive(10.0, 10.0, 300, 300, 0.45, 0.5, 0.01, protect=1.0, n_rays=3e6, coarse=64)
mi = lm.Map(gi, 0.45, 0.5, 0.01, lenses(3000, 0.02))
p = mi.precision()
out["precision"] = np.array([v for v in (p if isinstance(p, tuple) else tuple(p.values()))], float)
mi.shoot(stream=0)
out["interp"] = mi.counts()[0]
mi.close()
# 600000 lenses: an upload of 19 MB
mb = lm.Map(g, 0.45, 0.5, 0.01, lenses(600000, 1e-6))
i, j = rng.integers(0, 3000, 40), rng.integers(0, 2500, 40)
out.update(big_i=i, big_j=j, big=mb.trace_beta(i, j))
mb.close()
np.savez(sys.argv[3], refused=np.array([ctypes.c_int.in_dll(front, "front_refused").value]), **out)
print("done", flush=True)
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    d = tmp_path_factory.mktemp("front")
    (d / "front.cpp").write_text(FRONT)
    (d / "child.py").write_text(CHILD)
    front = str(d / "libfront.so")
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", str(d / "front.cpp"), "-o", front],
                   check=True)

    def call(name, pinned, streams, events):
        out = str(d / (name + ".npz"))
        r = subprocess.run([sys.executable, str(d / "child.py"), ROOT, front, out, str(pinned),
                            str(streams), str(events)], capture_output=True, text=True, timeout=100)
        assert r.returncode == 0 and "done" in r.stdout, r.stderr[-2000:]
        return dict(np.load(out))

    return call


@pytest.fixture(scope="module")
def plain(run):
    got = run("plain", 1 << 20, 1 << 20, 1 << 20)
    assert got.pop("refused")[0] == 0
    return got


@pytest.mark.parametrize("name,pinned,streams,events", [
    ("no_pinned", 0, 1 << 20, 1 << 20), ("one_stream", 1 << 20, 1, 1 << 20),
    ("no_stream", 1 << 20, 0, 1 << 20), ("three_events", 1 << 20, 1 << 20, 3)])
def test_results_do_not_depend_on_staging(run, plain, name, pinned, streams, events):
    got = run(name, pinned, streams, events)
    assert got.pop("refused")[0] > 0
    assert got.keys() == plain.keys()
    for k in plain:
        np.testing.assert_array_equal(got[k], plain[k], err_msg=k)


def test_upload_beyond_the_pinned_block(plain):
    """The source positions of the 600000-lens field against the sum in 64 bits."""
    import torch
    assert torch.cuda.is_available()  # torch's HIP runtime first
    import paper_2308_14278_amd.lensmap as lm
    rng = np.random.default_rng(11)
    g = lm.lm_geometry_derive(10.0, 10.0, 1300, 900, 0.45, 0.5, 0.01, protect=0.0, ray_nx=3000,
                              ray_ny=2500, scheme=lm.LM_SCHEME_DIRECT, coarse=64)

    def lenses(n, m):
        return rng.uniform(-9, 9, n), rng.uniform(-9, 9, n), np.full(n, m)

    lenses(40, 0)
    for n in (5, 800000):
        rng.integers(0, 3000, n), rng.integers(0, 2500, n)
    lenses(3000, 0)
    x, y, m = lenses(600000, 1e-6)
    i, j = rng.integers(0, 3000, 40), rng.integers(0, 2500, 40)
    np.testing.assert_array_equal(plain["big_i"], i)
    np.testing.assert_array_equal(plain["big_j"], j)
    for k in range(40):
        tx, ty = g.ray_x0 + (i[k] + 0.5) * g.ray_dx, g.ray_y0 + (j[k] + 0.5) * g.ray_dy
        dx, dy = tx - x, ty - y
        w = m / (dx * dx + dy * dy)
        kappa_s = 0.45 - 0.01  # smooth matter; the lenses make up the rest
        bx = (1 - kappa_s - 0.5) * tx - (dx * w).sum()
        by = (1 - kappa_s + 0.5) * ty - (dy * w).sum()
        # FP32 terms of a few roundings, FP32 sums over blocks of 256: at most
        # (256 + 16) 2^-24 of the sum of their magnitudes; offsets of nearby lenses
        # are exact to 2^-24 of the lens's distance from the cell's centre
        # (below 1 theta_E where it matters)
        r = np.sqrt(dx * dx + dy * dy)
        tol = (272 * (m / r).sum() + (m / r ** 2).sum()) * 2.0 ** -24
        assert abs(plain["big"][k, 0] - bx) <= tol and abs(plain["big"][k, 1] - by) <= tol
