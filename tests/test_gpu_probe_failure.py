"""A precision probe that fails half way waits for the kernels it has launched before its
scratch goes back to the device's sets, and the next probe is not changed by it.

In a process of its own, where a small library in front of the HIP runtime refuses the
copy of the probe's sums and counts the waits that follow."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

FRONT = r"""
#include <cstddef>
typedef int (*copy_t)(void*, const void*, size_t, int, void*);
typedef int (*wait_t)(void*);
static copy_t real_copy;
static wait_t real_wait;
static int armed;
extern "C" int front_refused, front_waits;
int front_refused = 0, front_waits = 0;
extern "C" void front_set(void* c, void* w)
{
    real_copy = (copy_t)c;
    real_wait = (wait_t)w;
}
extern "C" void front_arm(int on) { armed = on; }
extern "C" int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st)
{
    return armed ? (++front_refused, 2) : real_copy(d, s, n, k, st);
}
extern "C" int hipStreamSynchronize(void* s)
{
    if (armed && front_refused) ++front_waits;
    return real_wait(s);
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
front.front_set(f("hipMemcpyAsync"), f("hipStreamSynchronize"))
count = lambda n: ctypes.c_int.in_dll(front, n).value
rng = np.random.default_rng(11)
lenses = (rng.uniform(-9, 9, 3000), rng.uniform(-9, 9, 3000), np.full(3000, 0.02))
g = lm.lm_geometry_derive(10.0, 10.0, 300, 300, 0.45, 0.5, 0.01, protect=1.0, n_rays=3e6, coarse=64)
want = lm.Map(g, 0.45, 0.5, 0.01, lenses)
first = want.precision()
m = lm.Map(g, 0.45, 0.5, 0.01, lenses)
front.front_arm(1)
try:
    m.precision()
    raise SystemExit("the refused copy went unnoticed")
except lm.LensmapError:
    pass
front.front_arm(0)
assert count("front_refused") == 1, count("front_refused")
assert count("front_waits") >= 1, "the scratch went back before its kernels had ended"
assert m.precision() == first, (m.precision(), first)
print("done", flush=True)
"""


def test_failed_probe_waits_for_its_kernels(tmp_path):
    (tmp_path / "front.cpp").write_text(FRONT)
    (tmp_path / "child.py").write_text(CHILD)
    front = str(tmp_path / "libfront.so")
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", str(tmp_path / "front.cpp"), "-o", front],
                   check=True)
    r = subprocess.run([sys.executable, str(tmp_path / "child.py"), ROOT, front],
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "done" in r.stdout, (r.stdout + r.stderr)[-2000:]
