"""The pool of staging sets (DevicePool of the library's host code), compiled for the
host: each device keeps its own sets, whatever the others hold; the number kept is
bounded; the sets of a device go with its last map and no earlier; threads never
share one."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <atomic>
#include <cassert>
#include <cstdio>
#include <thread>
#include <vector>
#include "lm_pool.h"
static std::atomic<int> made{0}, gone{0};
struct Set {
    int device;
    std::atomic<int> in_use{0};
    explicit Set(int d) : device(d) { ++made; }
    ~Set() { ++gone; }
};
static DevicePool<Set, 4, 8> pool;
static void call(int device)
{
    Set* s = pool.take(device);
    if (!s) s = new Set(device);
    assert(s->device == device && s->in_use++ == 0);
    --s->in_use;
    if (!pool.keep(device, s)) delete s;
}
int main()
{
    // one map on each of eight devices, called in turn: a set each, made once
    for (int d = 0; d < 8; ++d) pool.enter(d);
    for (int r = 0; r < 100; ++r)
        for (int d = 0; d < 8; ++d) call(d);
    assert(made == 8 && gone == 0);
    // the last map of a device takes its set along, the others keep theirs
    pool.enter(3);
    pool.leave(3);
    assert(gone == 0);
    pool.leave(3);
    assert(gone == 1);
    call(3);  // no map: nothing is kept
    assert(made == 9 && gone == 2);
    for (int d = 0; d < 8; ++d)
        if (d != 3) call(d);
    assert(made == 9);
    // three threads on one device find a set each after the first calls
    pool.enter(3);
    std::vector<Set*> held;
    for (int k = 0; k < 6; ++k) held.push_back(new Set(3));
    int kept = 0;
    for (Set* s : held)
        if (pool.keep(3, s)) ++kept; else delete s;
    assert(kept == 4);
    const int before = made;
    std::vector<std::thread> th;
    for (int t = 0; t < 3; ++t)
        th.emplace_back([] { for (int r = 0; r < 20000; ++r) call(3); });
    for (auto& t : th) t.join();
    assert(made == before);
    // maps come and go while others are in use
    for (int t = 0; t < 3; ++t)
        th[t] = std::thread([t] {
            for (int r = 0; r < 5000; ++r) { pool.enter(t); call(t); pool.leave(t); }
        });
    for (auto& t : th) t.join();
    for (int d = 0; d < 8; ++d) pool.leave(d);
    assert(made == gone);
    // no such device: never kept
    pool.enter(8); pool.enter(-1);
    assert(!pool.take(8) && !pool.take(-1));
    call(8);
    assert(made == gone);
    std::puts("ok");
}
"""


def test_pool(tmp_path):
    src, exe = str(tmp_path / "pool.cpp"), str(tmp_path / "pool")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-Werror", "-pthread", "-I",
                    os.path.join(ROOT, "paper_2308_14278_amd", "csrc"), src, "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stderr
