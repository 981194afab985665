"""The rule by which a single map's launch shares its tiles out over workgroups
(lm_split of the library's internal header), compiled for the host: short lists are
not split where more workgroups cost more than they save, long chains are, and
narrow rectangles run as many rays per lane as they have columns for."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DIRECT, FP32, FP64 = 0, 1, 2

SRC = r"""
#include <cstdio>
#include "lm_internal.h"
int main()
{
    int form, R, ncc, cw, G, cus;
    long long tiles, ni, nj;
    double list, longest;
    while (std::scanf("%d %d %d %d %d %lld %lld %lld %lf %lf %d", &form, &R, &ncc, &cw, &G, &tiles,
                      &ni, &nj, &list, &longest, &cus) == 11) {
        const LmSplit e = lm_split(form, R, ncc, cw, G, tiles, ni, nj, list, longest, cus);
        std::printf("%d %d %d\n", e.split, e.cw, e.nr);
    }
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("split")
    src, exe = str(d / "split.cpp"), str(d / "split")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2308_14278_amd", "csrc"), src, "-o", exe], check=True)

    def call(form, R, ni, nj, lens, G=1, cus=256, longest=None):
        ncc = {64: 4, 128: 2, 192: 4, 320: 4, 512: 1}[R]
        tiles = -(-ni // R) * -(-nj // R)
        args = " ".join(str(v) for v in (form, R, ncc, R // ncc, G, tiles, ni, nj, lens,
                                         lens if longest is None else longest, cus))
        r = subprocess.run([exe], input=args, capture_output=True, text=True, check=True)
        return tuple(int(v) for v in r.stdout.split())

    return call


@pytest.mark.parametrize("form", [DIRECT, FP32, FP64])
@pytest.mark.parametrize("ni,nj", [(12000, 35), (1000, 1000), (1400, 1400), (2000, 2000)])
def test_short_lists_are_not_split(rule, form, ni, nj):
    # cells of 64 rays: 16 columns a chunk, one step; a split costs more than it saves
    for lens in (0, 1, 3, 10):
        assert rule(form, 64, ni, nj, lens) == (1, 16, 16)


@pytest.mark.parametrize("form,R,ni,nj,lens,want", [
    (DIRECT, 64, 250, 190, 31, (4, 4, 4)), (DIRECT, 64, 1000, 1000, 300, (2, 8, 8)),
    (FP32, 64, 1000, 1000, 300, (2, 8, 8)), (FP64, 64, 1000, 1000, 300, (2, 8, 8)),
    (FP32, 128, 1000, 1000, 10, (4, 16, 16)), (FP32, 128, 2000, 2000, 300, (4, 16, 16)),
    # five rows of 128: half the waves of a workgroup are idle
    (FP64, 128, 57000, 5, 300, (4, 16, 16))])
def test_long_chains_are_split(rule, form, R, ni, nj, lens, want):
    assert rule(form, R, ni, nj, lens) == want


def test_the_longest_list_makes_the_chain(rule):
    assert rule(FP32, 128, 2000, 2000, 3) == (1, 64, 16)
    assert rule(FP32, 128, 2000, 2000, 3, longest=60)[0] > 1


@pytest.mark.parametrize("form", [DIRECT, FP32, FP64])
def test_large_tiles_and_launches_stay_whole(rule, form):
    assert rule(form, 64, 1000, 1000, 200, G=2) == (1, 16, 16)
    for R in (64, 128, 192, 320, 512):
        split, cw, nr = rule(form, R, 400 * R, 30 * R, 200)
        assert split == 1 and nr == 16


@pytest.mark.parametrize("cus", [64, 256, 304])
@pytest.mark.parametrize("form", [DIRECT, FP32, FP64])
def test_chunks_cover_the_cells(rule, form, cus):
    for R in (64, 128, 192, 320, 512):
        for ni, nj in ((1, 1), (5, 5000), (64, 64), (4097, 3), (1000, 700), (3000, 3000)):
            for lens in (0, 7, 80, 5000):
                split, cw, nr = rule(form, R, ni, nj, lens, cus=cus)
                whole = R // {64: 4, 128: 2, 192: 4, 320: 4, 512: 1}[R]
                assert split * cw == whole and cw % 4 == 0 and nr in (4, 8, 16)


@pytest.mark.parametrize("form", [DIRECT, FP32, FP64])
@pytest.mark.parametrize("ni,nr", [(1, 4), (3, 4), (4, 8), (5, 8), (7, 8)])
def test_narrow_rectangles_run_fewer_rays_per_lane(rule, form, ni, nr):
    assert rule(form, 320, ni, 700 * 320, 0) == (1, 80, nr)


def test_long_direct_lists(rule):
    """Lists of several blocks of lenses run 16 rays per lane two waves to a SIMD: full
    launches take 8."""
    assert rule(DIRECT, 64, 9000, 9000, 256)[2] == 16
    assert rule(DIRECT, 64, 9000, 9000, 257)[2] == 8
