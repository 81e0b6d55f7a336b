"""CPU check of the rule that gives a launch the stencil's tile form
(``tile_plan.h``, compiled by g++): which of its launches take tiles on lattices
on both sides of each of its lines, and that a tile divides its lattice, fits its
block and its rows are whole lines."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "csrc/tile_plan.h"
using namespace ovl;
int main(int argc, char **argv)
{
    int E[4];
    for (int k = 0; k < 4; k++) E[k] = atoi(argv[1 + k]);
    const Tile t = pick_tile(E, (int64_t)E[0] * E[1] * E[2] * E[3]);
    std::printf("%d %d %d", t.nt, t.nt ? tile_sites(t) : 0, t.nt ? tile_count(t) : 0);
    for (int k = 0; k < 4; k++) std::printf(" %d", t.nt ? t.T[k] : 0);
    // FP64 and 48 bits: launches without partial sums, with them; 1, 2, 3 and 12 fields
    for (int f64 = 1; f64 >= 0; f64--)
        for (int sums = 0; sums < 2; sums++) {
            std::printf(" ");
            for (int n : {1, 2, 3, 12}) std::printf("%d", t.nt && tile_pays(t, f64, n, sums, tile_count(t) <= 512));
        }
    std::printf("\n");
    // division by the extents as the kernel does it
    if (t.nt)
        for (unsigned n = 0; n < 512; n++)
            if (n * t.m3 >> 20 != n / t.T[3] || n * t.m2 >> 20 != n / t.T[2] || n * t.m1 >> 20 != n / t.T[1]) return 1;
    return 0;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not on PATH")
    d = tmp_path_factory.mktemp("plan")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "plan")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_1410_7170_amd"),
                           str(d / "main.cpp"), "-o", exe])

    def run(dims):
        r = subprocess.run([exe] + [str(v) for v in dims], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0, (dims, r.stdout)
        w = r.stdout.split()
        return [int(v) for v in w[:3]], [int(v) for v in w[3:7]], w[7:]

    return run


NO = ["0000"] * 4
# lattice, threads a block, sites, tiles, then FP64 and 48 bits, each without
# and with partial sums, on 1, 2, 3 and 12 fields
CASES = [
    ((30, 16, 16, 16), 0, 0, 0, NO),                                        # below 131072 sites
    ((34, 2, 44, 46), 0, 0, 0, NO),                                         # rows of 46: neither whole nor in eights
    ((32, 16, 16, 16), 512, 512, 256, ["1111"] * 4),                        # every thread has a site
    ((8, 8, 32, 64), 512, 512, 256, ["1111"] * 4),                          # rows cut in two
    ((64, 16, 16, 8), 512, 512, 256, ["1111", "1111", "1110", "1111"]),     # rows of 8
    ((18, 18, 18, 24), 512, 288, 486, ["1100", "1000", "0000", "1000"]),    # share 0.56, carries
    ((36, 16, 16, 16), 512, 384, 384, ["1111", "1000", "0000", "1000"]),    # share 0.75, carries
    ((24, 22, 22, 22), 512, 352, 726, ["1100", "0000", "0000", "0000"]),    # share 0.69, too many sums
    ((28, 26, 30, 30), 512, 300, 2184, ["1000", "0000", "0000", "0000"]),   # above 2^19 sites
    ((20, 22, 26, 30), 512, 480, 715, ["1111", "1000", "1000", "1000"]),    # share 0.94
    ((10, 30, 26, 28), 256, 224, 975, ["1111", "1000", "1000", "1000"]),    # share 0.875 of 256
    ((26, 22, 22, 20), 256, 160, 1573, ["1100", "0000", "0000", "0000"]),
]


@pytest.mark.parametrize("dims,nt,sites,count,takes", CASES)
def test_rule(plan, dims, nt, sites, count, takes):
    head, extents, got = plan(dims)
    assert head == [nt, sites, count] and got == takes
    if nt:
        assert all(e % t == 0 for e, t in zip(dims, extents)) and nt // 2 < sites <= nt
        assert extents[3] == dims[3] or extents[3] % 8 == 0
