"""Workspace sizes of the emulated DGEMM, evaluated by a host program that
includes the library's own plan (no GPU): every group of a K-binned call fits
the area that the call reserves for its groups, and a short reduction fits a
limit whenever the smaller of its two layouts does."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2609_04663_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "dgemm_plan.h"
using namespace emu;

// groups of a K-binned call: cases, groups larger than the area with the shared
// layout choice, and with the choice that ignores the area
static void groups() {
    long cases = 0, over = 0, over_free = 0;
    for (int d = 1; d <= 11; ++d)
        for (int64_t M = 1; M <= 4200; M += M < 1300 ? 127 : 41)
            for (int64_t N = 1; N <= 4200; N += N < 1300 ? 127 : 41)
                for (int64_t KB = 1; KB <= 44; ++KB) {
                    const size_t area = dgemm_layout(d, M, N, KB * KBLK, true, 256).bytes;
                    for (int64_t kb = KB > 12 ? KB - 12 : 1; kb <= KB; ++kb) {
                        ++cases;
                        over += kbin_group_layout(d, M, N, kb * KBLK, 256, area).bytes > area;
                        over_free += dgemm_layout(d, M, N, kb * KBLK, true, 256).bytes > area;
                    }
                }
    printf("%ld %ld %ld\n", cases, over, over_free);
}

int main(int argc, char **argv) {
    if (!strcmp(argv[1], "groups")) {
        groups();
    } else {   // layout d M N K scaled limit -> bytes, panels
        const DgemmLayout L = dgemm_layout(atoi(argv[2]), atoll(argv[3]), atoll(argv[4]), atoll(argv[5]),
                                           atoi(argv[6]) != 0, 256, strtoull(argv[7], nullptr, 0));
        printf("%zu %d\n", L.bytes, (int)L.panels);
    }
}
"""
NO_LIMIT = str(2 ** 64 - 1)


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, exe = str(d / "plan.cpp"), str(d / "plan")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-I", CSRC, src, "-o", exe], check=True)

    def run(*args):
        out = subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True)
        return [int(x) for x in out.stdout.split()]
    return run


def test_kbin_groups_fit_the_shared_area(plan):
    cases, over, over_free = plan("groups")
    assert cases > 1_000_000 and over == 0
    # the choice that does not know the area exceeds it (d = 4, 25 k-blocks in all)
    assert over_free > 0


def test_group_of_24_of_25_k_blocks(plan):
    whole, panels = plan("layout", 4, 2112, 1536, 776, 1, NO_LIMIT)
    assert not panels
    group, panels = plan("layout", 4, 2112, 1536, 768, 1, NO_LIMIT)
    assert panels and group > whole
    fits, panels = plan("layout", 4, 2112, 1536, 768, 1, whole)
    assert not panels and fits <= whole


# the fixed scratch of emu_dgemm_noalloc: 64 MiB less its header
SCRATCH = (64 << 20) - 2048


@pytest.mark.parametrize("d,n,k", [(5, 6408, 320), (5, 10304, 289), (5, 4232, 545), (5, 5632, 545),
                                   (5, 3144, 800), (5, 4032, 800), (4, 7944, 512), (4, 3904, 1000)])
def test_short_reductions_within_the_scratch(plan, d, n, k):
    want, panels = plan("layout", d, n, n, k, 0, NO_LIMIT)
    got, other = plan("layout", d, n, n, k, 0, SCRATCH)
    assert want > SCRATCH and panels and got <= SCRATCH and not other
    # 2 d bytes an entry, rows to 64 and two tiles more, whole k-blocks of 32
    rows, kb = -(-n // 64) * 64 + 128, -(-k // 32)
    assert got == -(-2 * d * 2 * (kb * rows * 32 + 2048) // 256) * 256


def test_long_reductions_have_one_layout(plan):
    size, panels = plan("layout", 5, 4000, 4000, 1025, 0, NO_LIMIT)
    assert panels and plan("layout", 5, 4000, 4000, 1025, 0, size - 1) == [size, 1]


# 128 x 64 tiles at d = 4 and 64 x 64 ones at d = 6 against tiles of half the
# height: 2 rounds of 256 for 2, for 3, for 4; 3 for 5; 5 for 9
@pytest.mark.parametrize("d,m,n,panels", [
    (4, 1344, 1536, 0), (4, 1600, 1600, 0), (4, 2176, 1536, 1), (4, 3000, 3000, 1),
    (6, 1088, 1024, 0), (6, 1280, 1280, 1), (6, 1472, 1472, 1), (4, 1024, 1024, 0),
    (3, 1344, 1536, 1), (5, 1088, 1024, 1)])
def test_short_reductions_by_rounds(plan, d, m, n, panels):
    assert plan("layout", d, m, n, 1024, 0, NO_LIMIT)[1] == panels
    # longer ones as long as the tiles fill the CUs
    assert plan("layout", d, m, n, 1025, 0, NO_LIMIT)[1] == (m * n > 1024 * 1024 or d != 4)
