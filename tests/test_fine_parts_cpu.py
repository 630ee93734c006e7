"""Row ranges of the fine-tile plans, up to the most rows the entry points take:
the plan and the range arithmetic of the kernel are compiled for the host.  The
ranges are formed in constant expressions too, where an overflow of a 32-bit
value does not compile."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1902_02104_amd", "csrc")

SOURCE = r"""
#include <climits>
#include <cstdio>
#include <cstdlib>
#include "ata_plan.h"
using namespace atalib;
static_assert(part_end(INT_MAX, 511 * 4194304, 4194304) == INT_MAX, "");
static_assert(part_end(INT_MAX, 0, INT_MAX) == INT_MAX, "");
static_assert(part_stages(INT_MAX, 32) == 67108864, "");
// (the plain sums of the other calls: ra + rows and rb - ra + KS - 1, KS at most 32)
static_assert(!long_rows(511, 4194304) && long_rows(512, 4194304) && long_rows(1, INT_MAX - 32), "");
static_assert(part_end(100, 64, 32) == 96 && part_end(100, 96, 32) == 100 && part_stages(4, 8) == 1, "");
int main(int argc, char** argv) {
    const long long m = atoll(argv[1]), n = atoll(argv[2]);
    PlanOptions o;
    o.cutoff = 128;
    o.fine = atoi(argv[3]);
    if (!atoi(argv[4])) o.split_target = 0;
    const Plan P = build_plan(m, n, o);
    if (!P.fine_tb) return printf("no fine tiles\n"), 2;
    const int ks = 4096 / (P.fine_tb * (o.fine == 1 ? 8 : 4));
    long long next = 0;
    for (int p = 0; p < P.fine_parts; ++p) {
        const long long first = (long long)p * P.fine_rows;
        if (first != next || first >= m) return printf("part %d starts at %lld\n", p, first), 1;
        const int end = part_end((int)m, (int)first, P.fine_rows);
        const long long want = first + P.fine_rows < m ? first + P.fine_rows : m;
        const long long rows = end - first;
        if (end != want || part_stages((int)rows, ks) != (rows + ks - 1) / ks)
            return printf("part %d of %d: rows %lld to %d\n", p, P.fine_parts, first, end), 1;
        next = end;
    }
    return next == m ? 0 : 1;
}
"""


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    d = tmp_path_factory.mktemp("fine_parts")
    src, exe = str(d / "parts.cpp"), str(d / "parts")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-I", os.path.join(ROOT, "include"), src,
                    os.path.join(CSRC, "ata_plan.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("m", [1025, 262144, 2**31 - 20000, 2147480000, 2**31 - 33, 2**31 - 2,
                               2**31 - 1])
@pytest.mark.parametrize("n", [1, 16, 40])
def test_parts_cover_every_row_once(check, m, n):
    for fine in (1, 2):
        for split in (0, 1):
            r = subprocess.run([check, str(m), str(n), str(fine), str(split)], capture_output=True, text=True)
            assert r.returncode == 0, (fine, split, r.stdout)
