"""Row chunks of A^t B, compiled for the host: the partial sums are bounded
whatever the number of right-hand sides, and few right-hand sides still get a
workgroup for every 64 rows where rows are what there is."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include "ata_plan.h"
using namespace atalib;
int main() {
    const int64_t ms[] = {0, 1, 63, 64, 65, 1000, 131072, 262144, 10000000};
    const int64_t ns[] = {1, 64, 65, 333, 2048, 16384, 131072, 1 << 30};
    const int64_t rs[] = {1, 2, 9, 16, 17, 33, 100, 1024, 16384, 100000};
    for (int64_t m : ms)
        for (int64_t n : ns)
            for (int64_t r : rs) {
                const int64_t c = atb_chunks(m, n, r);
                // at most 2048 x 64 x 16 partial sums, rounded up to one more
                // chunk, and none where one chunk does
                const int64_t width = (n + 63) / 64 * 64 * ((r + 15) / 16 * 16);
                if (c < 1 || (m > 0 && c > (m + 63) / 64) || (c > 1 && (c - 1) * width >= 2048 * 64 * 16))
                    return printf("%lld %lld %lld: %lld\n", (long long)m, (long long)n, (long long)r, (long long)c), 1;
            }
    if (atb_chunks(20011, 333, 4) != 313 || atb_chunks(262144, 2048, 1) != 64 || atb_chunks(131072, 64, 16) != 2048)
        return printf("few right-hand sides\n"), 1;
    return 0;
}
"""


def test_partial_sums_are_bounded(tmp_path):
    src, exe = str(tmp_path / "chunks.cpp"), str(tmp_path / "chunks")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_1902_02104_amd", "csrc"), "-I",
                    os.path.join(ROOT, "include"), src, "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
