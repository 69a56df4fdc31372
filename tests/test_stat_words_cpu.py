"""128-bit sums kept over the 64-bit partials of a run of tiles (compiled from the
library's own header, run on the CPU with the alignment check on)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include <vector>
#include "mpcd_dev.h"
int main()
{
    using namespace mpcd;
    for (int ntile = 1025; ntile < 1400; ++ntile) {   // runs of 5 and 6 tiles
        const StatRuns r = stat_runs(ntile);
        std::vector<long long> words((size_t)ntile * kNumDiag + 2, 77);
        for (int off = 0; off < 2; ++off) {           // partials on 16 bytes, and 8 beyond
            long long* const p = words.data() + off;
            auto value = [&](int g, int j) {
                const __int128 v = ((__int128)(g * 1000003ll + j) << 61) + g * 7919ll + j;
                return (g + j) % 2 ? -v : v;
            };
            for (int g = 0; g < r.groups; ++g)
                for (int j = 0; j < kNumDiag; ++j) stat_put(p + (size_t)r.begin(g) * kNumDiag + 2 * j, value(g, j));
            for (int g = 0; g < r.groups; ++g)
                for (int j = 0; j < kNumDiag; ++j)
                    if (stat_get(p + (size_t)r.begin(g) * kNumDiag + 2 * j) != value(g, j)) {
                        std::printf("%d tiles, run %d, sum %d\n", ntile, g, j);
                        return 1;
                    }
        }
    }
    std::printf("ok\n");
    return 0;
}
"""


def test_sums_need_no_alignment_of_their_own(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    src, exe = tmp_path / "words.hip", str(tmp_path / "words")
    src.write_text(SOURCE)
    subprocess.run([hipcc, "-O0", "--offload-arch=gfx950", "-std=c++17", "-Xarch_host", "-fsanitize=alignment",
                    "-Xarch_host", "-fsanitize-trap=alignment",
                    "-I", os.path.join(ROOT, "paper_2212_11878_amd", "csrc"), str(src), "-o", exe],
                   check=True, capture_output=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.strip() == "ok", (out.returncode, out.stdout)
