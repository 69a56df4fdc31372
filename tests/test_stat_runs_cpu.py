"""Runs of tiles that the reduction of a box's partial sums folds (compiled from
the library's own header, run on the CPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include "mpcd_dev.h"
int main()
{
    for (int n = 2; n < 300000; ++n) {
        const mpcd::StatRuns r = mpcd::stat_runs(n);
        // every tile in one run, at most 256 runs; a run's record (kNumDiag
        // 128-bit sums) lies inside its own tiles' records (kNumDiag 64-bit)
        bool ok = r.groups >= 1 && r.groups <= mpcd::kBlock && r.begin(0) == 0 && r.end(r.groups - 1) == n;
        for (int g = 0; g < r.groups; ++g) {
            ok = ok && r.begin(g) == g * r.per && r.end(g) - r.begin(g) >= 2;
            ok = ok && (g + 1 == r.groups || r.end(g) == r.begin(g + 1));
        }
        if (!ok) { std::printf("stat_runs(%d): %d runs of %d\n", n, r.groups, r.per); return 1; }
    }
    std::printf("ok\n");
    return 0;
}
"""


def test_every_run_holds_its_record(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    src, exe = tmp_path / "runs.hip", str(tmp_path / "runs")
    src.write_text(SOURCE)
    subprocess.run([hipcc, "-O1", "--offload-arch=gfx950", "-std=c++17",
                    "-I", os.path.join(ROOT, "paper_2212_11878_amd", "csrc"), str(src), "-o", exe],
                   check=True, capture_output=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout
