"""Capacity that re-bucketing gives a bucket (compiled from the library's own
header, run on the CPU)."""
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
    for (uint32_t n = 0; n < 200000u; ++n) {
        const uint32_t c = mpcd::bucket_capacity(n), most = n + mpcd::bucket_slack(n);
        // whole lines from 256 particles on; never beyond what brick_slots
        // counts on, never without room to grow by n / 8
        const bool ok = n < 256u ? c == most : (c % 32u == 0u && c <= most && most - c < 32u && c >= n + n / 8u);
        if (!ok) { std::printf("bucket_capacity(%u) = %u\n", n, c); return 1; }
    }
    std::printf("ok\n");
    return 0;
}
"""


def test_bucket_capacity(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    src, exe = tmp_path / "capacity.hip", str(tmp_path / "capacity")
    src.write_text(SOURCE)
    subprocess.run([hipcc, "-O1", "--offload-arch=gfx950", "-std=c++17",
                    "-I", os.path.join(ROOT, "paper_2212_11878_amd", "csrc"), str(src), "-o", exe],
                   check=True, capture_output=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout
