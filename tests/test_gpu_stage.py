"""State transfers when pinned host memory is refused (C client)."""
import os
import subprocess

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_states_pass_without_pinned_memory(tmp_path):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_11878_amd import mpcd
    exe, libdir = str(tmp_path / "c_stage_client"), os.path.dirname(mpcd.LIB_PATH)
    rocm = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "lib")
    subprocess.run(["gcc", "-std=c99", "-O1", "-Wall", "-Werror", "-rdynamic", "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "c_stage_client.c"), "-L", libdir, "-lmpcd", "-L", rocm,
                    "-lamdhip64", "-Wl,-rpath," + libdir, "-Wl,-rpath," + rocm, "-ldl", "-o", exe], check=True)
    print("[case] c stage client", flush=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout.strip() == "ok", (out.returncode, out.stdout, out.stderr)
