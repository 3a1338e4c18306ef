"""Host-side check of whole register-plane programs (RunCompiler::program), cut
into parts, and of the bound on their blocks (rp_run_check.cpp).  No GPU needed."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def test_programs_in_parts(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "rp_run_check")
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-o", exe,
                    os.path.join(HERE, "rp_run_check.cpp"),
                    os.path.join(ROOT, "paper_2105_01533_amd", "csrc", "run_compiler.hip")],
                   check=True, capture_output=True)
    r = subprocess.run([exe, "2000"], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("OK"), r.stdout + r.stderr
