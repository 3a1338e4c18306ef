"""Host-side check of the register-plane kernel's program blocks
(RunCompiler::encode_program) against the segments they are packed from
(rp_block_check.cpp).  No GPU needed."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def test_program_blocks_match_segments(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "rp_block_check")
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-o", exe,
                    os.path.join(HERE, "rp_block_check.cpp"),
                    os.path.join(ROOT, "paper_2105_01533_amd", "csrc", "run_compiler.hip")],
                   check=True, capture_output=True)
    r = subprocess.run([exe, "500"], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("OK"), r.stdout + r.stderr
