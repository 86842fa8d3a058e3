"""Host-side checks of the skinny adapter products: their generated loops and how a contraction is split."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2305_14314_amd", "csrc")
CHECKS = os.path.join(ROOT, "tests", "host_checks")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

pytestmark = pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which(HIPCC)), reason="hipcc not available")


def test_loops_reload_nothing(tmp_path):
    from paper_2305_14314_amd import build
    asm = str(tmp_path / "small.s")
    subprocess.run([HIPCC, *build.FLAGS, "-x", "hip", "--cuda-device-only", "-S", os.path.join(CSRC, "small.hip"), "-o", asm],
                   check=True, capture_output=True)
    out = subprocess.run([sys.executable, os.path.join(CHECKS, "small_loop_check.py"), asm], check=False, capture_output=True,
                         text=True).stdout
    assert out.startswith("OK "), out
    assert int(out.split()[1]) >= 12
