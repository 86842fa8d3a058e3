"""Host check of the exact mean of the first-level constants: the 128-bit form the encode kernel takes for ordinary weights
against the general one, bit for bit."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(not shutil.which("g++"), reason="g++ not available")
def test_mean_forms_agree(tmp_path):
    exe = str(tmp_path / "dq_mean_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2305_14314_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host_checks", "dq_mean_check.cpp"), "-o", exe], check=True, capture_output=True)
    out = subprocess.run([exe], check=False, capture_output=True, text=True, timeout=120).stdout
    assert out.startswith("ok "), out
    assert int(out.split()[1]) > 300000                        # of 400000 cases, those of at most 60 binades
