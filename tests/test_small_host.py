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


def test_small_jobs_of_a_shared_launch_are_split():
    """A product of few tiles keeps workgroups of its own beside one of many, never more than in a launch of its own (the
    partials' buffer is sized for that), and a split is never empty of K-steps."""
    import ctypes
    from paper_2305_14314_amd import binding, build
    if not os.path.exists(binding.LIB_PATH):
        build.build(verbose=False)
    f = getattr(ctypes.CDLL(binding.LIB_PATH), "_ZN5qlora16small_job_splitsEiiiii")
    assert f(128, 64, 4096, 512, 256) == 64 and f(16384, 128, 4096, 2, 256) == 1       # dL2 beside dL1 of 16384 x 64, rank 128
    for I, J, K, other in [(64, 64, 4096, 1023), (1024, 64, 640, 80), (256, 1024, 4096, 256), (64, 22016, 1000, 128), (16, 64, 65, 9)]:
        own = ((I + 63) // 64) * ((J + 63) // 64)
        alone, shared, floored = f(I, J, K, 0, 0), f(I, J, K, other, 0), f(I, J, K, other, 256)
        assert 1 <= shared <= floored <= alone <= min(64, (K + 63) // 64)
        assert floored * own >= min(256, alone * own)
