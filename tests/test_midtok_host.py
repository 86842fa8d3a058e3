"""Host-side checks of the path for tens to hundreds of tokens: its work partition, and the operand hazards of its
inline-asm MFMAs in the generated code."""
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


def _run_check(tmp_path, name):
    from paper_2305_14314_amd import binding, build
    if not os.path.exists(binding.LIB_PATH):
        build.build(verbose=False)
    exe, pkg = str(tmp_path / name), os.path.dirname(binding.LIB_PATH)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O2", "-std=c++17", "-x", "hip", "-I", CSRC,
                    os.path.join(CHECKS, name + ".cpp"), "-o", exe, "-L", pkg, "-lqlora_hip", "-Wl,-rpath," + pkg],
                   check=True, capture_output=True)
    return subprocess.run([exe], check=False, capture_output=True, text=True, timeout=300).stdout


def test_mid_plan_tiles_the_work(tmp_path):
    out = _run_check(tmp_path, "mid_plan_check")
    assert out.startswith("OK "), out
    assert int(out.split()[1]) > 3000


def test_mid_is_taken_where_it_is_faster(tmp_path):
    out = _run_check(tmp_path, "mid_choice_check")
    assert out == "OK 30\n", out


def test_mid_plans_have_kernels(tmp_path):
    out = _run_check(tmp_path, "mid_variants_check")
    assert out == "OK 18\n", out


def test_mid_mfma_operands_are_written_in_time(tmp_path):
    from paper_2305_14314_amd import build
    asm = str(tmp_path / "midtok.s")
    subprocess.run([HIPCC, *build.FLAGS, "-x", "hip", "--cuda-device-only", "-S", os.path.join(CSRC, "midtok.hip"), "-o", asm],
                   check=True, capture_output=True)
    out = subprocess.run([sys.executable, os.path.join(CHECKS, "mfma_operand_check.py"), asm], check=False, capture_output=True,
                         text=True).stdout
    assert out.startswith("OK "), out
    assert int(out.split()[1]) > 3000


def test_several_tokens_decoded_once_thresholds():
    """From which call on a forward of up to 16 tokens leaves the streaming kernel: tokens, the longer side, rank, weights, and a
    contraction long enough that the host has the second launch out in time (called one by one)."""
    import ctypes
    from paper_2305_14314_amd import binding, build
    if not os.path.exists(binding.LIB_PATH):
        build.build(verbose=False)
    f = ctypes.CDLL(binding.LIB_PATH)._ZN5qlora13mid_beats_fewEllli
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_int64] * 3 + [ctypes.c_int]
    assert not f(11, 1024, 1024, 16) and f(12, 1024, 1024, 16)
    assert f(16, 2048, 2048, 64) and f(16, 2048, 2112, 64) and not f(16, 2112, 2048, 64)
    assert f(16, 2048, 2048, 128) and not f(16, 2048, 2048, 144)
    assert f(16, 4096, 16320, 64) and not f(16, 4096, 16384, 64)     # 4 weights / 2^20 against the square of the tokens
    assert f(13, 4096, 8192, 64) and not f(12, 4096, 9216, 64)
    assert f(12, 512, 4096, 16) and not f(16, 448, 4096, 64)         # short contractions stream in less than two launches take the host
    assert f(12, 256, 4096, 80) and not f(16, 192, 4096, 128)
    assert f(12, 2752, 4096, 0) and not f(12, 2688, 4096, 0) and not f(16, 2048, 4096, 0)
