"""Host check of the transforms' lazy ranges over whole networks (tests/native/ntt_growth_test.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_whole_transforms_stay_within_64_bits(tmp_path):
    src = os.path.join(ROOT, "tests", "native", "ntt_growth_test.cpp")
    exe = str(tmp_path / "growth")
    subprocess.check_call(["hipcc", "-O2", "-std=c++17", src, "-o", exe], stderr=subprocess.DEVNULL)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert " 0 failures" in out.stdout
