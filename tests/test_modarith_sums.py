"""Host check of the lazy modular reductions (tests/native/modarith_sums_test.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_lazy_reductions_host_exact(tmp_path):
    src = os.path.join(ROOT, "tests", "native", "modarith_sums_test.cpp")
    exe = str(tmp_path / "mas")
    subprocess.check_call(["hipcc", "-O2", "-std=c++17", src, "-o", exe], stderr=subprocess.DEVNULL)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert " 0 failures" in out.stdout
