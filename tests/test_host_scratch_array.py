"""The scratch arrays of a context when an allocation fails, on the host with a stand-in for the GPU runtime (a small array allocated
after a failure was taken for the piece of the first allocation, which it was not, and freed by nobody)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_growth_and_failures(tmp_path):
    exe = str(tmp_path / "scratch_array_test")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror",
                           "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                           "-I", os.path.join(ROOT, "paper_2605_07330_amd", "csrc"),
                           os.path.join(HERE, "host", "scratch_array_test.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "FAILED" not in out.stdout and out.stdout.count(": ok") == 18, out.stdout
