"""The rule that gives one graph column order by default, compiled from the
library's own header with the host compiler."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_column_rule(tmp_path):
    exe = tmp_path / "columns_check"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror",
                           "-I", os.path.join(ROOT, "paper_2508_16522_amd", "csrc"),
                           os.path.join(ROOT, "tests", "native", "columns_check.cpp"), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "all cases pass" in r.stdout
