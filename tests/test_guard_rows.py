"""CPU check of the row kernels' test for rows that lie outside their allocation with every byte."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_rows_outside_the_binding(tmp_path):
    exe = tmp_path / "guard_rows_check"
    subprocess.run(["g++", "-O2", "-std=c++17", os.path.join(HERE, "guard_rows_check.cpp"), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
