"""CPU check of how many workgroups a launch is given."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_a_launch_stays_below_the_threads_that_a_grid_holds(tmp_path):
    exe = tmp_path / "launch_grid_check"
    subprocess.run(["g++", "-O2", "-std=c++17", os.path.join(HERE, "launch_grid_check.cpp"), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
