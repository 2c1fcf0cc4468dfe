"""CPU check of how the workgroups of a launch find out which of them is done last."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_the_last_workgroup_is_found_whatever_earlier_launches_left(tmp_path):
    exe = tmp_path / "ticket_check"
    subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", os.path.join(HERE, "ticket_check.cpp"), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
