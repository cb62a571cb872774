"""The clustering builder's launches, planned on the host (g++, with the builder's own header): rounds that merge slower
than usual keep a workgroup for every tile they find."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_rounds_keep_their_workgroups(tmp_path):
    exe = tmp_path / "cluster_plan"
    subprocess.run(["g++", "-O2", "-std=c++17", os.path.join(ROOT, "tests", "cluster_plan.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.count("OK ") == 60, r.stdout + r.stderr
