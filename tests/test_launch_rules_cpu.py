"""The rules that choose a render's launches, run on the host (g++) with the library's own header."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_launch_rules(tmp_path):
    exe = tmp_path / "launch_rules"
    subprocess.run(["g++", "-O2", "-std=c++17", os.path.join(ROOT, "tests", "launch_rules.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "OK " in r.stdout, r.stdout + r.stderr
