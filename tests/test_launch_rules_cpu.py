"""The rules that choose a render's launches, run on the host (g++) with the library's own header."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_launch_rules(tmp_path):
    exe = tmp_path / "launch_rules"
    subprocess.run(["g++", "-O2", "-std=c++17", os.path.join(ROOT, "tests", "launch_rules.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "OK " in r.stdout, r.stdout + r.stderr


def test_traversal_left_free(tmp_path):
    """The build's occupancy setting at its "left free" value divides by nothing."""
    src = os.path.join(ROOT, "paper_1702_01530_amd", "csrc", "render.hip")
    cmd = ["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "--cuda-host-only", "-fsyntax-only", "-std=c++17", "-O1",
           "-DSRT_TRACE_WAVES_PER_EU=0", "-Werror=division-by-zero", src]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
