"""The launches whose grids grow with the requests of a group, laid out and
walked on the host."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_launch_layouts(tmp_path):
    from paper_2505_14372_amd import build_lib
    exe = tmp_path / "launch_check"
    src = os.path.join(ROOT, "tests", "host", "launch_check.cpp")
    r = subprocess.run([build_lib.hipcc(), "-std=c++17", "-O1", "-I", build_lib.CSRC, "-I", build_lib.INCLUDE,
                        src, "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
