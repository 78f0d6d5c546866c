"""The register-held 2D transform of the chain kernels, emulated thread by
thread on the host: exchange addresses, LDS banks and the transform itself."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_register_tile_transform_emulation(tmp_path):
    from paper_2505_14372_amd import build_lib
    exe = tmp_path / "chain_check"
    src = os.path.join(ROOT, "tests", "host", "chain_check.cpp")
    r = subprocess.run([build_lib.hipcc(), "-std=c++17", "-O1", "-I", build_lib.CSRC, "-I", build_lib.INCLUDE,
                        src, "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    print(r.stdout)
    assert r.returncode == 0, r.stdout
