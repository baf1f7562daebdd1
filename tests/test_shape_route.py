"""The rules that send a solve to three launches or five passes, on the CPU:
tests/host/route_driver.cpp compiled with the library's internal header."""
import os
import subprocess

from paper_2506_04489_amd import build as BUILD

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_shape_routes(tmp_path):
    exe = str(tmp_path / "route_driver")
    cmd = [BUILD.hipcc(), "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-Wall",
           os.path.join(ROOT, "tests", "host", "route_driver.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "0 failures" in r.stdout, r.stdout + r.stderr
