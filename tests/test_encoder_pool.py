"""The encoder's thread pool when a loop's body throws or threads cannot be
started (tests/simt/pool_check.cpp, built with the encoder's own source)."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.join(HERE, "simt"))


def test_pool_outlives_failures(tmp_path):
    import build as simt_build
    lib = simt_build.build()
    exe = str(tmp_path / "pool_check")
    subprocess.check_call([simt_build.CXX, "-x", "c++", "-std=c++17", "-O1", "-g", "-pthread",
                           "-I", os.path.join(HERE, "simt"), os.path.join(HERE, "simt", "pool_check.cpp"),
                           "-x", "none", lib, "-Wl,-rpath," + os.path.dirname(lib), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    print(r.stdout, r.stderr)
    assert r.returncode == 0
