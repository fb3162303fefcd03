"""The encoder when allocations fail at any point of a call
(tests/simt/encode_fail_check.cpp, built with the encoder's own source)."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.join(HERE, "simt"))


def test_failed_allocations_end_the_call_only(tmp_path):
    import build as simt_build
    lib = simt_build.build()
    exe = str(tmp_path / "encode_fail_check")
    subprocess.check_call([simt_build.CXX, "-x", "c++", "-std=c++17", "-O1", "-g", "-pthread", "-w",
                           "-I", os.path.join(HERE, "simt"), os.path.join(HERE, "simt", "encode_fail_check.cpp"),
                           "-x", "none", lib, "-Wl,-rpath," + os.path.dirname(lib), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=240)
    print(r.stdout[-3000:], r.stderr[-2000:])
    assert r.returncode == 0
