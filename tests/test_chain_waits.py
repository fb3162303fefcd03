"""The chained copy's own bounded waits, in CPU builds of the library whose
limits are cut down: the door that closes before all workgroups have arrived
(those that came do the work), and a hand-over that expires (the launch ends
and ace_check reports the timeout)."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
sys.path.insert(0, os.path.join(HERE, "simt"))

RUN = r"""
import sys
sys.path.insert(0, sys.argv[1])
sys.path.insert(0, sys.argv[2])
import gen, oracle, simt_lib
oracle.build()
x = gen.by_name("text", 60_000, 41)
a = oracle.encode(x, block_size=2000, interleave=16, min_match=8, hash_len=8, max_level=0, flags=2)
assert oracle.info(a)["depth"] >= 8
arc = simt_lib.Archive(a)
for _ in range(3):
    try:
        print("whole" if arc.decode_all() == x else "WRONG", flush=True)
    except simt_lib.AceError as e:
        print("code", e.code, flush=True)
"""


def _variant(tmp, limits):
    """The CPU build with constants of the sources replaced."""
    import build as simt_build
    csrc = os.path.join(tmp, "paper_2606_24531_amd", "csrc")
    shutil.copytree(simt_build.CSRC, csrc)
    shutil.copytree(os.path.join(ROOT, "include"), os.path.join(tmp, "include"))
    for name, old, new in limits:
        path = os.path.join(csrc, name)
        with open(path) as f:
            s = f.read()
        assert s.count(old) == 1, old
        with open(path, "w") as f:
            f.write(s.replace(old, new))
    objs = []
    for src in [os.path.join(csrc, n) for n in ("kernels.hip", "host.cpp", "encoder.cpp")] + simt_build.SOURCES[-1:]:
        objs.append(os.path.join(tmp, os.path.basename(src) + ".o"))
        subprocess.check_call([simt_build.CXX, "-c", "-x", "c++"] + simt_build.FLAGS + [src, "-o", objs[-1]])
    lib = os.path.join(tmp, "libvariant.so")
    subprocess.check_call([simt_build.CXX, "-shared", "-pthread", "-o", lib] + objs)
    return lib


def _decodes(lib, resident):
    env = dict(os.environ, SIMT_LIB=lib, SIMT_RESIDENT=str(resident))
    r = subprocess.run([sys.executable, "-c", RUN, ROOT, HERE], env=env, capture_output=True, text=True, timeout=200)
    assert r.returncode == 0, r.stderr[-2000:]
    return r.stdout.split("\n")[:3]


def test_door_closes_on_those_that_came(tmp_path):
    lib = _variant(str(tmp_path), [("kernels.hip", "kDoorPolls = 512", "kDoorPolls = 0")])
    for resident in (3, 24):
        assert _decodes(lib, resident) == ["whole"] * 3, resident


def test_expired_hand_overs_end_the_launch(tmp_path):
    """The door waits for every workgroup, and no other wait polls twice: members
    give up, the launch ends, and the decode reports the timeout (or is whole,
    where none had to wait)."""
    lib = _variant(str(tmp_path), [("host.cpp", "kMaxIdlePolls = 1u << 21", "kMaxIdlePolls = 0u"),
                                   ("kernels.hip", "kDoorPolls = 512", "kDoorPolls = 1u << 30")])
    for resident in (3, 24):
        out = _decodes(lib, resident)
        assert all(o in ("whole", "code -6") for o in out), out
        assert "code -6" in out
