"""Archive.seek(plan="host") plans on the host whatever the sizes: the
capacity passed stays below the one with which the library plans on the
device, also where the host plan's own workspace, its copy records counted, is
the larger."""
import ctypes as C

import numpy as np
import pytest

import gen

torch = pytest.importorskip("torch")


def _levels_archive(orc):
    """Levels whose blocks are too many for device-planned records together,
    few enough for a host plan of a part of them."""
    x = gen.by_name("text", 2120 * 24, 17)
    a = orc.encode(x, block_size=24, interleave=4, min_match=6, hash_len=6, max_level=3, flags=2)
    assert orc.info(a)["depth"] == 3 and orc.info(a)["n_blocks"] > 2048
    return x, a


class _Recorder:
    """The library with ace_seek replaced by a record of its capacity."""

    def __init__(self, real):
        self.real, self.caps = real, []

    def __getattr__(self, name):
        return getattr(self.real, name)

    def ace_seek(self, h, lo, hi, out, ws, cap, tuning, stream):
        self.caps.append(cap)
        return 0


def test_host_plan_stays_below_the_device_planners_size(orc, monkeypatch):
    from paper_2606_24531_amd import aceseek
    x, a = _levels_archive(orc)
    host = np.frombuffer(a, dtype=np.uint8)
    rec = _Recorder(aceseek.lib())
    h = C.c_void_p()
    assert rec.ace_archive_open(host.ctypes.data_as(C.c_void_p), len(a), None, C.byref(h)) == 0
    monkeypatch.setattr(aceseek, "lib", lambda: rec)
    monkeypatch.setattr(aceseek, "_stream_ptr", lambda s: None)
    arc = object.__new__(aceseek.Archive)
    arc._torch, arc._h, arc._ws, arc.device, arc.d_plan = torch, h, None, torch.device("cpu"), torch.zeros(1)
    dev = arc.seek_device_bytes()
    ranges = [(24 * k, len(x)) for k in range(0, 2000, 100)]
    host_need = [arc.workspace_bytes(list(r)) for r in ranges]
    assert any(n >= dev for n in host_need)
    ws = torch.zeros(max(host_need + [dev]), dtype=torch.uint8)
    for r in ranges:
        arc.seek(*r, ws=ws, plan="host")
        assert rec.caps[-1] < dev, r
    for r in ranges:
        arc.seek(*r, ws=ws, plan="device")
        assert rec.caps[-1] >= dev, r


@pytest.mark.gpu
def test_host_planned_seek_of_the_same_archive(orc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_24531_amd import Archive
    x, a = _levels_archive(orc)
    arc = Archive(a, device="cuda:0")
    for k in (0, 300, 700, 1200):
        got = arc.seek(24 * k, len(x), plan="host")
        arc.check()
        assert got.cpu().numpy().tobytes() == x[24 * k:], k
