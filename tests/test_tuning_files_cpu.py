"""Tuning files of both versions: saved as they were loaded, and refused where malformed."""
import ctypes

import pytest

from paper_2012_08655_amd import _native as N

V3 = ["fov-tune-v3 gfx950 256 0 0 3 32 6 11 0 : 2 32 1 0 0 87.500", "fov-tune-v3 gfx950 256 1 1 1 16 4 8 1 : 1 64 0 1 1 12.000"]
V4 = ["fov-tune-v4 gfx950 256 0 0 3 32 6 11 0 32 : 2 64 0 0 0 41.000", "fov-tune-v4 gfx950 256 0 0 3 64 6 13 0 33 : 1 64 0 -1 -1 40.125",
      "fov-tune-v4 gfx950 256 1 1 3 32 6 11 0 0 : 1 64 0 1 1 43.500"]


def load(tmp_path, lines):
    f = tmp_path / "in.txt"
    f.write_text("\n".join(["# comment", *lines, ""]))
    return N.lib().foveate_tuning_load(str(f).encode())


def test_round_trip(tmp_path):
    N.lib().foveate_tuning_clear()
    try:
        assert load(tmp_path, V3 + V4) == N.FOV_OK
        n = ctypes.c_int32()
        assert N.lib().foveate_tuning_count(ctypes.byref(n)) == N.FOV_OK and n.value == 5
        out = tmp_path / "out.txt"
        assert N.lib().foveate_tuning_save(str(out).encode()) == N.FOV_OK
        assert sorted(l for l in out.read_text().splitlines() if l[0] != "#") == sorted(V3 + V4)
    finally:
        N.lib().foveate_tuning_clear()


@pytest.mark.parametrize("bad", [V4[0].replace("v4", "v3"), V3[0].replace("v3", "v4"), V4[0].replace(" 32 :", " 33 :"), V4[0].replace(" 32 :", " -1 :"),
                                 V4[1].replace("-1 -1", "-2 -1"), V4[1].replace("-1 -1", "-1 2"), V3[0].replace("0 0 87", "-1 0 87"), V4[0] + " x",
                                 V4[0].replace(": 2", ": 3"), V4[2].replace(": 1", ": 2")])
def test_refused(tmp_path, bad):
    assert load(tmp_path, [bad]) == N.FOV_EINVAL
    assert b":2:" in N.lib().foveate_last_error()
