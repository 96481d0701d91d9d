"""What the library launches, without a GPU: the host code of every source runs against recorders in the place of the HIP
runtime (tests/launch_recorder.cpp), with made-up addresses that nothing reads."""
import ctypes
import math

import pytest

from paper_2602_11562_amd import binding


class Launch(ctypes.Structure):
    _fields_ = [("kernel", ctypes.c_char_p), ("grid", ctypes.c_uint), ("block", ctypes.c_uint), ("lds", ctypes.c_ulonglong),
                ("limit", ctypes.c_int)]


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    from paper_2602_11562_amd.build import build_launch_recorder
    path = build_launch_recorder(str(tmp_path_factory.mktemp("recorder") / "liblaunches.so"))
    loaded, binding._lib = binding._lib, None
    saved, binding.LIB_PATH = binding.LIB_PATH, path
    try:
        lib = binding.load_library()      # (the same prototypes)
    finally:
        binding._lib, binding.LIB_PATH = loaded, saved
    lib.launch_record.restype = ctypes.POINTER(Launch)
    return lib


A = 0x10000   # any 16-byte aligned address
F32, BF16 = binding.LASER_F32, binding.LASER_BF16


def launches(lib, call):
    lib.launch_clear()
    assert call(lib) == 0
    return [lib.launch_record(i).contents for i in range(lib.launch_count())]


def sta(U, C, L, w, lens=A):
    return lambda lib: lib.laser_sta_forward(A, A, A, lens, U, C, L, 128, 128, w, math.sqrt(128), BF16, A, A, None)


@pytest.mark.parametrize("U,C,L,w,dealt", [(40, 300, 2500, 100, True), (64, 128, 2800, 70, True), (16, 128, 10000, 256, False)])
@pytest.mark.parametrize("spw", [1, 2, 3, 16])
def test_forced_segments_per_workgroup_launch_the_whole_division(recorder, monkeypatch, U, C, L, w, dealt, spw):
    S, waves = -(-L // w), 4 if C <= 128 else 8
    tiles = -(-C // (32 * waves))
    own, = launches(recorder, sta(U, C, L, w))
    assert (own.grid == 256) == dealt
    monkeypatch.setenv("LASER_STA_SPW", str(spw))
    forced, = launches(recorder, sta(U, C, L, w))
    print(own.kernel, own.grid, forced.kernel, forced.grid)
    assert forced.block == own.block == 64 * waves
    assert forced.grid == U * tiles * -(-S // spw)
