"""What the library launches, without a GPU: the host code of every source runs against recorders in the place of the HIP
runtime (tests/launch_recorder.cpp), with made-up addresses that nothing reads."""
import ctypes
import math
import re

import pytest

from paper_2602_11562_amd import binding
from test_sta_backward_mfma_gpu import SETS
from test_sta_dealt_gpu import CASES as DEALT
from test_sta_mfma_shape_gpu import CASES as SHAPES, eight_waves
from test_sta_ring_gpu import CASES as RING, THREE


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


@pytest.mark.parametrize("whole", [False, True], ids=["sta", "whole_path"])
@pytest.mark.parametrize("U,C,L,w,lens,own,dealt", DEALT)
def test_calls_with_workgroups_dealt_out(recorder, U, C, L, w, lens, own, dealt, whole):
    head, sizes, P = (A, A, A), (L, 128, 128, w, math.sqrt(128)), U * C // 2
    if own and whole:
        call = lambda lib: lib.laser_forward_ragged(*head, A, A, A, A, A, A, U, C, P, *sizes, 1, BF16, A, A, A, None)
    elif own:
        call = lambda lib: lib.laser_sta_forward_ragged(*head, A, A, U, C, P, *sizes, BF16, A, A, None)
    elif whole:
        call = lambda lib: lib.laser_forward(*head, A, A, A, A, A, U, C, *sizes, 1, BF16, A, A, A, None)
    else:
        call = sta(U, C, L, w)
    first = launches(recorder, call)[0]
    waves = 4 if C <= 128 else 8
    assert f"19sta_mfma_dma_kernelILi{waves}ELb{int(not whole)}ELb{int(dealt)}EE" in first.kernel.decode()
    assert not dealt or first.grid == 256


def sta_heads(U, C, L, dq, d, w, heads):
    return lambda lib: lib.laser_sta_forward_heads(A, A, A, A, U, C, L, dq, d, w, math.sqrt(dq / heads), heads, BF16, A, A, None, binding.STA_AUTO)


def ring(launch):
    """(d_q, d, computing waves, heads, short segments) of a launch of the kernel with a wave of its own for the fetches."""
    m = re.search(r"15sta_ring_kernelILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELb(\d)E", launch.kernel.decode())
    return m and tuple(int(x) for x in m.groups())


@pytest.mark.parametrize("U,C,L,dq,d,w,heads", RING + THREE)
def test_calls_with_a_wave_for_the_fetches(recorder, U, C, L, dq, d, w, heads):
    launch, = launches(recorder, sta_heads(U, C, L, dq, d, w, heads))
    got = ring(launch)
    assert got and got[:2] == (dq, d) and got[3:] == (heads, int(w <= 32))
    assert launch.block == 64 * (got[2] + 1) and (got[2] == 1) == (C <= 32) and (got[2] < 3 or C > 64)
    assert got[2] == 3 or (U, C, L, dq, d, w, heads) not in THREE


# (users, candidates, items, d_q, d, w, heads): computing waves, segments per workgroup. Long segments with lengths that differ, where a
# second one per workgroup cost up to half the time; widths of which a compute unit holds more, or fewer, workgroups than its LDS
# tells; candidates that fill 96 places and not 64, and the other way round; exactly one round and a little more than one
PLANS = [(23, 487, 258, 128, 128, 81, 4, 2, 1), (32, 254, 517, 128, 128, 100, 4, 3, 1), (40, 78, 1631, 128, 64, 100, 2, 3, 1),
         (9, 88, 5262, 64, 128, 17, 4, 3, 4), (34, 370, 1831, 64, 128, 55, 4, 3, 2), (64, 64, 2048, 64, 64, 128, 1, 2, 1),
         (128, 64, 1280, 64, 128, 128, 1, 2, 2)]


@pytest.mark.parametrize("U,C,L,dq,d,w,heads,waves,segs", PLANS)
def test_waves_and_segments_of_a_workgroup(recorder, U, C, L, dq, d, w, heads, waves, segs):
    launch, = launches(recorder, sta_heads(U, C, L, dq, d, w, heads))
    print(launch.kernel, launch.grid)
    assert ring(launch)[2] == waves
    assert launch.grid == U * -(-C // (32 * waves)) * -(-(-(-L // w)) // segs)


# (users, candidates, items, w) at d_q = d = 128: whether the direct-to-LDS form takes the call, on both sides of each of its lines
@pytest.mark.parametrize("U,C,L,w,direct", [
    # 2400 tiles; 30 segments; 0.58 of the places; four waves
    (16, 256, 4800, 64, True), (16, 256, 4544, 64, True), (4, 256, 2000, 64, True), (4, 256, 1920, 64, False),
    (183, 296, 2400, 200, False), (183, 300, 2400, 200, True), (16, 64, 4800, 64, False), (16, 75, 9600, 64, True),
    # w = 48; below it half a tile, eighteen workgroups a compute unit, 0.7 of the places and eight waves
    (16, 256, 4700, 47, False), (16, 256, 4800, 48, True), (76, 490, 988, 28, True), (63, 490, 988, 28, False),
    (76, 490, 612, 17, True), (76, 490, 575, 16, False), (64, 180, 1241, 17, True), (1, 180, 1241, 17, False),
    (76, 350, 988, 28, False), (200, 128, 988, 28, False)])
def test_direct_or_with_a_wave_for_the_fetches(recorder, U, C, L, w, direct):
    launch, = launches(recorder, sta(U, C, L, w))
    print(launch.kernel, launch.grid)
    assert ("sta_mfma_dma_kernel" in launch.kernel.decode()) == direct and (ring(launch) is None) == direct


def gsta(P, S, d, views, M=1):
    if views:
        return lambda lib: lib.laser_gsta_forward_multires(A, A, A, A, A, A, P, 1, S, d, 1, M, BF16, A, 1, A, A, None)
    return lambda lib: lib.laser_gsta_forward(A, A, A, A, A, A, P, 1, S, d, 1, M, BF16, A, None)


def gsta_form(lib, call):
    """Which of the three bf16 forms a call of one layer runs."""
    names = " ".join(r.kernel.decode() for r in launches(lib, call))
    forms = [f for f, kernel in (("tiled", "gsta_tiled_kernel"), ("one", "gsta_one_kernel"), ("split", "gsta_pool_kernel")) if kernel in names]
    assert len(forms) == 1, names
    return forms[0]


# pairs, segments, d: the form, on both sides of the lines
@pytest.mark.parametrize("P,S,d,form", [
    (65536, 64, 64, "tiled"), (16385, 65, 64, "tiled"), (65536, 257, 64, "tiled"), (65536, 12, 128, "tiled"), (4096, 13, 128, "tiled"),
    (4097, 13, 128, "one"), (8192, 32, 128, "one"), (8193, 32, 128, "tiled"), (11264, 32, 128, "tiled"), (11265, 32, 128, "one"),
    (8192, 33, 128, "tiled"), (8193, 33, 128, "split")])
def test_forms_of_one_layer(recorder, P, S, d, form):
    for views in (False, True):
        assert gsta_form(recorder, gsta(P, S, d, views)) == form


@pytest.mark.parametrize("name", list(SHAPES))
def test_kernels_of_the_shapes(recorder, name):
    U, C, L, dq, d, w, heads = SHAPES[name]
    launch, = launches(recorder, sta_heads(U, C, L, dq, d, w, heads))
    assert ring(launch)
    launch, = launches(recorder, lambda lib: lib.laser_sta_forward_softmax(A, A, A, A, U, C, L, dq, d, w, 1.0, heads, BF16, A, A, None, 0))
    m = re.search(r"15sta_mfma_kernelILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E", launch.kernel.decode())
    got = tuple(int(x) for x in m.groups())
    assert got[:2] == (dq, d) and got[4] == heads
    assert got[2:4] == ((8, 2) if eight_waves(U, C, L, w) else ({1: 1, 2: 2}.get(-(-C // 32), 4), 1))


@pytest.mark.parametrize("S", [1, 8, 12, 13, 32, 33, 64, 65, 128, 129, 256, 257, 1000])
@pytest.mark.parametrize("d", [64, 128])
def test_kernel_name_is_what_a_large_batch_runs(recorder, d, S):
    for C in (1, 7, 1000):
        name = recorder.laser_gsta_kernel_name(C, S, d, BF16).decode()
        assert name == f"gsta_{gsta_form(recorder, gsta(-(-12000 // C) * C, S, d, False))}_bf16", C


@pytest.mark.parametrize("P,S,d,M,views,pool", [(4097, 65, 64, 1, True, True), (65536, 229, 64, 1, True, True), (65536, 229, 64, 1, False, False),
                                                (4097, 65, 64, 2, True, False), (4096, 65, 64, 1, True, False), (65536, 64, 64, 1, True, False),
                                                (2049, 33, 128, 1, True, True), (2048, 33, 128, 1, True, False), (8192, 32, 128, 1, True, False)])
def test_maxima_from_the_pass_over_the_rows(recorder, P, S, d, M, views, pool):
    launch = launches(recorder, gsta(P, S, d, views, M))[0]
    assert bool(re.search(rf"gsta_tiled_kernelItLi{d}ELi16ELi4ELb0ELb1E", launch.kernel.decode())) == pool


def folded(U, C, heads, L, d, w, lens=A):
    return lambda lib: lib.laser_sta_folded_forward(A, A, A, A, lens, U, C, L, 128, d, w, 1.0, heads, BF16, A, A, A, A, None)


def few(launch):
    """(d_q, d, folded columns, units by ticket) of a launch of the kernel for few rows."""
    m = re.search(r"14sta_few_kernelILi(\d+)ELi(\d+)ELi(\d+)ELb(\d)E", launch.kernel.decode())
    return m and tuple(int(x) for x in m.groups())


@pytest.mark.parametrize("d,waves", [(64, 8), (128, 7)])
def test_folded_calls_have_the_same_waves_by_ticket_and_in_turn(recorder, d, waves):
    for U, dealt in ((100, 0), (8000, 1)):
        launch = launches(recorder, folded(U, 2, 1, 1000, d, 20))[-1]
        assert few(launch) == (128, 128, d, dealt)
        assert launch.block == 64 * waves and launch.lds <= 160 * 1024 and launch.grid == 256


# users, rows, items, d_q, d, w: units a wave in thousandths; by ticket past four with lengths given, past six without
@pytest.mark.parametrize("U,C,L,dq,d,w,upw", [(2048, 3, 100, 64, 64, 50, 2000), (2048, 3, 200, 64, 64, 50, 4000), (2049, 3, 200, 64, 64, 50, 4002),
                                              (2048, 3, 300, 64, 64, 50, 6000), (2049, 3, 300, 64, 64, 50, 6003),
                                              (1024, 8, 240, 128, 128, 60, 4000), (1025, 8, 240, 128, 128, 60, 4004)])
def test_units_by_ticket(recorder, U, C, L, dq, d, w, upw):
    for lens, line in ((A, 4000), (None, 6000)):
        launch, = launches(recorder, lambda lib: lib.laser_sta_forward(A, A, A, lens, U, C, L, dq, d, w, 1.0, BF16, A, A, None))
        assert few(launch) == (dq, d, 0, int(upw > line))


# rows, d_q, d, w, MB of histories from which a call goes to the matrix cores: with full lengths, with lengths (None: at no size)
LARGE = [(1, 64, 64, 9, None, None), (1, 64, 64, 10, 256, 400), (1, 64, 64, 127, 256, 400), (1, 64, 64, 128, None, None),
         (1, 128, 128, 15, None, None), (1, 128, 128, 16, 256, 1000), (1, 128, 128, 32, 256, 1000), (1, 128, 128, 33, None, None),
         (1, 128, 128, 47, None, None), (1, 128, 128, 48, 256, 600), (1, 128, 128, 63, 256, 600), (1, 128, 128, 64, None, None),
         (1, 64, 128, 23, None, None), (1, 64, 128, 24, 300, None), (1, 64, 128, 48, 300, 1000), (1, 64, 128, 64, 300, 1000),
         (1, 64, 128, 72, None, None), (1, 32, 128, 30, None, None), (1, 32, 64, 30, None, None), (1, 128, 64, 30, None, None),
         (2, 32, 64, 7, None, None), (2, 32, 64, 8, 150, 150), (2, 32, 64, 32, 150, 150), (2, 32, 64, 48, 300, 600), (2, 32, 64, 65, None, None),
         (2, 32, 64, 72, 300, 600), (2, 32, 64, 399, 300, 600), (2, 32, 64, 400, None, None), (2, 128, 64, 200, 150, 150),
         (2, 128, 64, 201, 300, 600), (2, 32, 128, 15, None, None), (2, 32, 128, 16, 300, 600), (2, 64, 128, 8, 300, 600),
         (2, 128, 128, 399, 300, 600), (2, 128, 128, 400, None, None)]


@pytest.mark.parametrize("C,dq,d,w,full,lens", LARGE)
def test_one_and_two_rows_past_the_cache(recorder, C, dq, d, w, full, lens):
    L = 2000
    user = L * (dq + d) * 2
    for given, line in ((None, full), (A, lens)):
        least = -(-(line or 3000) * 1000000 // user)
        for U, here in ((least, line is not None), (least - 1, False)):
            launch, = launches(recorder, lambda lib: lib.laser_sta_forward(A, A, A + 0x10, given, U, C, L, dq, d, w, 1.0, BF16, A, A, None))
            assert bool(few(launch)) == here, (U, launch.kernel)
            launch, = launches(recorder, lambda lib: lib.laser_sta_forward(A, A, A, given, U, C, L, dq, d, w, 1.0, BF16, A, A, None))
            assert not few(launch)      # (keys and values of one array are read once there)


@pytest.mark.parametrize("name", list(SETS))
def test_backward_calls_with_two_sets_of_tiles(recorder, name):
    U, C, L, dq, d, w, grid, lds = SETS[name]
    first = launches(recorder, lambda lib: lib.laser_sta_backward(A, A, A, A, A, U, C, L, dq, d, w, 1.0, BF16, A, A, A, A, 1 << 40, None))[0]
    print(first.kernel, first.grid, first.lds)
    assert f"19sta_bwd_mfma_kernelILi{dq}ELi{d}ELb1EE" in first.kernel.decode()
    assert (first.grid, first.lds) == (grid, lds)


@pytest.mark.parametrize("C,w,mb", [(1, 64, 400), (2, 64, 150)])
def test_packed_rows_past_the_cache_count_the_users_that_have_some(recorder, C, w, mb):
    L, dq, d = 2000, 64 if C == 1 else 128, 64
    least = -(-mb * 1000000 // (L * (dq + d) * 2))
    for U in (least, 3 * least):
        for P, here in ((least * C, True), (least * C - 1, False)):
            launch = launches(recorder, lambda lib: lib.laser_sta_forward_ragged(A, A, A + 0x10, A, A, U, C, P, L, dq, d, w, 1.0, BF16, A, A, None))[0]
            assert bool(few(launch)) == here, (U, P, launch.kernel)


@pytest.mark.parametrize("S,ahead", [(1, 1), (2, 4), (4, 4), (5, 16), (16, 16), (17, 16)])
def test_no_more_runs_in_flight_than_a_user_has(recorder, S, ahead):
    last = launches(recorder, lambda lib: lib.laser_sta_backward(A, A, A, A, A, 3, 2, 10 * S, 24, 48, 10, 1.0, F32, A, A, A, A, 1 << 40, None))[-1]
    assert f"17sta_bwd_dq_kernelILi{ahead}E" in last.kernel.decode()


def gsta_backward(U, d, S, M, dt):
    return lambda lib: lib.laser_gsta_backward(A, A, A, A, A, A, A, U, 128, S * 8, d, 8, M, dt, A, A, A, A, A, A, 1 << 40, None)


def project(d_in, dt):
    return lambda lib: lib.laser_project_q_forward_variant(A, A, 2, 3, d_in, 128, dt, A, None, binding.PROJECT_GENERIC)


def project_heads(heads, d_in, dt):
    return lambda lib: lib.laser_project_heads_forward(A, A, 3, 5, d_in, 128, heads, dt, A, None, binding.PROJECT_GENERIC)


def ffn(d_ff, dt):
    return lambda lib: lib.laser_segment_ffn_forward_variant(A, A, A, A, A, A, A, A, 2, 3, 64, 256, d_ff, 8, 1e-5, dt, A, None,
                                                             binding.FFN_GENERIC)


# A kernel's limit of dynamic LDS belongs to the process: if every call sets its own need, a second thread with a smaller one
# lowers it between another's setting and launch. Calls of one kernel with different needs past 64 KB, the largest first.
LIMITS = {
    "gsta_bwd_tile_kernel": [gsta_backward(32, d, S, M, dt) for d in (64, 128) for dt in (F32, BF16) for M, S in ((2, 120), (2, 60), (1, 140), (1, 30))],
    "gsta_bwd_kernel": [gsta_backward(2, 256, S, M, dt) for dt in (F32, BF16) for M, S in ((2, 65), (2, 45), (1, 130), (1, 90))],
    "project_generic_kernel": [project(d_in, dt) for d_in in (4096, 3072, 2304) for dt in (F32, BF16)],
    "project_heads_generic_kernel": [project_heads(heads, d_in, dt) for heads, d_in in ((8, 512), (4, 768)) for dt in (F32, BF16)],
    "segment_ffn_generic_kernel": [ffn(d_ff, dt) for d_ff in (4096, 3072, 2048) for dt in (F32, BF16)],
}


@pytest.mark.parametrize("kernel", list(LIMITS))
def test_a_kernel_has_one_lds_limit(recorder, kernel):
    seen = {}
    for call in LIMITS[kernel]:
        for r in launches(recorder, call):
            name = r.kernel.decode()
            if f"{len(kernel)}{kernel}I" in name and r.lds > 64 * 1024:
                assert r.limit >= r.lds
                seen.setdefault(name, set()).add((r.lds, r.limit))
    print({k: sorted(v) for k, v in seen.items()})
    assert any(len({lds for lds, _ in v}) > 1 for v in seen.values())      # (the calls are what they are meant to be)
    for name, v in seen.items():
        assert len({limit for _, limit in v}) == 1, name
