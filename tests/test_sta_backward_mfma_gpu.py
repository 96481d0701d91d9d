"""GPU parity of STA's backward pass on the matrix cores (more than four candidates, bf16) at the edges of its tiles and
of its split into workgroups, against the fp64 checker. Both products with fp32 factors (the gates, the score gradients)
carry 24 bits, so the bounds are those of an fp32 sum: 1e-5, dk per user as in test_sta_backward_gpu.py (a row of dk
is a sum of signed terms that may cancel)."""
import math

import numpy as np
import pytest

import oracle

from parity_util import to_device, to_host_f64, vec_rel_err
from test_sta_backward_gpu import BWD_TOL, _store

pytestmark = pytest.mark.gpu

laser = pytest.importorskip("paper_2602_11562_amd")

# C, L, d_q, d, w, lens
CASES = {
    "five_candidates_one_item_tile": (5, 96, 32, 64, 32, [96, 33, 32, 31, 1, 0]),     # tile edges of the valid length
    "33_candidates_segments_of_one_item": (33, 12, 64, 64, 1, [12, 5]),
    "64_candidates_short_segments": (64, 130, 128, 64, 10, [130, 101]),              # four segments per workgroup
    "65_candidates_two_tiles_a_segment": (65, 200, 64, 128, 33, [200, 34]),          # 33 items: a tile of one row
    "130_candidates_long_segment": (130, 700, 128, 128, 300, [700, 301, 257]),       # several item blocks per segment
    "one_long_segment": (9, 260, 32, 128, 1000, [260, 129]),                         # w > L
}


@pytest.mark.parametrize("name", list(CASES))
def test_sta_backward_on_the_matrix_cores(name):
    import torch
    C, L, dq, d, w, lens = CASES[name]
    U, S = len(lens), -(-L // w)
    rng = np.random.default_rng(4100 + sum(map(ord, name)))
    (qs, qv), (ks, kv), (vs, vv), (gs, gv) = (_store(rng.normal(size=s), "bf16")
                                              for s in ((U, C, dq), (U, L, dq), (U, L, d), (U, C, S, d)))
    lens = np.array(lens, dtype=np.int32)
    for u, n in enumerate(lens):      # padding rows may hold anything
        ks[u, n:] = 0x7fc0
        vs[u, n:] = 0x7fc0
    gamma = math.sqrt(dq)
    print(f"case {name}", flush=True)
    ref = oracle.sta_backward(qv, kv, vv, lens, w, gamma, gv)
    args = (to_device(qs), to_device(ks), to_device(vs), to_device(lens), to_device(gs), w, gamma)
    got = laser.laser_sta_backward(*args)
    torch.cuda.synchronize()
    for nm, a, b in zip(("dq", "dk", "dv"), got, ref):
        a = to_host_f64(a)
        assert np.isfinite(a).all() and not a[b == 0].any()
        if nm == "dk":
            a, b = a.reshape(U, -1), b.reshape(U, -1)
        err = vec_rel_err(a, b)
        print(f"  {nm}: max relative error {err:.3e}", flush=True)
        assert err <= BWD_TOL, nm
    again = laser.laser_sta_backward(*args)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(got, again))      # fixed summation order


@pytest.mark.parametrize("C,w", [(5, 5), (8, 3), (9, 2), (8, 4)])   # either side of the line: nearly empty tiles
def test_many_short_segments(C, w):
    import torch
    L, dq, d, U = 60, 64, 64, 6144 * w // 60 + 1
    S = -(-L // w)
    rng = np.random.default_rng(4300 + C + w)
    (qs, qv), (ks, kv), (vs, vv), (gs, gv) = (_store(rng.normal(size=s), "bf16")
                                              for s in ((U, C, dq), (U, L, dq), (U, L, d), (U, C, S, d)))
    lens = rng.integers(0, L + 1, U).astype(np.int32)
    gamma = math.sqrt(dq)
    print(f"C {C} w {w} users {U}", flush=True)
    got = laser.laser_sta_backward(*(to_device(x) for x in (qs, ks, vs, lens, gs)), w, gamma)
    torch.cuda.synchronize()
    pick = [0, 1, 2, U // 2, U - 1]
    ref = oracle.sta_backward(qv[pick], kv[pick], vv[pick], lens[pick], w, gamma, gv[pick])
    for nm, a, b in zip(("dq", "dk", "dv"), got, ref):
        a = to_host_f64(a)[pick]
        if nm == "dk":
            a, b = a.reshape(len(pick), -1), b.reshape(len(pick), -1)
        assert vec_rel_err(a, b) <= BWD_TOL, nm


# The form with two sets of tiles on both sides. Users, C, L, d_q, d, w, workgroups and LDS of the launch (shown by
# test_launches_cpu.py): workgroups = users x (runs of segments x blocks of four candidate tiles + blocks of segments x blocks of item
# tiles). With 130 users a run is four of 13 segments: two steps of two segments with 33 to 64 candidates, four of one past them; 80 KB
# is the most that a call asks for
SETS = {
    "two_segments_in_work_64_64": (130, 40, 128, 64, 64, 10, 130 * 4 + 130 * 4, 40960),
    "two_segments_in_work_64_128": (130, 64, 121, 64, 128, 10, 130 * 4 + 130 * 4, 73728),
    "two_segments_in_work_128_128": (130, 33, 130, 128, 128, 10, 130 * 4 + 130 * 4, 81920),
    "two_tiles_a_segment_32_64": (130, 50, 500, 32, 64, 40, 130 * 4 + 130 * 7, 24576),
    "three_candidate_blocks_128_128": (130, 75, 400, 128, 128, 31, 130 * 4 + 130 * 4, 81920),
    "four_candidate_blocks_64_64": (17, 128, 200, 64, 64, 20, 17 * 10 + 17 * 3, 40960),
}


@pytest.mark.parametrize("name", list(SETS))
def test_two_sets_of_tiles(name):
    """Several steps of a workgroup on either side: every second block comes from the other set, and a step to the next segments
    takes their dH'. Lengths end inside tiles, runs and segments; what lies past them may hold anything."""
    import torch
    U, C, L, dq, d, w = SETS[name][:6]
    S = -(-L // w)
    rng = np.random.default_rng(4400 + sum(map(ord, name)))
    (qs, qv), (ks, kv), (vs, vv), (gs, gv) = (_store(rng.normal(size=s), "bf16")
                                              for s in ((U, C, dq), (U, L, dq), (U, L, d), (U, C, S, d)))
    lens = rng.integers(0, L + 1, U).astype(np.int32)
    lens[:4] = L, 4 * w + 1, 0, L - 1
    for u, n in enumerate(lens):
        ks[u, n:] = 0x7fc0
        vs[u, n:] = 0x7fc0
    gamma = math.sqrt(dq)
    print(f"case {name}", flush=True)
    args = (to_device(qs), to_device(ks), to_device(vs), to_device(lens), to_device(gs), w, gamma)
    got = laser.laser_sta_backward(*args)
    again = laser.laser_sta_backward(*args)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(got, again))
    pick = [0, 1, 2, 3, U // 2, U - 2, U - 1]
    ref = oracle.sta_backward(qv[pick], kv[pick], vv[pick], lens[pick], w, gamma, gv[pick])
    for nm, a, b in zip(("dq", "dk", "dv"), got, ref):
        a = to_host_f64(a)
        assert np.isfinite(a).all(), nm
        a = a[pick]
        assert not a[b == 0].any(), nm
        if nm == "dk":
            a, b = a.reshape(len(pick), -1), b.reshape(len(pick), -1)
        err = vec_rel_err(a, b)
        print(f"  {nm}: max relative error {err:.3e}", flush=True)
        assert err <= BWD_TOL, nm


def _classes(x):
    return np.where(np.isnan(x), 2, np.where(np.isposinf(x), 1, np.where(np.isneginf(x), -1, 0)))


# which input, its value, and where: candidates and items that share their tile with padding
@pytest.mark.parametrize("what", ["k", "v", "dh"])
@pytest.mark.parametrize("bits", [0x7f80, 0xff80, 0x7fc0], ids=["inf", "-inf", "nan"])
@pytest.mark.parametrize("name", ["five_candidates_one_item_tile", "33_candidates_segments_of_one_item",
                                  "64_candidates_short_segments", "65_candidates_two_tiles_a_segment", "one_long_segment"])
def test_not_finite_values_as_in_the_plain_sums(name, bits, what):
    """Infinities and NaN give the gradients that the sums over the valid items and the present candidates give: padding of
    the tiles takes no part."""
    import torch
    C, L, dq, d, w, lens = CASES[name]
    U, S = len(lens), -(-L // w)
    rng = np.random.default_rng(4200 + sum(map(ord, name)))
    (qs, qv), (ks, kv), (vs, vv), (gs, gv) = (_store(rng.normal(size=s), "bf16")
                                              for s in ((U, C, dq), (U, L, dq), (U, L, d), (U, C, S, d)))
    lens = np.array(lens, dtype=np.int32)
    x = {0x7f80: np.inf, 0xff80: -np.inf, 0x7fc0: np.nan}[bits]
    at = {"k": (ks, kv, (0, lens[0] - 1, 3)), "v": (vs, vv, (0, lens[0] - 1, 3)), "dh": (gs, gv, (1, C - 1, (lens[1] - 1) // w, 5))}
    stored, value, index = at[what]
    stored[index], value[index] = bits, x
    gamma = math.sqrt(dq)
    print(f"case {name} {what} {x}", flush=True)
    with np.errstate(invalid="ignore", over="ignore"):
        ref = oracle.sta_backward(qv, kv, vv, lens, w, gamma, gv)
    got = laser.laser_sta_backward(to_device(qs), to_device(ks), to_device(vs), to_device(lens), to_device(gs), w, gamma)
    torch.cuda.synchronize()
    for nm, a, b in zip(("dq", "dk", "dv"), got, ref):
        a = to_host_f64(a)
        assert np.array_equal(_classes(a), _classes(b)), nm
        a, b = np.where(np.isfinite(b), a, 0.0), np.where(np.isfinite(b), b, 0.0)
        if nm == "dk":
            a, b = a.reshape(U, -1), b.reshape(U, -1)
        assert vec_rel_err(a, b) <= BWD_TOL, nm
