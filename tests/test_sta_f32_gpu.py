"""GPU parity at the edges of the fp32 matrix-core STA kernel, against the fp64 checker (1e-5 per vector, as everywhere
for fp32 storage)."""
import math

import numpy as np
import pytest

import oracle

from parity_util import TOL, to_device, to_host_f64, vec_rel_err

pytestmark = pytest.mark.gpu

laser = pytest.importorskip("paper_2602_11562_amd")

# C, L, d_q, d, w, lens: item tiles of 16 shared by up to four waves, candidate tiles of 16 and 32
STA_CASES = {
    "one_candidate_one_item_segments": (1, 9, 32, 64, 1, [9, 4, 0]),
    "17_candidates_two_tiles": (17, 70, 64, 64, 17, [70, 18, 17, 16]),
    "33_candidates_three_tiles": (33, 150, 128, 64, 48, [150, 49]),
    "many_users_two_candidate_tiles": (40, 90, 64, 128, 30, list(range(91))[::1] * 6),   # 32 candidates a wave
    "one_segment_longer_than_the_history": (5, 77, 32, 128, 2000, [77, 76, 1]),
}


@pytest.mark.parametrize("name", list(STA_CASES))
def test_sta_f32(name):
    import torch
    C, L, dq, d, w, lens = STA_CASES[name]
    U, gamma = len(lens), math.sqrt(dq)
    rng = np.random.default_rng(5100 + sum(map(ord, name)))
    q, k, v = (rng.normal(size=s).astype(np.float32) for s in ((U, C, dq), (U, L, dq), (U, L, d)))
    lens = np.array(lens, dtype=np.int32)
    print(f"case {name}", flush=True)
    kn, vn = k.copy(), v.copy()
    for u, n in enumerate(lens):      # padding rows may hold anything
        kn[u, n:] = np.nan
        vn[u, n:] = np.nan
    seg, cnt = laser.laser_sta_forward(to_device(q), to_device(kn), to_device(vn), to_device(lens), w, gamma)
    torch.cuda.synchronize()
    assert np.array_equal(cnt.cpu().numpy(), oracle.segment_counts(lens, L, w))
    got = to_host_f64(seg)
    for u in (range(U) if U <= 8 else [0, 1, 30, 90, 91, 200, U - 1]):
        ref = oracle.sta_forward(q[u:u + 1].astype(np.float64), k[u:u + 1].astype(np.float64),
                                 v[u:u + 1].astype(np.float64), lens[u:u + 1], w, gamma)
        ref = ref[0] if isinstance(ref, tuple) else ref
        assert vec_rel_err(got[u:u + 1], ref) <= TOL["f32"], u


@pytest.mark.parametrize("x", [np.inf, -np.inf, np.nan], ids=["inf", "-inf", "nan"])
@pytest.mark.parametrize("name", ["one_candidate_one_item_segments", "17_candidates_two_tiles", "33_candidates_three_tiles",
                                  "many_users_two_candidate_tiles"])
def test_not_finite_items_stay_in_their_segment(name, x):
    """An infinite value is an infinite sum, also in the last valid row, which stands in for the rows past it."""
    import torch
    C, L, dq, d, w, lens = STA_CASES[name]
    U, gamma = len(lens), math.sqrt(dq)
    if U > 8:
        lens = [max(n, 6) for n in lens]
    rng = np.random.default_rng(5200 + sum(map(ord, name)))
    q, k, v = (rng.normal(size=s).astype(np.float32) for s in ((U, C, dq), (U, L, dq), (U, L, d)))
    lens = np.array(lens, dtype=np.int32)
    kn, vn = k.copy(), v.copy()
    last = min(w, lens[0]) - 1            # the last valid item of the first segment: a column
    vn[0, last, 3] = x
    kn[1, lens[1] - 1] = np.nan           # the last valid item of a user: its whole segment
    print(f"case {name} {x}", flush=True)
    seg, _ = laser.laser_sta_forward(to_device(q), to_device(kn), to_device(vn), to_device(lens), w, gamma)
    torch.cuda.synchronize()
    got = to_host_f64(seg)
    bad = np.zeros(got.shape, dtype=bool)
    bad[0, :, 0, 3] = True
    bad[1, :, (lens[1] - 1) // w] = True
    assert np.array_equal(~np.isfinite(got), bad)
    assert np.array_equal(got[0, :, 0, 3], np.full(C, x), equal_nan=True)
    ref, _ = oracle.sta_forward(q[:2].astype(np.float64), k[:2].astype(np.float64), v[:2].astype(np.float64), lens[:2], w, gamma)
    assert vec_rel_err(np.where(bad[:2], 0.0, got[:2]), np.where(bad[:2], 0.0, ref)) <= TOL["f32"]


@pytest.mark.parametrize("name", ["17_candidates_two_tiles", "33_candidates_three_tiles"])
def test_generic_by_name_in_fp32(name):
    """The generic kernel stays an independent check of the matrix-core one: asked for by name it runs."""
    import torch
    C, L, dq, d, w, lens = STA_CASES[name]
    U, gamma = len(lens), math.sqrt(dq)
    rng = np.random.default_rng(5300 + sum(map(ord, name)))
    q, k, v = (rng.normal(size=s).astype(np.float32) for s in ((U, C, dq), (U, L, dq), (U, L, d)))
    lens = np.array(lens, dtype=np.int32)
    print(f"case {name}", flush=True)
    args = [to_device(x) for x in (q, k, v, lens)]
    auto, generic = (laser.laser_sta_forward(*args, w, gamma, variant=x)[0] for x in (laser.STA_AUTO, laser.STA_GENERIC))
    torch.cuda.synchronize()
    assert not torch.equal(auto, generic)          # (sums in another order)
    ref, _ = oracle.sta_forward(q, k, v, lens, w, gamma)
    for seg in (auto, generic):
        assert vec_rel_err(to_host_f64(seg), ref) <= TOL["f32"]
