"""GPU parity at the edges of the matrix-core STA kernel for a few query rows per user and of its folded form, against the
fp64 checker (2e-2 per vector, as everywhere for bf16 storage), and: an item that is not finite stays in its segment."""
import math

import numpy as np
import pytest

import oracle
import workloads

from parity_util import TOL, to_device, to_host_f64, vec_rel_err

pytestmark = pytest.mark.gpu

laser = pytest.importorskip("paper_2602_11562_amd")

# C, L, d_q, d, w, lens: tiles of 32 items, blocks of 16 / 2^k segments, runs of about 64 items
CASES = {
    "one_item_segments": (3, 70, 32, 64, 1, [70, 0, 33, 1]),
    "two_rows": (2, 100, 64, 64, 7, [100, 99, 8]),
    "block_ends_inside_tiles": (8, 333, 128, 128, 10, [333, 331, 20, 19]),
    "segment_ends_with_the_tile": (5, 256, 64, 128, 32, [256, 255, 33, 32]),
    "short_last_segment": (7, 129, 128, 64, 64, [129, 128, 65]),
    "one_segment_longer_than_the_history": (4, 77, 32, 128, 2000, [77, 76, 1]),
    "more_units_than_waves": (4, 40, 64, 64, 4, [(7 * i) % 41 for i in range(700)]),
    # (one to six rows in calls too small to fill the machine run on the vector-ALU kernels; the same edges in larger ones)
    "one_item_segments_of_many_users": (3, 70, 32, 64, 1, [70, 0, 33, 1, 70, 69] * 50),
    "two_rows_of_many_users": (2, 100, 64, 64, 7, [100, 99, 8, 0] * 170),
    "three_wide_rows_of_many_users": (3, 130, 128, 128, 9, [130, 129, 28, 9] * 130),
    "long_segments_of_many_users": (4, 133, 32, 128, 131, [133, 132, 131, 1] * 130),
    "two_rows_long_segments": (2, 134, 64, 64, 2000, [134, 33, 1, 0] * 1030),
}


def _bf16(x):
    bits = workloads.f32_to_bf16_bits(np.asarray(x, dtype=np.float32))
    return bits, workloads.bf16_bits_to_f32(bits).astype(np.float64)


def _inputs(name):
    C, L, dq, d, w, lens = CASES[name]
    rng = np.random.default_rng(6200 + sum(map(ord, name)))
    U = len(lens)
    return [_bf16(rng.normal(size=s)) for s in ((U, C, dq), (U, L, dq), (U, L, d))], np.array(lens, dtype=np.int32), w, math.sqrt(dq)


@pytest.mark.parametrize("name", list(CASES))
def test_sta_few(name):
    import torch
    (q, k, v), lens, w, gamma = _inputs(name)
    U, L = k[0].shape[:2]
    print(f"case {name}", flush=True)
    kn, vn = k[0].copy(), v[0].copy()
    for u, n in enumerate(lens):      # padding rows may hold anything
        kn[u, n:] = 0x7fc0
        vn[u, n:] = 0x7fc0
    seg, cnt = laser.laser_sta_forward(to_device(q[0]), to_device(kn), to_device(vn), to_device(lens), w, gamma)
    torch.cuda.synchronize()
    assert np.array_equal(cnt.cpu().numpy(), oracle.segment_counts(lens, L, w))
    got = to_host_f64(seg)
    for u in (range(U) if U <= 8 else [0, 1, 2, 3, 5, 6, 40, 41, U // 2, U - 1]):
        ref, _ = oracle.sta_forward(q[1][u:u + 1], k[1][u:u + 1], v[1][u:u + 1], lens[u:u + 1], w, gamma)
        assert vec_rel_err(got[u:u + 1], ref) <= TOL["bf16"], u


@pytest.mark.parametrize("name", ["two_rows", "block_ends_inside_tiles", "short_last_segment", "two_rows_of_many_users"])
@pytest.mark.parametrize("bits", [0x7f80, 0xff80, 0x7fc0], ids=["inf", "-inf", "nan"])
def test_not_finite_items_stay_in_their_segment(name, bits):
    import torch
    (q, k, v), lens, w, gamma = _inputs(name)
    kn, vn = k[0].copy(), v[0].copy()
    vn[0, 5, 3] = bits                # segment 5 // w of the first user, one column
    kn[1, 2 * w % lens[1]] = 0x7fc0   # a whole segment of the second
    seg, _ = laser.laser_sta_forward(to_device(q[0]), to_device(kn), to_device(vn), to_device(lens), w, gamma)
    torch.cuda.synchronize()
    got = to_host_f64(seg)
    got, lens = got[:8], lens[:8]
    ref, _ = oracle.sta_forward(q[1][:8], k[1][:8], v[1][:8], lens, w, gamma)
    bad = np.zeros(ref.shape, dtype=bool)
    bad[0, :, 5 // w, 3] = True
    bad[1, :, (2 * w % lens[1]) // w] = True
    assert np.array_equal(~np.isfinite(got), bad)
    assert np.isnan(got[bad]).all() == (bits == 0x7fc0)
    assert vec_rel_err(np.where(bad, 0.0, got), np.where(bad, 0.0, ref)) <= TOL["bf16"]


def test_packed_rows_keep_to_their_user():
    import torch
    (q, k, v), lens, w, gamma = _inputs("block_ends_inside_tiles")
    counts = [3, 0, 8, 1]
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    qp = np.concatenate([q[0][u, :c] for u, c in enumerate(counts)])
    seg, cnt, _ = laser.laser_forward_ragged(to_device(qp), to_device(k[0]), to_device(v[0]), None, None, None, None,
                                             to_device(lens), to_device(off), 8, w, gamma, stage="sta")
    dense, cnt_d = laser.laser_sta_forward(to_device(q[0]), to_device(k[0]), to_device(v[0]), to_device(lens), w, gamma)
    torch.cuda.synchronize()
    assert torch.equal(cnt, cnt_d)
    assert torch.equal(seg, torch.cat([dense[u, :c] for u, c in enumerate(counts)]))


# C, heads, d, L, w, lens
FOLDED = {
    "two_heads": (1, 2, 128, 129, 10, [129, 128, 33, 0]),
    "four_heads": (1, 4, 128, 100, 3, [100, 1]),
    "two_candidates_two_heads": (2, 2, 64, 200, 33, [200, 66, 67]),
    "three_candidates": (3, 1, 128, 65, 64, [65, 64]),
    "one_row": (1, 1, 64, 50, 50, [50, 0]),
    # three launches: more rows than the ring holds; one and two rows, long segments and few of them
    "five_rows": (5, 1, 128, 130, 10, [130, 101]),
    "eight_rows": (4, 2, 64, 200, 64, [200, 65, 64]),
    "one_row_long_segments": (1, 1, 128, 300, 140, [300, 141, 0]),
    "two_rows_long_segments": (1, 2, 128, 300, 260, [300, 259]),
}


@pytest.mark.parametrize("name", list(FOLDED))
def test_folded(name):
    import torch
    C, heads, d, L, w, lens = FOLDED[name]
    U, din, dq = len(lens), 128, 64
    rng = np.random.default_rng(6300 + sum(map(ord, name)))
    t, h = _bf16(rng.normal(size=(U, C, din))), _bf16(rng.normal(size=(U, L, din)))
    wq, wk, wv = (_bf16(rng.normal(size=(din, n)) / math.sqrt(din)) for n in (dq, dq, d))
    lens, gamma, S = np.array(lens, dtype=np.int32), math.sqrt(dq / heads), -(-L // w)
    print(f"case {name}", flush=True)
    hn = h[0].copy()
    for u, n in enumerate(lens):
        hn[u, n:] = 0x7fc0
    A = laser.laser_fold_query_weights(to_device(wq[0]), to_device(wk[0]), heads)
    qf = torch.empty((U, C * heads, din), dtype=torch.bfloat16, device="cuda")
    g = torch.empty((U, C * heads, S, din), dtype=torch.bfloat16, device="cuda")
    seg, cnt = laser.laser_sta_folded_forward(to_device(t[0]), to_device(hn), A, to_device(wv[0]), to_device(lens), w,
                                              gamma, heads, qf_work=qf, g_work=g)
    torch.cuda.synchronize()
    g_ref, cnt_ref = oracle.sta_forward(to_host_f64(qf), h[1], h[1], lens, w, gamma)
    assert np.array_equal(cnt.cpu().numpy(), cnt_ref)
    assert vec_rel_err(to_host_f64(g), g_ref) <= TOL["bf16"]
    ref = oracle.project_heads(to_host_f64(g).reshape(U * C, heads, S, din), wv[1], heads).reshape(U, C, S, -1)
    assert vec_rel_err(to_host_f64(seg), ref) <= TOL["bf16"]


# Histories past the last-level cache, which are read with the non-temporal hint. rows, L, d_q, d, w, users (lengths full)
@pytest.mark.parametrize("rows,dq,d,w", [(3, 64, 64, 10), (1, 64, 64, 10), (1, 64, 64, 100), (3, 128, 128, 64), (2, 128, 128, 64),
                                         (1, 128, 128, 20), (1, 64, 128, 30), (1, 32, 128, 30), (2, 32, 128, 11), (1, 32, 128, 10),
                                         (2, 32, 64, 8)])
def test_histories_past_the_cache(rows, dq, d, w):
    import torch
    L = 1000
    U = 300_000_000 // (L * (dq + d) * 2) + 1
    gen = torch.Generator(device="cuda").manual_seed(rows * w)
    q, k, v = (torch.randn(*s, device="cuda", generator=gen).bfloat16() for s in ((U, rows, dq), (U, L, dq), (U, L, d)))
    gamma = math.sqrt(dq)
    print(f"rows {rows} {dq}/{d} w {w} users {U}", flush=True)
    seg, _ = laser.laser_sta_forward(q, k, v, None, w, gamma)
    torch.cuda.synchronize()
    for u in (0, 1, U // 2, U - 1):
        ref, _ = oracle.sta_forward(*(to_host_f64(x[u:u + 1]) for x in (q, k, v)), None, w, gamma)
        assert vec_rel_err(to_host_f64(seg[u:u + 1]), ref) <= TOL["bf16"], u


@pytest.mark.parametrize("rows", [1, 4])
def test_folded_histories_past_the_cache(rows):
    import torch
    U, L, w, din = 1201, 1000, 10, 128
    gen = torch.Generator(device="cuda").manual_seed(rows)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=gen).bfloat16()
    t, h = rnd(U, rows, din), rnd(U, L, din)
    A, wv = rnd(din, din) / math.sqrt(din), rnd(din, din) / math.sqrt(din)
    lens = torch.full((U,), L, device="cuda", dtype=torch.int32)
    g = torch.empty((U, rows, L // w, din), dtype=torch.bfloat16, device="cuda")
    qf = torch.empty((U, rows, din), dtype=torch.bfloat16, device="cuda")
    print(f"rows {rows}", flush=True)
    seg, _ = laser.laser_sta_folded_forward(t, h, A, wv, lens, w, 4.0, 1, qf_work=qf, g_work=g)
    torch.cuda.synchronize()
    for u in (0, 1, U // 2, U - 1):
        ref, _ = oracle.sta_forward(*(to_host_f64(x[u:u + 1]) for x in (qf, h, h)), None, w, 4.0)
        assert vec_rel_err(to_host_f64(g[u:u + 1]), ref) <= TOL["bf16"], u
        ref = to_host_f64(g[u]) @ to_host_f64(wv)
        assert vec_rel_err(to_host_f64(seg[u]), ref) <= TOL["bf16"], u


# Launches of many units a wave, whose workgroups deal their units out by ticket, and some of fewer: every unit is worked on exactly
# where it belongs (outputs start as NaN); folded with 64 columns, the tickets' counter is in a word's place of W_v. folded, rows (heads
# when folded), d_q, d, L, w, users
@pytest.mark.parametrize("folded,rows,dq,d,L,w,U", [(False, 4, 32, 128, 330, 10, 1300), (False, 8, 64, 64, 200, 3, 500),
                                                    (False, 3, 128, 128, 97, 33, 2100), (True, 2, 128, 128, 330, 10, 1200),
                                                    (True, 4, 128, 128, 97, 7, 1100), (True, 1, 128, 64, 130, 65, 3300),
                                                    (False, 8, 64, 64, 200, 3, 5000), (True, 4, 128, 128, 97, 7, 5500),
                                                    (True, 1, 128, 64, 130, 65, 5500), (True, 2, 128, 64, 97, 7, 7000)])
def test_units_dealt_by_ticket(folded, rows, dq, d, L, w, U):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(U)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=gen).bfloat16()
    nan = lambda *s: torch.full(s, float("nan"), device="cuda", dtype=torch.bfloat16)
    lens = torch.randint(0, L + 1, (U,), device="cuda", generator=gen, dtype=torch.int32)
    S, gamma = -(-L // w), 4.0
    print(f"folded {folded} rows {rows} {dq}/{d} w {w} users {U}", flush=True)
    if folded:
        t, h, A, wv = rnd(U, 1, dq), rnd(U, L, dq), rnd(dq, rows * dq) / math.sqrt(dq), rnd(dq, d) / math.sqrt(dq)
        q, sums = nan(U, rows, dq), nan(U, rows, S, dq)
        seg, cnt = laser.laser_sta_folded_forward(t, h, A, wv, lens, w, gamma, rows, qf_work=q, g_work=sums, seg_out=nan(U, 1, S, d))
        k = v = h
    else:
        q, k, v = rnd(U, rows, dq), rnd(U, L, dq), rnd(U, L, d)
        sums, cnt = laser.laser_sta_forward(q, k, v, lens, w, gamma, seg_out=nan(U, rows, S, d))
    torch.cuda.synchronize()
    some = list(range(0, U, 97)) + [U - 1]
    n = lens[some].cpu().numpy()
    ref, _ = oracle.sta_forward(*(to_host_f64(x[some]) for x in (q, k, v)), n, w, gamma)
    assert vec_rel_err(to_host_f64(sums[some]), ref) <= TOL["bf16"]
    assert np.array_equal(cnt.cpu().numpy(), oracle.segment_counts(lens.cpu().numpy(), L, w))
    empty = (cnt == 0)[:, None, :, None]
    for x in (sums, seg) if folded else (sums,):
        assert torch.isfinite(x).all() and not torch.where(empty, x, 0).any()
    if folded:
        ref = oracle.project_heads(to_host_f64(sums[some]).reshape(len(some), rows, S, dq), to_host_f64(wv), rows)
        assert vec_rel_err(to_host_f64(seg[some]), ref.reshape(len(some), 1, S, d)) <= TOL["bf16"]
