"""GPU parity at the edges of the GSTA kernel with tiles of 1 to 16 pairs, against the fp64 checker. fp32 storage is held to 1e-5 and bf16 to 2e-2 per vector, as everywhere (TOL)."""
import math

import numpy as np
import pytest

import oracle

from parity_util import TOL, to_device, to_host_f64, vec_rel_err
from test_sta_backward_gpu import _store

pytestmark = pytest.mark.gpu

laser = pytest.importorskip("paper_2602_11562_amd")

# dtype, U, C, L, w, d, M: pairs per workgroup 1, 2, 4, 8, 16 and a last workgroup that is not full; blocks of H' that
# stay in registers (four and eight rows a lane) and blocks that are read again in every layer
GSTA_CASES = {
    "one_pair_long": ("bf16", 1, 1, 700, 1, 128, 3),
    "resident_f32": ("f32", 3, 5, 130, 9, 128, 2),
    "streamed_f32": ("f32", 3, 3, 1000, 3, 64, 2),
    "two_pairs_a_workgroup_f32": ("f32", 3, 343, 12, 5, 64, 2),
    "four_pairs_a_workgroup_eight_rows": ("bf16", 3, 229, 60, 1, 128, 2),
    "eight_pairs_a_workgroup_f32": ("f32", 3, 457, 30, 1, 128, 1),
    "eight_pairs_a_workgroup_streamed": ("bf16", 3, 417, 180, 2, 128, 2),
    "eight_pairs_a_workgroup_d64": ("bf16", 3, 1367, 40, 1, 64, 2),
    "sixteen_pairs_a_workgroup": ("bf16", 3, 700, 32, 1, 128, 2),
    "sixteen_pairs_a_workgroup_f32": ("f32", 3, 1400, 20, 1, 64, 1),
    "eight_pairs_of_three_rows": ("bf16", 3, 417, 3, 1, 128, 2),       # one and two rows a lane
    "eight_pairs_of_seven_rows": ("bf16", 3, 417, 7, 1, 128, 3),
    "sixteen_pairs_of_one_row": ("bf16", 3, 700, 1, 1, 128, 2),        # two and three rows a lane
    "sixteen_pairs_of_eight_rows": ("bf16", 3, 700, 8, 1, 128, 3),
    "sixteen_pairs_of_twelve_rows": ("bf16", 3, 1400, 12, 1, 128, 2),
    "one_row_a_lane_f32": ("f32", 3, 5, 32, 1, 64, 2),                 # one and two rows a lane, and eight of few pairs
    "two_rows_a_lane": ("bf16", 3, 1367, 16, 1, 64, 2),
    "two_rows_a_lane_f32": ("f32", 3, 700, 15, 1, 64, 1),
    "two_rows_a_lane_and_one_more": ("bf16", 3, 1367, 17, 1, 64, 1),
    "one_pair_a_workgroup_eight_rows": ("bf16", 1, 7, 200, 1, 128, 2),
    "two_pairs_a_workgroup_eight_rows": ("bf16", 3, 110, 100, 1, 128, 2),
    "four_pairs_a_workgroup_eight_rows_f32": ("f32", 3, 229, 60, 1, 128, 3),
}


@pytest.mark.parametrize("name", list(GSTA_CASES))
def test_gsta_tiled(name):
    import torch
    dtype, U, C, L, w, d, M = GSTA_CASES[name]
    S = -(-L // w)
    rng = np.random.default_rng(6100 + sum(map(ord, name)))
    lens = np.array(([L, max(1, L // 3), 0] * U)[:U], dtype=np.int32)
    cnt = oracle.segment_counts(lens, L, w)
    Hs, Hv = _store(rng.normal(size=(U, C, S, d)), dtype)
    ts, tv = _store(rng.normal(size=(U, C, d)), dtype)
    (wqs, wqv), (wks, wkv), (wvs, wvv) = (_store(rng.normal(size=(M, d, d)) / math.sqrt(d), dtype) for _ in range(3))
    print(f"case {name}", flush=True)
    for u, n in enumerate(lens):      # rows of segments without a valid item are never read
        Hs[u, :, -(-int(n) // w):] = np.nan if dtype == "f32" else 0x7fc0
    z = laser.laser_gsta_forward(to_device(Hs), to_device(ts), to_device(wqs), to_device(wks), to_device(wvs),
                                 to_device(lens), L, w, variant=laser.GSTA_AUTO if dtype == "f32" else laser.GSTA_TILED)
    torch.cuda.synchronize()
    pick = slice(None) if C <= 8 else [0, 1, 2, 3, 5, 8, C // 2, C - 2, C - 1]
    ref = oracle.gsta_forward(Hv[:, pick], tv[:, pick], wqv, wkv, wvv, cnt)
    assert vec_rel_err(to_host_f64(z)[:, pick], ref) <= TOL[dtype]
    assert np.array_equal(to_host_f64(z)[lens == 0], tv[lens == 0])     # z = t0 exactly without a valid segment


# pairs, S, d, r: the views from the tiled form (waves that share a pair, one and several pairs a wave, streamed rows) and,
# from larger batches on from the one-kernel form (with and without room for the recent rows) and the split form; equal to
# the two entry points apart, bit for bit
@pytest.mark.parametrize("P,S,d,r", [(3, 5, 128, 5), (300, 40, 128, 3), (1200, 9, 64, 1), (2500, 70, 128, 8),
                                     (5000, 33, 64, 0), (8193, 33, 128, 2), (4097, 9, 128, 3), (4099, 30, 128, 30),
                                     (8195, 20, 64, 2), (4097, 40, 64, 3), (16385, 70, 64, 5)])
def test_views_of_every_form(P, S, d, r):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(P)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=gen).bfloat16()
    seg, t0 = rnd(P, 1, S, d), rnd(P, 1, d)
    W = [(rnd(1, d, d).float() / math.sqrt(d)).bfloat16() for _ in range(3)]
    lens = torch.randint(0, S + 1, (P,), device="cuda", generator=gen, dtype=torch.int32)
    lens[0] = 0
    print(f"P {P} S {S} d {d} r {r}", flush=True)
    z, pool, recent = laser.laser_gsta_forward_multires(seg, t0, *W, lens, S, 1, r)
    z2 = laser.laser_gsta_forward(seg, t0, *W, lens, S, 1)
    pool2, recent2 = laser.laser_multires_forward(seg, lens, S, 1, r)
    torch.cuda.synchronize()
    assert torch.equal(z, z2) and torch.equal(pool.view(torch.int16), pool2.view(torch.int16))
    assert r == 0 or torch.equal(recent.view(torch.int16), recent2.view(torch.int16))


# pairs per workgroup 1, 2, 4, 8, 16 (few pairs: several waves share a pair's rows) and, for S = 300, rows that are streamed
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("P,S", [(12, 9), (300, 9), (600, 20), (1100, 9), (2100, 9), (12, 300), (2100, 300)])
def test_values_that_are_not_finite_reach_the_result(P, S, dtype):
    """A valid segment vector that is not finite, or scores that overflow, make z NaN as in the softmax they stand for; a pair
    whose scores are all near the lowest finite value still has the weights of its softmax. Other pairs are untouched."""
    import torch
    d, w = 128, 3
    L = S * w
    rng = np.random.default_rng(6600 + P + S)
    Hs, Hv = _store(rng.normal(size=(P, S, d)), dtype)
    ts, tv = _store(rng.normal(size=(P, d)), dtype)
    (wqs, wqv), (wks, wkv), (wvs, wvv) = (_store(rng.normal(size=(1, d, d)) / math.sqrt(d), dtype) for _ in range(3))
    nv = np.full(P, S)
    nv[1], nv[8] = S // 2, 0
    special = {0: (0, np.nan), 1: (S // 2 - 1, np.inf), 2: (S // 2, -np.inf), 3: (S - 1, np.nan), 4: (5, np.inf)}
    for p, (row, x) in special.items():
        Hs[p, row, 7] = x if dtype == "f32" else {np.inf: 0x7f80, -np.inf: 0xff80}.get(x, 0x7fc0)
    # scores of one value x in the units of the kernel's exponential (base 2 for bf16): below -3e38 and finite, past the range
    unit = 1.0 if dtype == "f32" else 1.4426950408889634
    for p, x in ((5, -3.2e38), (6, -1e39)):
        ts[p], tv[p] = _store(1e10 * tv[p], dtype)
        r = wkv[0] @ (tv[p] @ wqv[0]) / math.sqrt(d)
        Hs[p], Hv[p] = _store(np.broadcast_to(x / unit * r / (r @ r), (S, d)), dtype)
    lens = (nv * w).astype(np.int32)
    print(f"P {P} S {S} {dtype}", flush=True)
    z = laser.laser_gsta_forward(to_device(Hs[:, None]), to_device(ts[:, None]), to_device(wqs), to_device(wks), to_device(wvs),
                                 to_device(lens), L, w)
    torch.cuda.synchronize()
    got = to_host_f64(z)[:, 0]
    for p in (0, 1, 2, 3, 4, 6):
        assert np.isnan(got[p]).all(), p
    fine = [5, 7, 8, 9, 10, P - 1]
    ref = oracle.gsta_forward(Hv[fine][:, None], tv[fine][:, None], wqv, wkv, wvv, oracle.segment_counts(lens[fine], L, w))
    assert vec_rel_err(got[fine], ref[:, 0]) <= TOL[dtype]
    assert np.isfinite(np.delete(got, (0, 1, 2, 3, 4, 6), axis=0)).all()


@pytest.mark.parametrize("P,S", [(3, 5), (300, 40), (1200, 9), (2500, 70), (4097, 9)])   # tiled form, one-kernel form
def test_pooled_columns_of_minus_infinity(P, S):
    """The pooled view is a selection of stored values: -inf where that is all a column holds, not the zero of a pair without
    a valid segment. (z of such a pair is NaN in every form.)"""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(P)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=gen).bfloat16()
    seg, t0 = rnd(P, 1, S, 128), rnd(P, 1, 128)
    W = [(rnd(1, 128, 128).float() / math.sqrt(128)).bfloat16() for _ in range(3)]
    seg[0, 0, :, 5] = -math.inf
    seg[1, 0, :2, 127] = -math.inf
    seg[2] = -math.inf
    lens = torch.full((P,), S, device="cuda", dtype=torch.int32)
    lens[1], lens[2] = 2, 0
    print(f"P {P} S {S}", flush=True)
    _, pool, _ = laser.laser_gsta_forward_multires(seg, t0, *W, lens, S, 1, 0)
    torch.cuda.synchronize()
    for p, n in ((0, S), (1, 2)):
        assert torch.equal(pool[p, 0], seg[p, 0, :n].max(dim=0).values)
    assert not pool[2].any()


@pytest.mark.parametrize("U,C,S,d,M", [(2, 3, 11, 64, 2), (3, 100, 20, 128, 1)])
def test_generic_by_name_in_fp32(U, C, S, d, M):
    """The generic kernel stays an independent check of the tiled one in single precision: asked for by name it runs."""
    import torch
    rng = np.random.default_rng(6700 + C)
    lens = np.array(([S, S // 3, 0] * U)[:U], dtype=np.int32)
    seg, t0 = rng.normal(size=(U, C, S, d)).astype(np.float32), rng.normal(size=(U, C, d)).astype(np.float32)
    W = [(rng.normal(size=(M, d, d)) / math.sqrt(d)).astype(np.float32) for _ in range(3)]
    args = [to_device(x) for x in (seg, t0, *W, lens)]
    print(f"U {U} C {C} S {S} d {d} M {M}", flush=True)
    auto, generic = (laser.laser_gsta_forward(*args, S, 1, variant=v) for v in (laser.GSTA_AUTO, laser.GSTA_GENERIC))
    torch.cuda.synchronize()
    assert not torch.equal(auto, generic)          # (sums in another order)
    ref = oracle.gsta_forward(seg[:, :3], t0[:, :3], *W, oracle.segment_counts(lens, S, 1))
    for z in (auto, generic):
        assert vec_rel_err(to_host_f64(z)[:, :3], ref) <= TOL["f32"]


@pytest.mark.parametrize("d,P,S", [(64, 8193, 1), (64, 9000, 33), (64, 8200, 64), (64, 16500, 5), (128, 4097, 12), (128, 16390, 3), (128, 8193, 32)])
def test_one_layer_of_many_pairs(d, P, S):
    """Sizes at which the form is chosen for batches that fill the machine: against fp64 of the same inputs (fp32 sums, the factors
    of H' in three bf16 parts: 1e-5 of a vector's largest component) and the other forms (two parts there: 1e-4)."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(P)
    w, C = 4, 1
    seg = torch.randn(P, C, S, d, device="cuda", generator=gen).to(torch.bfloat16)
    t0 = (torch.randn(P, C, d, device="cuda", generator=gen) * 0.3).to(torch.bfloat16)
    ws = [(torch.randn(1, d, d, device="cuda", generator=gen) * d ** -0.5).to(torch.bfloat16) for _ in range(3)]
    lens = torch.randint(0, 4 * S + 1, (P,), device="cuda", generator=gen, dtype=torch.int32)
    z = laser.laser_gsta_forward(seg, t0, *ws, lens, 4 * S, w)
    one = laser.laser_gsta_forward(seg, t0, *ws, lens, 4 * S, w, variant=laser.binding.GSTA_ONE)
    torch.cuda.synchronize()
    H, t = seg[:, 0].cpu().double(), t0[:, 0].cpu().double()
    wq, wk, wv = (x[0].cpu().double() for x in ws)
    r = (t @ wq) @ wk.T / math.sqrt(d)
    nv = (lens.cpu() + w - 1) // w
    scores = (H * r[:, None]).sum(-1).masked_fill(torch.arange(S)[None] >= nv[:, None], float("-inf"))
    a = torch.softmax(scores, 1).nan_to_num(0.0)
    ref = t + (a[:, :, None] * H).sum(1) @ wv
    scale = ref.abs().amax(-1, keepdim=True)
    assert ((z[:, 0].cpu().double() - ref).abs() / scale).max() <= 1e-5
    assert ((one[:, 0].cpu().double() - ref).abs() / scale).max() <= 1e-4


@pytest.mark.parametrize("d,P,S,few", [(64, 4097, 65, 4000), (64, 16400, 33, 4000), (64, 16385, 130, 4000), (128, 8200, 30, 4096), (128, 2050, 33, 2000), (128, 5000, 140, 2000)])
def test_views_of_many_pairs(d, P, S, few):
    """Sixteen pairs of streamed rows take their maxima in the pass over the rows, a few pairs, and other forms, read them once
    more: the same stored values, and z as close as the forms of one layer are to each other (1e-4 of a vector's largest component)."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(S)
    seg = torch.randn(P, 1, S, d, device="cuda", generator=gen).to(torch.bfloat16)
    t0 = (torch.randn(P, 1, d, device="cuda", generator=gen) * 0.3).to(torch.bfloat16)
    ws = [(torch.randn(1, d, d, device="cuda", generator=gen) * d ** -0.5).to(torch.bfloat16) for _ in range(3)]
    lens = torch.randint(0, S + 1, (P,), device="cuda", generator=gen, dtype=torch.int32)
    lens[:3] = torch.tensor([0, 1, S])
    seg[5, 0, 0] = float("-inf")      # a maximum of -inf, and NaN, as the rows read again give them
    seg[6, 0, :, 3] = float("nan")
    lens[5], lens[6] = 1, S
    z, pool, recent = laser.laser_gsta_forward_multires(seg, t0, *ws, lens, S, 1, 3)
    zf, poolf, recentf = laser.laser_gsta_forward_multires(seg[:few], t0[:few], *ws, lens[:few], S, 1, 3)
    only, _ = laser.laser_multires_forward(seg, lens, S, 1, 0)
    torch.cuda.synchronize()
    bits = lambda x: x.view(torch.int16)
    assert torch.equal(bits(pool[:few]), bits(poolf)) and torch.equal(bits(recent[:few]), bits(recentf))
    assert torch.equal(bits(pool[7:]), bits(only[7:])) and torch.equal(bits(pool[:6]), bits(only[:6]))
    ok = torch.ones(few, dtype=torch.bool, device="cuda")
    ok[5:7] = False
    assert ((z[:few] - zf).abs() / zf.abs().amax(-1, keepdim=True))[ok].max() <= 1e-4
    assert z[5].isnan().all() and z[6].isnan().all()
