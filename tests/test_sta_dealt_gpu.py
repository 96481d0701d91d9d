"""The direct-to-LDS STA kernel (d_q = d = 128) with its workgroups dealt out by the users' lengths: every row of H' and every
count is written, whatever the lengths and the candidates' counts, and nothing beside them, alone and in the whole path, against
the generic kernel (bf16 results: the two differ by the gates' rounding, 2e-2 as everywhere). test_launches_cpu.py shows that
these calls launch the dealt form, or do not, as listed."""
import math

import pytest

from parity_util import TOL

pytestmark = pytest.mark.gpu

laser = pytest.importorskip("paper_2602_11562_amd")

# users, candidates, items, w, lengths, own counts per user, whether workgroups are dealt out: with own counts from three
# segments of a workgroup on, dense calls from four, up to 64 users, both workgroup sizes. Among them the last tile of a segment of
# one item, users without candidates or items, full and empty histories, and histories that divided anew have runs no shorter.
# Not dealt out: one round of the launch's own division, 65 users, segments of a tile or less
CASES = [(29, 201, 3001, 100, "mixed", True, True), (40, 300, 2500, 100, "mixed", False, True),
         (40, 300, 2500, 100, "full", False, True), (64, 70, 2910, 97, "mixed", True, True),
         (64, 128, 2800, 70, "mixed", False, True), (13, 500, 3500, 65, "mixed", True, True),
         (64, 300, 640, 80, "empty", True, True), (33, 257, 1500, 129, "full", True, True),
         (9, 480, 6000, 80, "one_short", True, True), (64, 128, 2800, 70, "one_short", False, True),
         (12, 128, 6400, 100, "last_only", True, True),
         (37, 436, 1069, 117, "mixed", False, True), (45, 85, 5390, 238, "full", False, True), (12, 453, 4905, 243, "mixed", False, False),
         (7, 129, 3001, 100, "mixed", False, False), (65, 70, 900, 40, "mixed", True, False), (5, 257, 1000, 64, "mixed", True, False),
         # segments shorter than the tile of 32 items and as long, both workgroup sizes: partial tiles alone, a segment done every step
         (5, 130, 203, 1, "mixed", True, False), (9, 96, 301, 2, "mixed", True, False), (5, 200, 303, 10, "one_short", True, False),
         (6, 100, 333, 10, "mixed", True, False), (3, 300, 500, 31, "mixed", True, False), (6, 257, 640, 32, "full", True, False),
         (20, 70, 645, 31, "mixed", True, False), (4, 128, 641, 32, "mixed", True, False), (70, 90, 200, 33, "mixed", True, False)]


@pytest.mark.parametrize("whole", [False, True], ids=["sta", "whole_path"])
@pytest.mark.parametrize("U,C,L,w,lens,own,dealt", CASES)
def test_every_row_is_written(U, C, L, w, lens, own, dealt, whole):
    import torch
    d = 128
    S = -(-L // w)
    gen = torch.Generator(device="cuda").manual_seed(U * C + L)
    rnd = lambda *s: (torch.randn(*s, device="cuda", generator=gen) * d ** -0.5).bfloat16()
    k, v = rnd(U, L, d), rnd(U, L, d)
    n = torch.randint(0, L + 1, (U,), device="cuda", generator=gen, dtype=torch.int32)
    if lens == "full":
        n[:] = L
    elif lens == "empty":
        n[:] = 0
    elif lens == "one_short":
        n[:] = L
        n[U // 2] = L - 1
    elif lens == "last_only":
        n[:] = 0
        n[-2] = L
    else:
        n[0] = L
        n[U // 2:U // 2 + 1] = 0 if U > 1 else L
    print(f"U {U} C {C} L {L} w {w} {lens} {own} {whole}", flush=True)
    counts = torch.full((U,), C)
    if own:
        counts = torch.randint(0, C + 1, (U,), generator=torch.Generator().manual_seed(U))
        counts[0], counts[-1] = C, 0
        if lens == "last_only":
            counts[-2] = C
    off = torch.cat([torch.zeros(1, dtype=torch.int64), counts.cumsum(0)]).to(torch.int32).cuda()
    P = int(counts.sum())
    q, t0, weights = rnd(P, d), rnd(P, d), [rnd(1, d, d) for _ in range(3)]
    # a row more before and after each output
    outs = [torch.full((P + 2, S, d), math.nan, device="cuda").bfloat16(), torch.full((U + 2, S), -7, device="cuda", dtype=torch.int32),
            torch.full((P + 2, d), math.nan, device="cuda")]
    out, cnt, z = (x[1:-1] for x in outs)
    g = math.sqrt(d)
    if own:
        laser.laser_forward_ragged(q, k, v, t0, *weights, n, off, C, w, g, seg_out=out, seg_cnt=cnt, z_out=z,
                                   stage="both" if whole else "sta")
        _, _, z_ref = laser.laser_forward_ragged(None, k, v, t0, *weights, n, off, C, w, g, seg_out=out, stage="gsta")
    else:
        q4, t4, o4, z4 = q.view(U, C, d), t0.view(U, C, d), out.view(U, C, S, d), z.view(U, C, d)
        if whole:
            laser.laser_forward(q4, k, v, t4, *weights, n, w, g, seg_out=o4, seg_cnt=cnt, z_out=z4)
        else:
            laser.laser_sta_forward(q4, k, v, n, w, g, seg_out=o4, seg_cnt=cnt, variant=laser.STA_MFMA)
        z_ref = laser.laser_gsta_forward(o4, t4, *weights, n, L, w).view(P, d)
    user = torch.repeat_interleave(torch.arange(U), counts)
    place = torch.cat([torch.arange(int(c)) for c in counts])
    qd = torch.zeros(U, C, d, device="cuda").bfloat16()
    qd[user, place] = q
    ref, ref_cnt = laser.laser_sta_forward(qd, k, v, n, w, g, variant=laser.STA_GENERIC)
    ref = ref[user, place].float()
    torch.cuda.synchronize()
    assert torch.equal(cnt, ref_cnt)
    assert torch.isfinite(out).all()
    top = ref.abs().amax(-1)
    assert ((out.float() - ref).abs().amax(-1) <= TOL["bf16"] * top).all()      # rows of empty segments are zeros exactly
    if whole:
        assert torch.equal(z, z_ref)
    for x in outs:
        edge = x[[0, -1]]
        assert (edge == -7).all() if x.dtype == torch.int32 else edge.isnan().all()


def test_many_segments_shorter_than_a_tile():
    """Dense calls of enough segments of 17 items and more: the rows that each user's call of its own gives (another kernel with the
    same arithmetic), bit for bit; test_launches_cpu.py shows which kernels these are."""
    import torch
    U, C, L, w, d = 64, 180, 1241, 17, 128
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn(*s, device="cuda", generator=gen).bfloat16() for s in ((U, C, d), (U, L, d), (U, L, d)))
    n = torch.randint(0, L + 1, (U,), device="cuda", generator=gen, dtype=torch.int32)
    n[0], n[1], n[2] = L, 0, L - 1
    for u in range(U):
        v[u, int(n[u]):] = math.nan
    out, cnt = laser.laser_sta_forward(q, k, v, n, w, math.sqrt(d))
    for u in (0, 1, 2, 31, 63):
        ref, ref_cnt = laser.laser_sta_forward(*(x[u:u + 1] for x in (q, k, v, n)), w, math.sqrt(d))
        assert torch.equal(out[u].view(torch.int16), ref[0].view(torch.int16)) and torch.equal(cnt[u], ref_cnt[0]), u


@pytest.mark.parametrize("kind", ["above_the_count", "past_the_pairs", "decreasing", "huge"])
def test_offsets_that_break_the_rules_stay_inside_the_buffers(kind):
    """The kernel clamps every user's range for itself, also where it shares the empty rows of all users."""
    import torch
    U, C, P, L, w, d = 13, 500, 900, 3500, 65, 128
    S = -(-L // w)
    off = {"above_the_count": [0, 600, 620] + [700] * 10 + [P], "past_the_pairs": [P + 50, P + 60] + [3] * 11 + [P],
           "decreasing": [0, 400, 401, 90, 300, 10, 500, 20, 600, 30, 700, 40, 800, P], "huge": [0] * 12 + [1 << 30, -(1 << 30)]}[kind]
    rnd = lambda *s: torch.randn(*s, device="cuda").bfloat16()
    lens = (torch.arange(U, device="cuda", dtype=torch.int32) * 271) % (L + 1)
    out, cnt = torch.full((P + 2, S, d), 3.0, device="cuda").bfloat16(), torch.full((U + 2, S), -7, device="cuda", dtype=torch.int32)
    print(kind, flush=True)
    laser.laser_forward_ragged(rnd(P, d), rnd(U, L, d), rnd(U, L, d), None, None, None, None, lens,
                               torch.tensor(off, dtype=torch.int32, device="cuda"), C, w, math.sqrt(d), seg_out=out[1:-1],
                               seg_cnt=cnt[1:-1], stage="sta")
    torch.cuda.synchronize()
    assert (out[[0, -1]] == 3.0).all() and (cnt[[0, -1]] == -7).all() and out.isfinite().all()
    items = (lens[:, None] - torch.arange(S, device="cuda")[None, :] * w).clamp(0, w)
    items[:, -1] = items[:, -1].clamp(max=L - (S - 1) * w)
    assert torch.equal(cnt[1:-1], items.to(torch.int32))


@pytest.mark.parametrize("U,C,L,w,valid", [(6, 277, 6781, 83, [1, 1, 12, 1, 0, 3]), (13, 452, 7755, 67, [1, 116] + [2] * 11),
                                           (16, 106, 9845, 68, [145, 145] + [3] * 14)])
def test_short_histories_take_no_longer_than_full_ones(U, C, L, w, valid):
    """The rows of empty segments are everybody's work: left to the few workgroups of a short history they took up to 2.3 times the
    time of the whole launch."""
    import torch
    d, S = 128, -(-L // w)
    k, v, q = (torch.randn(*s, device="cuda").bfloat16() for s in ((U, L, d), (U, L, d), (U * C, d)))
    off = torch.arange(0, U * C + 1, C, dtype=torch.int32, device="cuda")
    out, cnt = torch.empty(U * C, S, d, device="cuda", dtype=torch.bfloat16), torch.empty(U, S, device="cuda", dtype=torch.int32)

    def us(lens):
        best = math.inf
        for _ in range(20):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(10):
                laser.laser_forward_ragged(q, k, v, None, None, None, None, lens, off, C, w, math.sqrt(d), seg_out=out, seg_cnt=cnt,
                                           stage="sta")
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 100)
        return best

    full, short = (us(torch.tensor(x, dtype=torch.int32, device="cuda").clamp(max=S) * w) for x in ([S] * U, valid))
    print(f"U {U} C {C} L {L} w {w}: {full:.1f} us with full histories, {short:.1f} with short ones", flush=True)
    assert short <= 1.15 * full
