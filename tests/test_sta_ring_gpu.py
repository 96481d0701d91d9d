"""The matrix-core STA kernel with a wave of its own for the fetches, where its form or its edges change: segments around half a
block, a block and several (1 .. 3 of them per chunk), candidates around 32, 64 and 96, several heads, short last segments, lengths
that end inside a block; a history that is not finite past the valid length and in the next segment, and nothing written beside
the outputs. Against the generic kernel (fp32 arithmetic; the gates are rounded to bf16 here and not there: 2e-2 as everywhere)."""
import math

import pytest

from parity_util import TOL

pytestmark = pytest.mark.gpu

laser = pytest.importorskip("paper_2602_11562_amd")

# U, C, L, d_q, d, w, heads
CASES = [(3, 9, 97, 32, 64, 1, 1), (4, 33, 203, 64, 64, 10, 1), (3, 32, 120, 64, 128, 11, 1), (5, 65, 333, 32, 128, 16, 2),
         (3, 64, 170, 128, 64, 17, 1), (4, 40, 310, 64, 128, 31, 4), (4, 31, 321, 128, 128, 32, 1), (2, 97, 331, 64, 64, 33, 2),
         (3, 50, 400, 128, 128, 63, 4), (2, 129, 700, 32, 64, 65, 1), (70, 70, 64, 64, 64, 7, 1), (1, 20, 25, 32, 128, 400, 1),
         (300, 200, 30, 32, 64, 3, 1), (6, 300, 900, 128, 128, 45, 1)]
# ... and with three computing waves: candidates around 96 and its multiples
THREE = [(60, 95, 300, 32, 64, 33, 1), (60, 96, 200, 64, 64, 15, 1), (40, 193, 203, 128, 64, 16, 1), (30, 193, 150, 64, 128, 31, 4),
         (30, 280, 300, 64, 128, 70, 4), (60, 90, 260, 128, 128, 64, 2), (3, 96, 400, 32, 128, 9, 2), (50, 95, 210, 128, 64, 63, 2),
         (70, 190, 96, 64, 128, 40, 1), (40, 258, 64, 128, 128, 33, 1), (7, 160, 260, 128, 128, 10, 4)]


@pytest.mark.parametrize("U,C,L,dq,d,w,heads", CASES + THREE)
def test_edges(U, C, L, dq, d, w, heads):
    import torch
    S = -(-L // w)
    gen = torch.Generator(device="cuda").manual_seed(L + w)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=gen).bfloat16()
    q, k, v = rnd(U, C, dq), rnd(U, L, dq), rnd(U, L, d)
    n = torch.randint(0, L + 1, (U,), device="cuda", generator=gen, dtype=torch.int32)
    n[0] = L
    if U > 2:
        n[1], n[2] = 0, max(1, L - w - 1)
    for u in range(min(U, 8)):      # what lies past the valid length never enters
        k[u, int(n[u]):] = math.nan
        v[u, int(n[u]):] = math.inf
    g = math.sqrt(dq / heads)
    out = torch.full((U * C + 2, S, d), 3.0, device="cuda").bfloat16()
    cnt = torch.full((U + 2, S), -7, device="cuda", dtype=torch.int32)
    print(f"U {U} C {C} L {L} d_q {dq} d {d} w {w} heads {heads}", flush=True)
    laser.laser_sta_forward(q, k, v, n, w, g, seg_out=out[1:-1].view(U, C, S, d), seg_cnt=cnt[1:-1], heads=heads)
    ref, ref_cnt = laser.laser_sta_forward(q, k, v, n, w, g, heads=heads, variant=laser.STA_GENERIC)
    torch.cuda.synchronize()
    assert (out[[0, -1]] == 3.0).all() and (cnt[[0, -1]] == -7).all()
    assert torch.equal(cnt[1:-1], ref_cnt)
    ref = ref.float().view(U * C, S, d)
    top = ref.abs().amax(-1)
    assert ((out[1:-1].float() - ref).abs().amax(-1) <= TOL["bf16"] * top).all()      # (rows of empty segments: zeros exactly)


@pytest.mark.parametrize("w", [10, 40])
@pytest.mark.parametrize("what", [math.inf, math.nan])
def test_values_that_are_not_finite_stay_in_their_segment(w, what):
    import torch
    U, C, L, d = 2, 48, 200, 64
    gen = torch.Generator(device="cuda").manual_seed(w)
    q, k, v = (torch.randn(*s, device="cuda", generator=gen).bfloat16() for s in ((U, C, d), (U, L, d), (U, L, d)))
    hit = v.clone()
    hit[1, 2 * w] = what            # the first item of segment 2
    hit[1, 4 * w - 1] = what        # the last of segment 3
    n = torch.tensor([L, 4 * w], device="cuda", dtype=torch.int32)
    a, _ = laser.laser_sta_forward(q, k, v, n, w, 8.0)
    b, _ = laser.laser_sta_forward(q, k, hit, n, w, 8.0)
    torch.cuda.synchronize()
    bad = torch.zeros_like(a, dtype=torch.bool)
    bad[1, :, 2:4] = True
    assert torch.equal(a[~bad], b[~bad])
    got = b[bad]
    assert (got.isnan() if math.isnan(what) else got == math.inf).all()


@pytest.mark.parametrize("U,C,L,w", [(1, 70, 300, 9), (5, 130, 400, 3), (16, 90, 203, 40), (17, 90, 203, 40), (19, 200, 120, 11)])
def test_counts_of_their_own(U, C, L, w):
    """Up to 16 users the workgroups run in the order in which they are dealt, past them in ranges per XCD: either way every
    user's rows are those of a call of its own, bit for bit, users without candidates among them."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(U)
    counts = [C] + [int(x) for x in torch.randint(0, C + 1, (U - 1,), generator=torch.Generator().manual_seed(U))]
    if U > 2:
        counts[1] = 0
    off = torch.tensor([0] + counts, device="cuda").cumsum(0).to(torch.int32)
    P = sum(counts)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=gen).bfloat16()
    q, k, v = rnd(P, 64), rnd(U, L, 64), rnd(U, L, 128)
    n = torch.randint(0, L + 1, (U,), device="cuda", generator=gen, dtype=torch.int32)
    n[0] = L
    print(f"U {U} C {C} L {L} w {w}", flush=True)
    out, cnt, _ = laser.laser_forward_ragged(q, k, v, None, None, None, None, n, off, C, w, 8.0, stage="sta")
    for u in range(U):
        lo, c = int(off[u]), counts[u]
        if c < 9:      # (a dense call of so few runs another kernel)
            continue
        ref, ref_cnt = laser.laser_sta_forward(q[lo:lo + c].view(1, c, 64), k[u:u + 1], v[u:u + 1], n[u:u + 1], w, 8.0)
        assert torch.equal(out[lo:lo + c].view(torch.int16), ref[0].view(torch.int16)), u
        assert torch.equal(cnt[u], ref_cnt[0])
