"""The matrix-core STA kernel with a wave of its own for the fetches, where its form or its edges change: segments around half a
block, a block and several (1 .. 3 of them per chunk), candidates around 32 and 64, several heads, short last segments, lengths
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


@pytest.mark.parametrize("U,C,L,dq,d,w,heads", CASES)
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
