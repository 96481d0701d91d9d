"""The direct-to-LDS STA kernel (d_q = d = 128) with its workgroups dealt out by the users' lengths: every row of H' and every
count is written, once, whatever the lengths and the candidates' counts, against the generic kernel (bf16 results: the two differ
by the gates' rounding, 2e-2 as everywhere)."""
import math

import pytest

from parity_util import TOL

pytestmark = pytest.mark.gpu

laser = pytest.importorskip("paper_2602_11562_amd")

# users, candidates, items, w, lengths, own counts per user. Dealt out: own counts from three segments of a workgroup on, dense
# calls past eight, up to 64 users, both workgroup sizes, the last tile of a segment of one item, users without candidates or
# items, full and empty histories. Not: one round of the launch's own division, 65 users, segments of a tile or less
CASES = [(29, 201, 3001, 100, "mixed", True), (40, 300, 2500, 100, "mixed", False), (40, 300, 2500, 100, "full", False),
         (64, 70, 2910, 97, "mixed", True), (64, 128, 2800, 70, "mixed", False), (13, 500, 3500, 65, "mixed", True),
         (64, 300, 640, 80, "empty", True), (33, 257, 1500, 129, "full", True),
         (7, 129, 3001, 100, "mixed", False), (65, 70, 900, 40, "mixed", True), (5, 257, 1000, 64, "mixed", True)]


@pytest.mark.parametrize("U,C,L,w,lens,own", CASES)
def test_every_row_is_written(U, C, L, w, lens, own):
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
    else:
        n[0] = L
        n[U // 2:U // 2 + 1] = 0 if U > 1 else L
    print(f"U {U} C {C} L {L} w {w} {lens} {own}", flush=True)
    if own:
        counts = torch.randint(0, C + 1, (U,), generator=torch.Generator().manual_seed(U))
        counts[0], counts[-1] = C, 0
        off = torch.cat([torch.zeros(1, dtype=torch.int64), counts.cumsum(0)]).to(torch.int32).cuda()
        user = torch.repeat_interleave(torch.arange(U), counts)
        P = int(counts.sum())
        q = rnd(P, d)
        out, cnt = torch.full((P, S, d), math.nan, device="cuda").bfloat16(), torch.full((U, S), -7, device="cuda", dtype=torch.int32)
        laser.laser_forward_ragged(q, k, v, None, None, None, None, n, off, C, w, math.sqrt(d), seg_out=out, seg_cnt=cnt, stage="sta")
        qd = torch.zeros(U, C, d, device="cuda").bfloat16()
        place = torch.cat([torch.arange(int(c)) for c in counts])
        qd[user, place] = q
        ref, ref_cnt = laser.laser_sta_forward(qd, k, v, n, w, math.sqrt(d), variant=laser.STA_GENERIC)
        ref = ref[user, place]
    else:
        q = rnd(U, C, d)
        out, cnt = torch.full((U, C, S, d), math.nan, device="cuda").bfloat16(), torch.full((U, S), -7, device="cuda", dtype=torch.int32)
        laser.laser_sta_forward(q, k, v, n, w, math.sqrt(d), seg_out=out, seg_cnt=cnt, variant=laser.STA_MFMA)
        ref, ref_cnt = laser.laser_sta_forward(q, k, v, n, w, math.sqrt(d), variant=laser.STA_GENERIC)
    torch.cuda.synchronize()
    assert torch.equal(cnt, ref_cnt)
    out, ref = out.float(), ref.float()
    assert torch.isfinite(out).all()
    top = ref.abs().amax(-1)
    assert ((out - ref).abs().amax(-1) <= TOL["bf16"] * top).all()      # rows of empty segments are zeros exactly


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
