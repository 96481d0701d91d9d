"""The projections around a separate GSTA pass, through the split form: every pair of every tile against the layer in fp64."""
import math

import pytest

pytestmark = pytest.mark.gpu

laser = pytest.importorskip("paper_2602_11562_amd")


# tiles of 16 pairs: one and part of one, either side of a tile's end, and more tiles than the 512 workgroups (d = 128; 1024 at d = 64)
# that walk them, with a last tile of one pair, of fifteen and full. Factors enter the products with 24 bits and are summed in
# fp32, so a vector's error is some 2^-24 of its largest component for each of the chain's steps: below 1e-5 with a margin.
@pytest.mark.parametrize("d,P", [(64, 1), (64, 15), (64, 16), (64, 17), (64, 16385), (64, 16399), (64, 32768), (128, 1), (128, 15),
                                 (128, 17), (128, 8193), (128, 8207), (128, 16384)])
def test_split_form_every_pair(d, P):
    import torch
    S, w = 7, 1
    gen = torch.Generator(device="cuda").manual_seed(P + d)
    rnd = lambda *s, sd=1.0: (torch.randn(*s, device="cuda", generator=gen) * sd).bfloat16()
    seg, t0 = rnd(P, 1, S, d), rnd(P, 1, d)
    wq, wk, wv = (rnd(1, d, d, sd=d ** -0.5) for _ in range(3))
    lens = torch.randint(0, S + 1, (P,), device="cuda", generator=gen, dtype=torch.int32)
    if P > 1:
        lens[P - 2], lens[P - 1] = 0, S
    print(f"d {d} pairs {P}", flush=True)
    z = laser.laser_gsta_forward(seg, t0, wq, wk, wv, lens, S, w, variant=laser.GSTA_SPLIT,
                                 z_out=torch.full((P, 1, d), float("nan"), device="cuda"))
    torch.cuda.synchronize()
    h, t = seg[:, 0].double(), t0[:, 0].double()
    r = t @ wq[0].double() @ wk[0].double().T.contiguous()
    empty = torch.arange(S, device="cuda")[None] >= lens[:, None]
    score = ((h * r[:, None]).sum(-1) / math.sqrt(d)).masked_fill(empty, float("-inf"))
    a = torch.nan_to_num(torch.softmax(score, 1))       # (no valid segment: nothing is added)
    ref = t + (a[:, :, None] * h).sum(1) @ wv[0].double()
    err = (z[:, 0].double() - ref).abs().amax(1) / ref.abs().amax(1)
    print(f"largest error {err.max().item():.1e}")
    assert (err <= 1e-5).all(), err.argmax().item()
    assert torch.equal(z[:, 0][lens == 0], t0[:, 0][lens == 0].float())
