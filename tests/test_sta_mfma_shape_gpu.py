"""GPU parity of the matrix-core STA kernels where the choice of their workgroups changes (candidates per workgroup, segments per
workgroup, segments shorter than the register-staged kernel's tile of 64 items), against the fp64 checker (2e-2 per vector). With
sigmoid gates these calls run the kernel with a wave of its own for the fetches, with softmax the register-staged one, whose eight
waves prefetch into a second tile; test_launches_cpu.py shows both."""
import math

import numpy as np
import pytest

import oracle
import workloads

from parity_util import TOL, to_device, to_host_f64, vec_rel_err

pytestmark = pytest.mark.gpu

laser = pytest.importorskip("paper_2602_11562_amd")

# U, C, L, d_q, d, w, heads
CASES = {
    "129_candidates_w63": (3, 129, 200, 64, 64, 63, 1),
    "129_candidates_w64": (3, 129, 200, 64, 64, 64, 1),
    "257_candidates_short_last_segment": (2, 257, 101, 32, 128, 20, 1),
    "two_heads_many_segments": (4, 140, 251, 32, 128, 2, 2),
    "65_candidates_runs_past_the_end": (30, 65, 190, 128, 64, 10, 1),
    # softmax, eight waves below w = 64: an even number of fours and enough segments; else four
    "200_candidates_w40": (45, 200, 240, 64, 64, 40, 1),
    "300_candidates_w40": (45, 300, 240, 64, 64, 40, 1),
    "256_candidates_w20": (45, 256, 240, 64, 64, 20, 1),
    "384_candidates_two_heads_w21": (20, 384, 270, 32, 128, 21, 2),
    "512_candidates_two_heads_w20": (20, 512, 270, 64, 64, 20, 2),
    # softmax: eight waves at four heads, a prefetch that spans a segment's end, last tiles of one and of 65 items
    "160_candidates_four_heads_w130": (3, 160, 391, 64, 128, 130, 4),
    "256_candidates_wide_w65": (2, 256, 261, 128, 128, 65, 1),
}


def eight_waves(U, C, L, w):
    """Whether the register-staged kernel takes this softmax call with eight waves and two tiles."""
    S = -(-L // w)
    return C > 128 and (w >= 64 or (-(-C // 128) % 2 == 0 and U * -(-C // 256) * S > 384))


@pytest.mark.parametrize("softmax", [False, True], ids=["sigmoid", "softmax"])
@pytest.mark.parametrize("name", list(CASES))
def test_workgroup_choice(name, softmax):
    import torch
    U, C, L, dq, d, w, heads = CASES[name]
    rng = np.random.default_rng(6400 + sum(map(ord, name)))
    bits = [workloads.f32_to_bf16_bits(rng.normal(size=s).astype(np.float32)) for s in ((U, C, dq), (U, L, dq), (U, L, d))]
    q, k, v = (workloads.bf16_bits_to_f32(b).astype(np.float64) for b in bits)
    lens = np.array([L, 0, w, w + 1][:U] + list(rng.integers(1, L + 1, max(0, U - 4))), dtype=np.int32)
    gamma = math.sqrt(dq / heads)
    print(f"case {name} softmax {softmax}", flush=True)
    seg, cnt = laser.laser_sta_forward(*(to_device(b) for b in bits), to_device(lens), w, gamma, heads=heads, softmax=softmax)
    torch.cuda.synchronize()
    assert np.array_equal(cnt.cpu().numpy(), oracle.segment_counts(lens, L, w))
    got = to_host_f64(seg)
    for u in range(min(U, 6)):
        ref, _ = oracle.sta_forward(q[u:u + 1], k[u:u + 1], v[u:u + 1], lens[u:u + 1], w, gamma, heads=heads, softmax=softmax)
        assert vec_rel_err(got[u:u + 1], ref) <= TOL["bf16"], u
