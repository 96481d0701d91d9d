"""GPU parity where the choice of the register-staged matrix-core STA kernel's workgroup changes (candidates per workgroup,
segments per workgroup, segments shorter than a staged tile of 64 items), against the fp64 checker (2e-2 per vector)."""
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
    # eight waves below w = 64 (an even number of fours, enough segments), and four for an odd number or short segments
    "200_candidates_w40": (45, 200, 240, 64, 64, 40, 1),
    "300_candidates_w40": (45, 300, 240, 64, 64, 40, 1),
    "256_candidates_w20": (45, 256, 240, 64, 64, 20, 1),
    "384_candidates_two_heads_w21": (20, 384, 270, 32, 128, 21, 2),
    "512_candidates_two_heads_w20": (20, 512, 270, 64, 64, 20, 2),
}


@pytest.mark.parametrize("name", list(CASES))
def test_workgroup_choice(name):
    import torch
    U, C, L, dq, d, w, heads = CASES[name]
    rng = np.random.default_rng(6400 + sum(map(ord, name)))
    bits = [workloads.f32_to_bf16_bits(rng.normal(size=s).astype(np.float32)) for s in ((U, C, dq), (U, L, dq), (U, L, d))]
    q, k, v = (workloads.bf16_bits_to_f32(b).astype(np.float64) for b in bits)
    lens = np.array([L, 0, w, w + 1][:U] + list(rng.integers(1, L + 1, max(0, U - 4))), dtype=np.int32)
    gamma = math.sqrt(dq / heads)
    print(f"case {name}", flush=True)
    seg, cnt = laser.laser_sta_forward(*(to_device(b) for b in bits), to_device(lens), w, gamma, heads=heads)
    torch.cuda.synchronize()
    assert np.array_equal(cnt.cpu().numpy(), oracle.segment_counts(lens, L, w))
    got = to_host_f64(seg)
    for u in range(min(U, 6)):
        ref, _ = oracle.sta_forward(q[u:u + 1], k[u:u + 1], v[u:u + 1], lens[u:u + 1], w, gamma, heads=heads)
        assert vec_rel_err(got[u:u + 1], ref) <= TOL["bf16"], u
