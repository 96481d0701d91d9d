"""GPU parity at the edges of the GSTA kernel that keeps the layers' matrices in
registers, against the fp64 checker. fp32 storage is held to 1e-5 and bf16 to 2e-2 per vector, as everywhere (TOL)."""
import math

import numpy as np
import pytest

import oracle

from parity_util import TOL, to_device, to_host_f64, vec_rel_err
from test_sta_backward_gpu import _store

pytestmark = pytest.mark.gpu

laser = pytest.importorskip("paper_2602_11562_amd")

# dtype, U, C, L, w, d, M: pairs per workgroup 1, 2, 4, 8 and a last workgroup that is not full; blocks of H' that stay
# in registers and blocks that are read again in every layer
GSTA_CASES = {
    "one_pair_long": ("bf16", 1, 1, 700, 1, 128, 3),
    "resident_f32": ("f32", 3, 5, 130, 9, 128, 2),
    "streamed_f32": ("f32", 3, 3, 1000, 3, 64, 2),
    "two_pairs_a_workgroup": ("f32", 3, 343, 12, 5, 64, 2),
    "four_pairs_a_workgroup": ("f32", 3, 685, 70, 2, 64, 1),
    "eight_pairs_a_workgroup": ("f32", 3, 1367, 9, 1, 128, 1),
    "bf16_streamed_four_pairs": ("bf16", 3, 685, 180, 2, 128, 2),
}


@pytest.mark.parametrize("name", list(GSTA_CASES))
def test_gsta_rows(name):
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
                                 to_device(lens), L, w, variant=laser.GSTA_GENERIC)
    torch.cuda.synchronize()
    pick = slice(None) if C <= 8 else [0, 1, 2, 3, 5, 8, C // 2, C - 2, C - 1]
    ref = oracle.gsta_forward(Hv[:, pick], tv[:, pick], wqv, wkv, wvv, cnt)
    assert vec_rel_err(to_host_f64(z)[:, pick], ref) <= TOL[dtype]
    assert np.array_equal(to_host_f64(z)[lens == 0], tv[lens == 0])     # z = t0 exactly without a valid segment
