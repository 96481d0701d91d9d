"""GPU parity of GSTA's backward pass in tiles of pairs (d in {64, 128}) against the fp64 checker at the edges of the tiles:
1 to 16 pairs per workgroup with a last one that is not full, rows of H' shared by several waves, several layers, pairs
without a valid segment. fp32 results of fp32 arithmetic: 1e-5; dH' in the storage type as everywhere (TOL)."""
import math

import numpy as np
import pytest

import oracle

from parity_util import TOL, to_device, to_host_f64, vec_rel_err
from test_sta_backward_gpu import _store

pytestmark = pytest.mark.gpu

laser = pytest.importorskip("paper_2602_11562_amd")

# dtype, U, C, L, w, d, M
CASES = {
    "one_pair_many_rows": ("bf16", 1, 1, 261, 1, 128, 1),
    "one_pair_a_workgroup_deep": ("f32", 3, 5, 37, 3, 128, 4),
    "two_pairs_a_workgroup": ("bf16", 3, 171, 20, 3, 64, 2),
    "four_pairs_a_workgroup": ("f32", 3, 229, 9, 1, 64, 1),
    "eight_pairs_a_workgroup": ("bf16", 3, 457, 33, 4, 128, 2),
    "sixteen_pairs_a_workgroup": ("bf16", 3, 1367, 5, 1, 64, 1),
    "eight_layers_that_halve_the_tile": ("bf16", 3, 342, 90, 1, 128, 8),
}


@pytest.mark.parametrize("name", list(CASES))
def test_gsta_backward_tiles(name):
    import torch
    dtype, U, C, L, w, d, M = CASES[name]
    S = -(-L // w)
    rng = np.random.default_rng(7100 + sum(map(ord, name)))
    lens = np.array(([L, max(1, L // 3), 0] * U)[:U], dtype=np.int32)
    cnt = oracle.segment_counts(lens, L, w)
    Hp = rng.normal(size=(U, C, S, d)) * (cnt[:, None, :, None] > 0)
    st = {"seg": _store(Hp, dtype), "t0": _store(rng.normal(size=(U, C, d)), dtype)}
    for nm in ("wq", "wk", "wv"):
        st[nm] = _store(rng.normal(size=(M, d, d)) / math.sqrt(d), dtype)
    dz = rng.normal(size=(U, C, d)).astype(np.float32)
    val = {k: v[1] for k, v in st.items()}
    print(f"case {name}", flush=True)
    ref = oracle.gsta_backward(val["seg"], val["t0"], val["wq"], val["wk"], val["wv"], cnt, dz.astype(np.float64))
    dev = {k: to_device(v[0]) for k, v in st.items()}
    args = (dev["seg"], dev["t0"], dev["wq"], dev["wk"], dev["wv"], to_device(lens), to_device(dz), L, w)
    got = laser.laser_gsta_backward(*args)
    torch.cuda.synchronize()
    for nm, a, b, tol in zip(("dseg", "dt0", "dwq", "dwk", "dwv"), got, ref, (TOL[dtype], 1e-5, 1e-5, 1e-5, 1e-5)):
        a = to_host_f64(a)
        if nm.startswith("dw"):
            a, b = a.reshape(M, -1), b.reshape(M, -1)
        err = vec_rel_err(a, b)
        print(f"  {nm}: {err:.3e}", flush=True)
        assert err <= tol, nm
    again = laser.laser_gsta_backward(*args)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(got, again))      # fixed summation order
