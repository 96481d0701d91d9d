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


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("P,S", [(12, 9), (300, 9), (600, 20), (1100, 9), (2100, 9)])   # 1, 2, 4, 8, 16 pairs a workgroup
@pytest.mark.parametrize("M", [1, 2])
def test_values_that_are_not_finite_reach_the_gradients(P, S, M, dtype):
    """A valid segment vector that is not finite, or scores that overflow: the pair's gradients are NaN, as those of the
    softmax they stand for, and other pairs' are untouched; scores near the lowest finite value still have their softmax."""
    import torch
    d, w = 128, 3
    L = S * w
    rng = np.random.default_rng(7600 + P + S + M)
    Hs, Hv = _store(rng.normal(size=(P, S, d)), dtype)
    ts, tv = _store(rng.normal(size=(P, d)), dtype)
    (wqs, wqv), (wks, wkv), (wvs, wvv) = (_store(rng.normal(size=(M, d, d)) / math.sqrt(d), dtype) for _ in range(3))
    dz = rng.normal(size=(P, d)).astype(np.float32)
    nv = np.full(P, S)
    nv[1], nv[8] = S // 2, 0
    for p, row, x in ((0, 0, np.nan), (1, S // 2 - 1, np.inf), (2, S // 2, -np.inf), (3, S - 1, np.nan), (4, 5, np.inf)):
        Hs[p, row, 7] = x if dtype == "f32" else {np.inf: 0x7f80, -np.inf: 0xff80}.get(x, 0x7fc0)
    # equal scores of one value, as in the forward test: past the range, and (pair 5) below -3e38 and finite
    unit = 1.0 if dtype == "f32" else 1.4426950408889634
    for p, x in ((5, -3.2e38), (6, -1e39)):
        ts[p], tv[p] = _store(1e10 * tv[p], dtype)
        r = wkv[0] @ (tv[p] @ wqv[0]) / math.sqrt(d)
        Hs[p], Hv[p] = _store(np.broadcast_to(x / unit * r / (r @ r), (S, d)), dtype)
    lens = (nv * w).astype(np.int32)
    print(f"P {P} S {S} M {M} {dtype}", flush=True)
    args = [to_device(x) for x in (Hs[:, None], ts[:, None], wqs, wks, wvs, lens, dz[:, None])]
    dseg, dt0 = laser.laser_gsta_backward(*args, L, w)[:2]
    torch.cuda.synchronize()
    dseg, dt0 = to_host_f64(dseg)[:, 0], to_host_f64(dt0)[:, 0]
    nans = (0, 1, 2, 3, 4, 6)
    for p in nans:
        assert np.isnan(dt0[p]).all() and np.isnan(dseg[p, :nv[p]]).all() and not dseg[p, nv[p]:].any(), p
    fine = [7, 8, 9, 10, P - 1]
    cnt = oracle.segment_counts(lens[fine], L, w)
    ref = oracle.gsta_backward(Hv[fine][:, None], tv[fine][:, None], wqv, wkv, wvv, cnt, dz[fine][:, None].astype(np.float64))
    assert vec_rel_err(dseg[fine], ref[0][:, 0]) <= TOL[dtype]
    assert vec_rel_err(dt0[fine], ref[1][:, 0]) <= 1e-5
    others = np.delete(np.arange(P), nans + (5,))
    assert np.isfinite(dt0[others]).all() and np.isfinite(dseg[others]).all()
    if M == 1:
        # pair 5: p is its one row, whose outer product with dz (1e28 times every other pair's) is dW_v. (Its score gradients
        # are differences of numbers of that size, so nothing is said about the others.)
        lens[list(nans)] = 0
        args[5] = to_device(lens)
        dwv = to_host_f64(laser.laser_gsta_backward(*args, L, w)[4])[0]
        ref = np.outer(Hv[5, 0], dz[5].astype(np.float64))
        assert vec_rel_err(dwv.reshape(1, -1), ref.reshape(1, -1)) <= 1e-5


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("P", [12, 300, 600, 1100, 2100])
def test_pairs_without_a_segment_add_nothing_to_the_weight_gradients(P, dtype):
    """Whatever their target and upstream gradient hold: the latter passes through to dt0 and that is all."""
    import torch
    d, S, M = 128, 5, 2
    rng = np.random.default_rng(7700 + P)
    Hs, _ = _store(rng.normal(size=(P, 1, S, d)), dtype)
    ts, _ = _store(rng.normal(size=(P, 1, d)), dtype)
    W = [to_device(_store(rng.normal(size=(M, d, d)) / math.sqrt(d), dtype)[0]) for _ in range(3)]
    dz = rng.normal(size=(P, 1, d)).astype(np.float32)
    lens = np.full(P, S, dtype=np.int32)
    lens[3] = lens[8] = 0
    print(f"P {P} {dtype}", flush=True)
    call = lambda: laser.laser_gsta_backward(to_device(Hs), to_device(ts), *W, to_device(lens), to_device(dz), S, 1)
    plain = call()
    ts[3, 0, 7] = np.nan if dtype == "f32" else 0x7fc0
    dz[8, 0, 9] = np.inf
    got = call()
    torch.cuda.synchronize()
    for a, b in zip(got[2:], plain[2:]):
        assert torch.equal(a, b)
    assert torch.equal(got[1], to_device(dz).where(to_device(lens == 0)[:, None, None], got[1]))
