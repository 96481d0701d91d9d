"""laser_forward through the binding's native marshalling and without it: the same results, and the same refusals."""
import types

import numpy as np
import pytest

import oracle

from parity_util import TOL, to_host_f64, vec_rel_err

pytestmark = pytest.mark.gpu

laser = pytest.importorskip("paper_2602_11562_amd")
binding = pytest.importorskip("paper_2602_11562_amd.binding")


def _state(dtype, lens=True):
    import torch
    U, C, L, d_q, d, w = 2, 5, 70, 32, 64, 16
    gen = torch.Generator(device="cuda").manual_seed(9)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=gen).to(dtype)
    a = [rnd(U, C, d_q), rnd(U, L, d_q), rnd(U, L, d), rnd(U, C, d), rnd(2, d, d), rnd(2, d, d), rnd(2, d, d),
         torch.tensor([70, 33], dtype=torch.int32, device="cuda") if lens else None, w, 4.0]
    out = dict(seg_out=rnd(U, C, 5, d), seg_cnt=torch.full((U, 5), -1, dtype=torch.int32, device="cuda"),
               z_out=torch.full((U, C, d), 7.0, device="cuda"))
    return a, out


def _call(monkeypatch, native, a, out, **kw):
    """What the call gives or raises, and how many times the native part took it."""
    import torch
    took = []
    real = binding._fast().forward

    def forward(*args):
        code = real(*args) if native else None
        took.append(code is not None)
        return code
    monkeypatch.setattr(binding, "_fast_module", types.SimpleNamespace(forward=forward))
    own = {k: v.clone() if v is not None else None for k, v in out.items()}
    torch.cuda.synchronize()     # (the call may be on another stream than the copies)
    try:
        r = laser.laser_forward(*a, **own, **kw)
        torch.cuda.synchronize()
    except Exception as e:
        r = type(e)
    monkeypatch.undo()
    return r, sum(took)


@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
@pytest.mark.parametrize("lens,count,stream", [(True, True, False), (False, False, False), (True, True, True)])
def test_native_and_plain_marshalling_agree(monkeypatch, dtype, lens, count, stream):
    import torch
    a, out = _state(getattr(torch, dtype), lens)
    kw = {} if count else {"want_cnt": False}
    if not count:
        out["seg_cnt"] = None
    if stream:
        kw["stream"] = torch.cuda.Stream()
    one, took = _call(monkeypatch, True, a, out, **kw)
    two, _ = _call(monkeypatch, False, a, out, **kw)
    assert took == 1
    for x, y, fill in zip(one, two, (out["seg_out"], out["seg_cnt"], out["z_out"])):
        assert (x is None and y is None) or torch.equal(x, y)
        assert x is None or not (x == fill).all(-1).any()     # (every row written, none left as it was)
    q, k, v, n = (x if x is None else to_host_f64(x) for x in (a[0], a[1], a[2], a[7]))
    seg, cnt = oracle.sta_forward(q, k, v, n, *a[8:])
    assert vec_rel_err(to_host_f64(one[0]), seg) <= TOL["f32" if dtype == "float32" else "bf16"]
    assert one[1] is None or np.array_equal(one[1].cpu().numpy(), cnt)


@pytest.mark.parametrize("at,change", [(0, lambda t: t.transpose(0, 1)), (1, lambda t: t.float()), (2, lambda t: t.cpu()),
                                       (7, lambda t: t.long()), (4, lambda t: t.transpose(1, 2)), (0, lambda t: t[0]),
                                       (8, lambda w: 0), (9, lambda g: 0.0), (9, lambda g: 4)],
                         ids=["q turned", "k fp32", "v on the host", "lens int64", "wq turned", "q of two axes", "w 0", "gamma 0", "gamma int"])
def test_other_forms_are_refused_or_taken_as_without_it(monkeypatch, at, change):
    import torch
    a, out = _state(torch.bfloat16)
    a[at] = change(a[at])
    one, _ = _call(monkeypatch, True, a, out)
    two, _ = _call(monkeypatch, False, a, out)
    if isinstance(two, type):
        assert one is two
    else:
        assert all(torch.equal(x, y) for x, y in zip(one, two))
