"""What users of the library run, as measurable cases.

Six paths through the public entry points:
  forward   a batch of requests with stored keys and values: laser_forward (STA, then M layers of GSTA)
  packed    the same with each request's own number of candidates: laser_forward_ragged
  head      the complete ranking head from raw embeddings: projections, STA with heads, then FFN + LayerNorm + GSTA and
            the two other views from one call
  folded    raw embeddings to H' without forming keys and values, then GSTA (few targets per user)
  train     forward and backward of both attention steps: every gradient the library computes
Sizes are those of the benchmark workloads and of the paper's own setting (L = 1000, w = 10, d = 128, d_q = 32), beside
single requests, odd sizes and single precision. `lens` names the distribution of the history lengths: "full",
"uniform" in [L / 5, L] or "log" (log-uniform in [L / 64, L]).
"""
import math

import torch

import paper_2602_11562_amd as laser

BF16, F32 = "bf16", "f32"


# ------------------------------------------------------------------------------------------------ cases
def _forward(dtype, U, C, L, w, d, d_q, M, lens):
    return {"path": "forward", "dtype": dtype, "U": U, "C": C, "L": L, "w": w, "d": d, "d_q": d_q, "M": M, "lens": lens}


def _packed(U, C, L, w, d, d_q, M, lens):
    return {"path": "packed", "dtype": BF16, "U": U, "C": C, "L": L, "w": w, "d": d, "d_q": d_q, "M": M, "lens": lens}


def _head(U, C, L, w, heads, d_ff, r, M, lens):
    return {"path": "head", "dtype": BF16, "U": U, "C": C, "L": L, "w": w, "d": 128, "d_q": 32, "heads": heads,
            "d_ff": d_ff, "r": r, "M": M, "lens": lens}


def _folded(U, C, L, w, heads, M, lens):
    return {"path": "folded", "dtype": BF16, "U": U, "C": C, "L": L, "w": w, "d": 128, "d_q": 32, "heads": heads, "M": M,
            "lens": lens}


def _train(U, C, L, w, d, d_q, M, grads_bf16, lens):
    return {"path": "train", "dtype": BF16, "U": U, "C": C, "L": L, "w": w, "d": d, "d_q": d_q, "M": M,
            "grads_bf16": grads_bf16, "lens": lens}


def listed():
    return [
        # one small request in single precision: latency and launches
        dict(_forward(F32, 1, 16, 1024, 64, 64, 64, 1, "full"), name="request_f32"),
        # one request of ordinary size at the paper's dimensions and depth
        dict(_forward(BF16, 1, 100, 1000, 10, 128, 32, 2, "full"), name="request_bf16"),
        # a serving batch with histories of different lengths
        dict(_forward(BF16, 64, 64, 2048, 128, 64, 64, 1, "uniform"), name="batch_bf16"),
        # many candidates for each of a few users: the configuration the benchmark quotes
        dict(_forward(BF16, 32, 256, 4096, 128, 128, 128, 1, "full"), name="high_fanout"),
        # one candidate for each of many users: the history is streamed
        dict(_forward(BF16, 4096, 1, 4096, 256, 64, 64, 1, "log"), name="low_fanout"),
        # lifelong histories, two layers, a short last segment
        dict(_forward(BF16, 16, 128, 10000, 256, 128, 128, 2, "full"), name="lifelong"),
        # offline scoring in single precision, odd counts
        dict(_forward(F32, 24, 50, 1500, 100, 64, 64, 2, "uniform"), name="batch_f32"),
        # each request brings its own number of candidates; sizes that are no multiple of anything
        dict(_packed(29, 201, 3001, 100, 128, 128, 1, "uniform"), name="packed_odd"),
        # ranking from raw embeddings with the complete head, at the paper's dimensions
        dict(_head(64, 256, 1000, 10, 2, 128, 8, 1, "uniform"), name="ranking_head"),
        # the paper's training batch seen by a scorer: one target per user, raw embeddings
        dict(_folded(2048, 1, 1000, 10, 2, 1, "uniform"), name="folded_scoring"),
        # the paper's training batch: one target per sample, gradients of the history in bf16
        dict(_train(2048, 1, 1000, 10, 128, 32, 1, True, "uniform"), name="train_single"),
        # training on whole requests: all shown candidates of a user share one pass over the history
        dict(_train(64, 64, 2048, 128, 64, 64, 1, False, "uniform"), name="train_grouped"),
    ]


def _log(rng, lo, hi):
    """An integer spread evenly over the logarithm of [lo, hi]."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["request", "batch", "fanout", "few", "f32", "packed", "head", "folded", "single", "grouped"])
    lens = rng.choice(["full", "uniform", "uniform"])
    d, d_q = rng.choice([(64, 64), (128, 32), (128, 64), (128, 128)])
    while True:
        if kind == "request":
            c = _forward(rng.choice([F32, BF16]), rng.randint(1, 4), _log(rng, 1, 200), _log(rng, 60, 2048),
                         _log(rng, 8, 128), d, d_q, rng.randint(1, 3), "full")
        elif kind == "batch":
            c = _forward(BF16, _log(rng, 8, 128), _log(rng, 9, 128), _log(rng, 500, 5000), _log(rng, 10, 256), d, d_q,
                         rng.choice([1, 1, 2]), lens)
        elif kind == "fanout":
            c = _forward(BF16, _log(rng, 8, 48), _log(rng, 129, 512), _log(rng, 1000, 10000), _log(rng, 32, 256), d, d_q,
                         rng.choice([1, 1, 2]), lens)
        elif kind == "few":
            c = _forward(BF16, _log(rng, 256, 4096), _log(rng, 1, 8), _log(rng, 500, 8192), _log(rng, 10, 512), d, d_q,
                         1, rng.choice(["full", "uniform", "log"]))
        elif kind == "f32":
            c = _forward(F32, _log(rng, 4, 48), _log(rng, 9, 96), _log(rng, 400, 2500), _log(rng, 16, 160), d, d_q,
                         rng.choice([1, 1, 2]), lens)
        elif kind == "packed":
            c = _packed(_log(rng, 8, 64), _log(rng, 16, 300), _log(rng, 800, 5000), _log(rng, 32, 256), d, d_q,
                        rng.choice([1, 1, 2]), lens)
        elif kind == "head":
            c = _head(_log(rng, 8, 96), _log(rng, 24, 320), _log(rng, 300, 1500), _log(rng, 8, 64), rng.choice([1, 2]),
                      rng.choice([64, 128]), rng.randint(1, 8), 1, lens)
        elif kind == "folded":
            c = _folded(_log(rng, 128, 2048), 1, _log(rng, 300, 1500), _log(rng, 8, 100), rng.choice([1, 2]), 1, lens)
        elif kind == "single":
            c = _train(_log(rng, 128, 2048), _log(rng, 1, 4), _log(rng, 300, 1500), _log(rng, 8, 100), d, d_q,
                       rng.choice([1, 1, 2]), rng.choice([True, True, False]), lens)
        else:
            c = _train(_log(rng, 8, 96), _log(rng, 9, 96), _log(rng, 400, 2500), _log(rng, 16, 160), d, d_q,
                       rng.choice([1, 1, 2]), False, lens)
        c["r"] = min(c["r"], -(-c["L"] // c["w"])) if "r" in c else 0
        if not c["r"]:
            del c["r"]
        if _fits(kind, c):
            return c


def _fits(kind, c):
    """A drawn case costs no more than the largest listed one, and its tensors have fewer than 2^31 elements."""
    inner = c["U"] * c["C"] * c["L"] * (c["d"] + c["d_q"])       # multiply-adds of the attention over items
    most = {"f32": 24 * 50 * 1500 * 128 * 4, "grouped": 64 * 64 * 2048 * 128, "single": 2048 * 1000 * 160 * 2}
    pairs_rows = c["U"] * c["C"] * -(-c["L"] // c["w"])
    return inner <= most.get(kind, 1 << 62) and work(c)["bytes"] <= 1.0e9 and work(c)["flops"] <= 4e10 and \
        pairs_rows <= 1_700_000


# ------------------------------------------------------------------------------------------------ inputs
def _lens(c, gen):
    U, L = c["U"], c["L"]
    if c["lens"] == "full":
        return torch.full((U,), L, dtype=torch.int32, device="cuda")
    x = torch.rand(U, device="cuda", generator=gen)
    lo = max(1, L // 5) if c["lens"] == "uniform" else max(1, L // 64)
    n = lo + x * (L + 1 - lo) if c["lens"] == "uniform" else lo * torch.exp(x * math.log((L + 1) / lo))
    return n.floor().clamp(lo, L).to(torch.int32)


def _mean_len(c):
    L = c["L"]
    if c["lens"] == "full":
        return float(L)
    lo = max(1, L // 5) if c["lens"] == "uniform" else max(1, L // 64)
    return (lo + L) / 2 if c["lens"] == "uniform" else (L - lo) / max(1e-9, math.log((L + 1) / lo)) if L > lo else L


def _counts(c):
    """Candidates of each user: between one and the largest count, one user without any (the seed deals them out)."""
    counts = torch.randint(1, c["C"] + 1, (c["U"],), generator=torch.Generator().manual_seed(c["U"] * c["C"]))
    counts[0], counts[1] = 0, c["C"]
    return counts


def prepare(case, seed):
    c = dict(case)
    U, C, L, w, d, d_q, M = (c[n] for n in ("U", "C", "L", "w", "d", "d_q", "M"))
    S = -(-L // w)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.float32 if c["dtype"] == F32 else torch.bfloat16

    def rnd(*shape, sd=1.0, dtype=dt):
        return (torch.randn(*shape, device="cuda", generator=gen) * sd).to(dtype)

    def out(*shape, dtype=dt):
        return torch.empty(*shape, device="cuda", dtype=dtype)

    f32 = torch.float32
    s = {"case": c, "w": w, "L": L, "lens": _lens(c, gen)}
    s["gsta"] = [rnd(M, d, d, sd=d ** -0.5) for _ in range(3)]
    if c["path"] in ("head", "folded"):
        heads, d_in = c["heads"], 128
        s["gamma"] = math.sqrt(d_q / heads)
        s["t"], s["h"] = rnd(U, C, d_in), rnd(U, L, d_in)
        s["w_q"], s["w_k"], s["w_v"] = (rnd(d_in, n, sd=d_in ** -0.5) for n in (d_q, d_q, d))
        s["seg"], s["z"] = out(U, C, S, d), out(U, C, d, dtype=f32)
        if c["path"] == "folded":
            s["a_fold"] = laser.laser_fold_query_weights(s["w_q"], s["w_k"], heads)
            s["qf"], s["g"] = out(U, C * heads, d_in), out(U, C * heads, S, d_in)
        else:
            d_ff = c["d_ff"]
            s["q"], s["k"], s["v"] = out(U, C, d_q), out(U, L, d_q), out(U, L, d)
            s["ffn"] = [rnd(d, d_ff, sd=d ** -0.5), rnd(d_ff, sd=0.3, dtype=f32), rnd(d_ff, d, sd=d_ff ** -0.5),
                        rnd(d, sd=0.3, dtype=f32), 1.0 + rnd(d, sd=0.2, dtype=f32), rnd(d, sd=0.1, dtype=f32)]
            s["pool"], s["recent"] = out(U, C, d), out(U, C, c["r"], d)
        return s
    s["gamma"] = math.sqrt(d_q)
    if c["path"] == "packed":
        counts = _counts(c)[torch.randperm(U, generator=torch.Generator().manual_seed(seed))]
        s["P"] = int(counts.sum())
        s["off"] = torch.cat([torch.zeros(1, dtype=torch.int64), counts.cumsum(0)]).to(torch.int32).cuda()
        s["q"] = rnd(s["P"], d_q, sd=d_q ** -0.5)
        s["t0"] = rnd(s["P"], d, sd=d ** -0.5)
        s["seg"], s["z"] = out(s["P"], S, d), out(s["P"], d, dtype=f32)
    else:
        s["q"] = rnd(U, C, d_q, sd=d_q ** -0.5)
        s["t0"] = rnd(U, C, d, sd=d ** -0.5)
        s["seg"], s["z"] = out(U, C, S, d), out(U, C, d, dtype=f32)
    s["k"], s["v"] = rnd(U, L, d_q, sd=d_q ** -0.5), rnd(U, L, d, sd=d ** -0.5)
    if c["path"] != "packed" and L > 20:      # one item in twenty resembles a candidate of its user
        at = torch.arange(0, L, 20, device="cuda")
        of = torch.randint(0, C, (U, at.numel()), device="cuda", generator=gen)
        like = torch.gather(s["q"], 1, of[:, :, None].expand(-1, -1, d_q)).float()
        s["k"][:, at] = (0.8 * like + 0.6 * s["k"][:, at].float()).to(dt)
    s["cnt"] = out(U, S, dtype=torch.int32)
    if c["path"] == "train":
        gdt = dt if c["grads_bf16"] else f32
        s["dz"] = rnd(U, C, d, dtype=f32)
        s["dq"], s["dk"], s["dv"] = out(U, C, d_q, dtype=f32), out(U, L, d_q, dtype=gdt), out(U, L, d, dtype=gdt)
        lib = laser.load_library()
        s["sta_work"] = out(max(16, lib.laser_sta_backward_work_bytes(U, C, L, d_q, w)), dtype=torch.uint8)
        s["gsta_work"] = out(max(16, lib.laser_gsta_backward_work_bytes(U, C, d, M)), dtype=torch.uint8)
    return s


# ------------------------------------------------------------------------------------------------ one pass
def run(s):
    c, w, gamma, lens = s["case"], s["w"], s["gamma"], s["lens"]
    path = c["path"]
    if path == "forward":
        return laser.laser_forward(s["q"], s["k"], s["v"], s["t0"], *s["gsta"], lens, w, gamma, seg_out=s["seg"],
                                   seg_cnt=s["cnt"], z_out=s["z"])
    if path == "packed":
        return laser.laser_forward_ragged(s["q"], s["k"], s["v"], s["t0"], *s["gsta"], lens, s["off"], c["C"], w, gamma,
                                          seg_out=s["seg"], seg_cnt=s["cnt"], z_out=s["z"])
    if path == "head":
        laser.laser_project_q_forward(s["t"], s["w_q"], q_out=s["q"])
        laser.laser_project_kv_forward(s["h"], s["w_k"], s["w_v"], k_out=s["k"], v_out=s["v"])
        laser.laser_sta_forward(s["q"], s["k"], s["v"], lens, w, gamma, seg_out=s["seg"], want_cnt=False,
                                heads=c["heads"])
        _, z, pool, recent = laser.laser_ffn_gsta_forward(s["seg"], s["t"], *s["gsta"], lens, *s["ffn"], s["L"], w,
                                                          z_out=s["z"], want_seg=False, r=c["r"], pool_out=s["pool"],
                                                          recent_out=s["recent"])
        return z, pool, recent
    if path == "folded":
        seg, _ = laser.laser_sta_folded_forward(s["t"], s["h"], s["a_fold"], s["w_v"], lens, w, gamma, c["heads"],
                                                qf_work=s["qf"], g_work=s["g"], seg_out=s["seg"], want_cnt=False)
        return seg, laser.laser_gsta_forward(seg, s["t"], *s["gsta"], lens, s["L"], w, z_out=s["z"])
    seg, _, z = laser.laser_forward(s["q"], s["k"], s["v"], s["t0"], *s["gsta"], lens, w, gamma, seg_out=s["seg"],
                                    z_out=s["z"], want_cnt=False)
    dseg, dt0, dwq, dwk, dwv = laser.laser_gsta_backward(seg, s["t0"], *s["gsta"], lens, s["dz"], s["L"], w,
                                                         work=s["gsta_work"])
    dq, dk, dv = laser.laser_sta_backward(s["q"], s["k"], s["v"], lens, dseg, w, gamma, dq_out=s["dq"], dk_out=s["dk"],
                                          dv_out=s["dv"], work=s["sta_work"], grads_bf16=c["grads_bf16"])
    return z, dt0, dwq, dwk, dwv, dq, dk, dv


# ------------------------------------------------------------------------------------------------ accounting
def work(case):
    """Inputs read once and outputs written once; two operations per multiply-add, over valid items and segments."""
    c = case
    U, C, L, w, d, d_q, M = (c[n] for n in ("U", "C", "L", "w", "d", "d_q", "M"))
    e = 4 if c["dtype"] == F32 else 2
    S, n = -(-L // w), _mean_len(c)
    sv = min(S, n / w + (0.5 if c["lens"] != "full" else 0.0))
    pairs = int(_counts(c).sum()) if c["path"] == "packed" else U * C
    weights = 3 * M * d * d * e
    sta = 2.0 * pairs * n * (d_q + d)
    gsta = 2.0 * M * pairs * (3 * d * d + 2 * sv * d)
    if c["path"] in ("forward", "packed"):
        return {"bytes": U * n * (d_q + d) * e + pairs * (d_q + d) * e + weights + pairs * S * d * e + pairs * d * 4
                + U * S * 4, "flops": sta + gsta}
    if c["path"] == "head":
        d_in, d_ff, r = 128, c["d_ff"], c["r"]
        ffn = 4.0 * pairs * sv * d * d_ff
        project = 2.0 * (U * n * d_in * (d_q + d) + pairs * d_in * d_q)
        return {"bytes": U * n * d_in * e + pairs * d_in * e + weights + (d_in * (2 * d_q + d) + 2 * d * d_ff) * e
                + pairs * d * (4 + e) + pairs * r * d * e, "flops": project + sta + ffn + gsta}
    if c["path"] == "folded":
        d_in, heads = 128, c["heads"]
        return {"bytes": U * n * d_in * e + pairs * d_in * e + weights + pairs * S * d * e + pairs * d * 4,
                "flops": 2.0 * pairs * heads * (d_in * d_in + 2 * n * d_in) + 2.0 * pairs * S * d_in * d + gsta}
    g = 2 if c["grads_bf16"] else 4
    back = 2.0 * pairs * n * (2 * d + 3 * d_q) + 2.0 * M * pairs * (8 * d * d + 6 * sv * d)
    return {"bytes": U * n * (d_q + d) * e + pairs * (d_q + d) * e + weights + U * L * (d_q + d) * g
            + pairs * (2 * d * 4 + d_q * 4 + d * 4) + 3 * M * d * d * 4, "flops": sta + gsta + back}


def tolerance(case):
    """About four times what each path differs by from the same path in 64 bits without any rounding in between, over the
    listed and a few dozen drawn cases: 3e-7 in single precision; in bf16 2.5e-3 (the gates and H' are rounded once each),
    and up to 3.7e-3 where more intermediates are stored in bf16 (transformed rows, folded queries and sums, dH')."""
    if case["dtype"] == F32:
        return {"rel": 1.2e-6, "max": 1e-5}
    if case["path"] in ("forward", "packed"):
        return {"rel": 1e-2, "max": 0.06}
    return {"rel": 1.4e-2, "max": 0.25 if case["path"] == "train" else 0.15}
