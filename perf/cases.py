"""The work that a user of this library has it do, as timed cases: attention forward and training
steps in bf16 and fp32, grouped heads, ring steps, per-chunk partials with their merge, the backward
through stored dS, and the multi-fidelity tokenizer.

A case is a dict of plain values.  `listed()` gives the named ones, `draw(rng)` others of the same
ranges, `prepare(case, seed)` the tensors a program holds before the call, `run(state)` one pass
through the public entry points, `exact(case, seed)` the same results in 64 bits.
"""

import math

import torch

from paper_2507_16697_amd import ring, ringx

DEVICE = "cuda"


# ------------------------------------------------------------------------------------------------
# cases


def _attn(name, dtype, B, H, Nq, Nk, d, R, bwd, Hkv=None, tokens="iid"):
    return {"name": name, "kind": "attn", "dtype": dtype, "B": B, "H": H, "Hkv": Hkv or H, "Nq": Nq,
            "Nk": Nk, "d": d, "R": R, "bwd": bwd, "tokens": tokens}


def listed():
    return [
        # a smoke test, a unit test or the first layers of a toy model: one tiny training step,
        # a few microseconds of work behind four kernel launches
        _attn("tiny_step", "bf16", 1, 2, 200, 700, 128, 3, True),
        # the exactness workload: the fp32 forward on 1024 tokens, as used to validate a pipeline
        _attn("fp32_n1k", "fp32", 1, 2, 1024, 1024, 64, 4, False),
        # an fp32 reference training step at sizes and a head dim that fit no tile
        _attn("fp32_ragged_step", "fp32", 1, 3, 1531, 3001, 100, 5, True),
        # a training step over one 16^3 token grid, 16 heads of 64
        _attn("grid16_step", "bf16", 1, 16, 4096, 4096, 64, 1, True),
        # inference over a batch of short sequences (about 2K tokens each, 6 heads of 64, odd
        # length), on spatially correlated tokens
        _attn("batch_forward", "bf16", 8, 6, 2001, 2001, 64, 1, False, tokens="smooth"),
        # a training step over one 32 x 32 x 16 token grid in 4 chunks
        _attn("shard16k_step", "bf16", 1, 16, 16384, 16384, 64, 4, True),
        # grouped-query training step (4 query heads per K/V head), ragged sizes and chunks
        _attn("gqa_step", "bf16", 2, 16, 3000, 10007, 128, 3, True, Hkv=4),
        # one rank's training step of an 8-way ring over a 64^3 token grid: the headline workload
        _attn("ring8_step", "bf16", 1, 16, 32768, 262144, 128, 8, True),
        # the same kind of step taken one ring step at a time, the next chunk arriving meanwhile:
        # 6 heads of 64, 8 chunks of unequal length
        {"name": "ring_steps", "kind": "ring", "B": 1, "H": 6, "Nq": 8192, "Nk": 65601, "d": 64,
         "R": 8},
        # a rank that serves another rank's queries: per-chunk fp32 partials, then their merge
        {"name": "partials_merge", "kind": "partials", "B": 1, "H": 16, "Nq": 2048, "Nk": 32768,
         "d": 128, "R": 8},
        # the backward of a program with memory to spare: dQ from stored dS
        {"name": "stored_ds", "kind": "stored_ds", "B": 1, "H": 8, "Hkv": 8, "Nq": 4096,
         "Nk": 16384, "d": 128, "R": 4},
        # the three fidelity modes of one 512^3 snapshot with 4 channels, patch 2, to bf16 tokens;
        # the centre puts the crops off any alignment
        {"name": "tokenize_512", "kind": "tokenize", "C": 4, "D": 512, "p": 2, "cz": 301, "cy": 77,
         "cx": 203, "k0": 1, "k1": 4, "k2": 8, "dtype": "bf16"},
    ]


def _log(rng, lo, hi):
    """An integer whose logarithm is uniform over [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "forward", "gqa", "fp32", "fp32", "ring", "partials",
                       "stored_ds", "tokenize"])
    if kind in ("step", "forward", "gqa"):
        d = rng.choice([64, 128])
        B = rng.choice([1, 1, 2, 4])
        Hkv = rng.choice([1, 2, 4]) if kind == "gqa" else rng.choice([2, 3, 6, 16])
        H = Hkv * rng.choice([2, 4, 8]) if kind == "gqa" else Hkv
        # a rank's queries are between all of the sequence and an eighth of it
        Nq = _log(rng, 100, 16384)
        Nk = int(Nq * math.exp(rng.uniform(0.0, math.log(8.0))))
        R = min(Nk, rng.choice([1, 2, 3, 4, 8]))
        tokens = rng.choice(["iid", "smooth"]) if kind == "forward" else "iid"
        c = _attn(None, "bf16", B, H, Nq, Nk, d, R, kind != "forward", Hkv=Hkv, tokens=tokens)
    elif kind == "fp32":
        d = rng.choice([16, 32, 64, 100, 128, rng.randint(1, 128)])
        H = rng.choice([1, 2, 3, 4])
        Nq = _log(rng, 64, 1531)
        Nk = _log(rng, 64, 3001)
        R = min(Nk, rng.choice([1, 2, 4, 5, 8]))
        c = _attn(None, "fp32", 1, min(H, 3) if d > 64 else H, Nq, Nk, d, R, rng.random() < 0.5)
    elif kind == "ring":
        Nq = _log(rng, 512, 16384)
        R = rng.choice([2, 4, 8])
        c = {"kind": "ring", "B": rng.choice([1, 2]), "H": rng.choice([2, 3, 6]), "Nq": Nq,
             "Nk": Nq * R + rng.randint(0, 200), "d": rng.choice([64, 128]), "R": R}
    elif kind == "partials":
        Nq = _log(rng, 256, 4096)
        R = rng.choice([2, 4, 8])
        c = {"kind": "partials", "B": rng.choice([1, 2]), "H": rng.choice([3, 6, 16]), "Nq": Nq,
             "Nk": Nq * rng.choice([1, 4, 16]) + rng.randint(0, 100), "d": rng.choice([64, 128]),
             "R": R}
    elif kind == "stored_ds":
        Hkv = rng.choice([1, 2, 4, 8])
        Nq = _log(rng, 512, 8192)
        c = {"kind": "stored_ds", "B": 1, "H": Hkv * rng.choice([1, 2]), "Hkv": Hkv, "Nq": Nq,
             "Nk": Nq * rng.choice([1, 2, 4]) + rng.randint(0, 100), "d": 128,
             "R": rng.choice([1, 2, 4])}
    else:
        D = rng.choice([128, 256, 512])
        p = rng.choice([1, 2])
        k0, k1, k2 = rng.choice([(1, 4, 8), (2, 8, 16)]) if p == 1 else (1, 4, 8)
        c = {"kind": "tokenize", "C": rng.choice([1, 3, 4]), "D": D, "p": p,
             "cz": rng.randrange(D), "cy": rng.randrange(D), "cx": rng.randrange(D), "k0": k0,
             "k1": k1, "k2": k2, "dtype": rng.choice(["bf16", "fp32"])}
    c.pop("name", None)
    return c


# ------------------------------------------------------------------------------------------------
# inputs


def _scale(c):
    return 1.0 / math.sqrt(c["d"])


def _std(c):
    """Spread of Q, K, V and of dO, as in the library's workloads."""
    if c.get("dtype") == "fp32":
        return 1.0, 1.0
    return (0.5, 1.0) if c["d"] == 64 else (2 ** -0.5, 2 ** -0.5)


def _gen(seed):
    return torch.Generator(device=DEVICE).manual_seed(int(seed))


def _randn(gen, shape, std, dtype):
    return torch.randn(shape, generator=gen, device=DEVICE, dtype=torch.float32).mul_(std).to(dtype)


def _smooth_qkv(c, gen):
    """Q, K, V of spatially correlated tokens: a random-phase field with a decaying spectrum on a
    3D grid, embedded, layer-normalised and projected."""
    B, H, d = c["B"], c["H"], c["d"]
    n, modes, width = max(c["Nq"], c["Nk"]), 64, H * d
    side = int(math.ceil(n ** (1.0 / 3.0)))
    t = torch.arange(n, device=DEVICE)
    pos = torch.stack([t % side, t // side % side, t // (side * side)], 1).float() / side
    mag = 1.0 + 15.0 * torch.rand((B, modes, 1), generator=gen, device=DEVICE) ** 2
    way = torch.randn((B, modes, 3), generator=gen, device=DEVICE)
    way = way / way.norm(dim=2, keepdim=True)
    phase = 2 * math.pi * torch.rand((B, 1, modes), generator=gen, device=DEVICE)
    out = {x: [] for x in "qkv"}
    emb = torch.randn((modes, width), generator=gen, device=DEVICE) / math.sqrt(modes)
    proj = {x: torch.randn((width, width), generator=gen, device=DEVICE) / math.sqrt(width)
            for x in "qkv"}
    for b in range(B):
        f = torch.sin(2 * math.pi * (pos @ (mag[b] * way[b]).t().contiguous()) + phase[b])
        x = (f * mag[b].reshape(1, modes) ** (-5.0 / 6.0)) @ emb
        x = torch.nn.functional.layer_norm(x, (width,))
        for name, rows in (("q", c["Nq"]), ("k", c["Nk"]), ("v", c["Nk"])):
            y = (x[:rows] @ proj[name]).to(torch.bfloat16)
            out[name].append(y.reshape(rows, H, d).transpose(0, 1).contiguous())
    return [torch.stack(out[x]) for x in "qkv"]


def _qkv(c, gen):
    dtype = torch.float32 if c.get("dtype") == "fp32" else torch.bfloat16
    if c.get("tokens") == "smooth":
        return _smooth_qkv(c, gen)
    std = _std(c)[0]
    kv = (c["B"], c.get("Hkv", c["H"]), c["Nk"], c["d"])
    return [_randn(gen, (c["B"], c["H"], c["Nq"], c["d"]), std, dtype),
            _randn(gen, kv, std, dtype), _randn(gen, kv, std, dtype)]


def _bounds(c):
    return [ringx.ringx_chunk_bounds(c["Nk"], c["R"], r) for r in range(c["R"])]


def _modes(c):
    """(filter, size ratio) of the three fidelity modes."""
    return [(c["k0"], 8), (c["k1"], 2), (c["k2"], 1)]


def prepare(case, seed):
    c, gen = case, _gen(seed)
    s = {"case": c}
    if c["kind"] == "tokenize":
        s["field"] = _randn(gen, (c["C"], c["D"], c["D"], c["D"]), 1.0, torch.float32)
        return s
    s["q"], k, v = _qkv(c, gen)
    if c["kind"] == "ring":
        s["k"] = [k[:, :, lo:hi].contiguous() for lo, hi in _bounds(c)]
        s["v"] = [v[:, :, lo:hi].contiguous() for lo, hi in _bounds(c)]
    else:
        s["k"], s["v"] = k, v
    if c["kind"] in ("ring", "stored_ds") or c.get("bwd"):
        s["do"] = _randn(gen, s["q"].shape, _std(c)[1], s["q"].dtype)
    if c["kind"] == "stored_ds":
        # the backward's saved tensors
        fwd = ringx.ringx_attn_fwd if c["H"] == c["Hkv"] else ringx.ringx_attn_fwd_gqa
        s["out"], s["lse"] = fwd(s["q"], k, v, c["R"])
    return s


# ------------------------------------------------------------------------------------------------
# one pass


def run(state):
    s, c = state, state["case"]
    kind = c["kind"]
    if kind == "attn":
        if c["H"] == c["Hkv"]:
            out, lse = ringx.ringx_attn_fwd(s["q"], s["k"], s["v"], c["R"])
        else:
            out, lse = ringx.ringx_attn_fwd_gqa(s["q"], s["k"], s["v"], c["R"])
        if not c["bwd"]:
            return {"out": out, "lse": lse}
        bwd = ringx.ringx_attn_bwd if c["H"] == c["Hkv"] else ringx.ringx_attn_bwd_gqa
        dq, dk, dv = bwd(s["q"], s["k"], s["v"], out, s["do"], lse, c["R"])
        return {"out": out, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    if kind == "ring":
        out, lse = ring.ring_forward(s["q"], s["k"], s["v"])
        dq, dk, dv = ring.ring_backward(s["q"], s["k"], s["v"], out, s["do"], lse)
        return {"out": out, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    if kind == "partials":
        po, pl = ringx.ringx_attn_fwd_partials(s["q"], s["k"], s["v"], c["R"])
        out, lse = ringx.ringx_lse_merge(po, pl, out_dtype=torch.bfloat16)
        return {"part_out": po, "part_lse": pl, "out": out, "lse": lse}
    if kind == "stored_ds":
        dq, dk, dv = ringx.ringx_attn_bwd_ds(s["q"], s["k"], s["v"], s["out"], s["do"], s["lse"],
                                             c["R"])
        return {"dq": dq, "dk": dk, "dv": dv}
    dtype = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    centre = (c["cz"], c["cy"], c["cx"])
    return [ringx.ringx_tt_tokenize(s["field"], k, ratio, centre, c["p"], out_dtype=dtype)
            for k, ratio in _modes(c)]


# ------------------------------------------------------------------------------------------------
# what a pass cannot do without


def work(case):
    c = case
    if c["kind"] == "tokenize":
        es, n_in, n_out, flops = (2 if c["dtype"] == "bf16" else 4), 0, 0, 0
        for k, ratio in _modes(c):
            cells = c["C"] * (c["D"] // ratio) ** 3
            n_in += cells
            n_out += cells // k ** 3
            flops += 2 * cells if k > 1 else 0
        return {"bytes": 4 * n_in + es * n_out, "flops": flops}
    es = 4 if c.get("dtype") == "fp32" else 2
    rows, nq = c["B"] * c["H"] * c["Nq"], c["B"] * c["H"] * c["Nq"] * c["d"]
    nkv = c["B"] * c.get("Hkv", c["H"]) * c["Nk"] * c["d"]
    pairs = 2 * c["B"] * c["H"] * c["Nq"] * c["Nk"] * c["d"]       # one contraction
    fwd_bytes = es * (2 * nq + 2 * nkv) + 4 * rows                 # q, k, v, out, lse
    bwd_bytes = es * (3 * nq + 2 * nkv) + 4 * rows + 4 * nq + 8 * nkv
    if c["kind"] == "partials":
        return {"bytes": fwd_bytes + 4 * c["R"] * (nq + rows), "flops": 2 * pairs}
    if c["kind"] == "stored_ds":
        return {"bytes": bwd_bytes, "flops": 4 * pairs}
    if c["kind"] == "attn" and not c["bwd"]:
        return {"bytes": fwd_bytes, "flops": 2 * pairs}
    # a training step: q, k, v once, dO, the outputs and the gradients (out and lse stay inside)
    return {"bytes": fwd_bytes + es * nq + 4 * nq + 8 * nkv, "flops": 6 * pairs}


def tolerance(case):
    """Relative 2-norm differences between correct implementations."""
    if case["kind"] == "tokenize":
        # fp32 weighted sums of k^3 cells; bf16 tokens may round the other way at a tie
        return {"rel": 1e-3} if case["dtype"] == "bf16" else {"rel": 1e-6}
    if case.get("dtype") == "fp32":
        return {"rel": 1e-5}
    # P, dS and the stored output are rounded to bf16
    return {"rel": 1e-2}


# ------------------------------------------------------------------------------------------------
# the same results in 64 bits


def _exact_attn(q, k, v, do, scale, bounds=None):
    """Plain softmax attention and its gradients, one (batch, query head) at a time in row blocks;
    with `bounds`, also each chunk's own output and log-sum-exp."""
    B, H, Nq, d = q.shape
    Hkv, Nk = k.shape[1], k.shape[2]
    new = dict(dtype=torch.float64, device=q.device)
    r = {"out": torch.empty((B, H, Nq, d), **new), "lse": torch.empty((B, H, Nq), **new)}
    if do is not None:
        r["dq"] = torch.empty((B, H, Nq, d), **new)
        r["dk"] = torch.zeros((B, Hkv, Nk, d), **new)
        r["dv"] = torch.zeros((B, Hkv, Nk, d), **new)
    if bounds is not None:
        r["part_out"] = torch.empty((len(bounds), B, H, Nq, d), **new)
        r["part_lse"] = torch.empty((len(bounds), B, H, Nq), **new)
    step = max(16, min(Nq, (1 << 28) // Nk))
    for b in range(B):
        for h in range(H):
            m = h // (H // Hkv)
            kk, vv = k[b, m].double(), v[b, m].double()
            kt, vt = kk.t().contiguous(), vv.t().contiguous()
            for i in range(0, Nq, step):
                rows = slice(i, min(Nq, i + step))
                qq = q[b, h, rows].double()
                P = (qq @ kt).mul_(scale)
                for j, (lo, hi) in enumerate(bounds or []):
                    l = torch.logsumexp(P[:, lo:hi], 1)
                    r["part_lse"][j, b, h, rows] = l
                    r["part_out"][j, b, h, rows] = (P[:, lo:hi] - l[:, None]).exp_() @ vv[lo:hi]
                top = P.amax(1, keepdim=True)
                P.sub_(top).exp_()
                total = P.sum(1, keepdim=True)
                P.div_(total)
                o = P @ vv
                r["out"][b, h, rows] = o
                r["lse"][b, h, rows] = (top + total.log()).squeeze(1)
                if do is None:
                    continue
                dd = do[b, h, rows].double()
                r["dv"][b, m] += P.t() @ dd
                dS = (dd @ vt).sub_((dd * o).sum(1, keepdim=True)).mul_(P).mul_(scale)
                r["dq"][b, h, rows] = dS @ kk
                r["dk"][b, m] += dS.t() @ qq
    return r


def _exact_tokens(field, k, ratio, centre, p):
    C, D = field.shape[0], field.shape[1]
    n = D // ratio
    x = field
    for axis, at in enumerate(centre):
        idx = (torch.arange(n, device=field.device) + at - n // 2) % D
        x = x.index_select(axis + 1, idx)
    x = x.double()
    u = torch.arange(k, device=field.device, dtype=torch.float64) - (k - 1) / 2.0
    w = torch.exp(-u * u / (2.0 * (k / 2.0) ** 2))
    w = w / w.sum()
    g = n // k
    x = (x.reshape(C, n, n, g, k) * w).sum(-1)
    x = (x.reshape(C, n, g, k, g) * w[:, None]).sum(-2)
    x = (x.reshape(C, g, k, g, g) * w[:, None, None]).sum(-3)
    P = g // p
    x = x.reshape(C, P, p, P, p, P, p).permute(1, 3, 5, 0, 2, 4, 6)
    return x.reshape(P * P * P, C * p ** 3)


def exact(case, seed):
    c = case
    s = prepare(c, seed)
    if c["kind"] == "tokenize":
        centre = (c["cz"], c["cy"], c["cx"])
        return [_exact_tokens(s["field"], k, ratio, centre, c["p"]) for k, ratio in _modes(c)]
    k, v = s["k"], s["v"]
    if c["kind"] == "ring":
        k, v = torch.cat(k, 2), torch.cat(v, 2)
    bounds = _bounds(c) if c["kind"] == "partials" else None
    r = _exact_attn(s["q"], k, v, s.get("do"), _scale(c), bounds)
    if c["kind"] == "ring":
        for name in ("dk", "dv"):
            r[name] = [r[name][:, :, lo:hi].contiguous() for lo, hi in _bounds(c)]
    if c["kind"] == "stored_ds":
        del r["out"], r["lse"]
    return r
