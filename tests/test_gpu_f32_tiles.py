"""The fp32 matrix-core kernels at the edges of their tiles (needs an MI355X): head dims around the
16- and 64-dim groups and of every alignment class, query and key counts around the 16-row blocks
and 64-key tiles, and every number of waves that share a block (1 for many rows, up to 8).

Bar: the library's fp32 bar, max abs 1e-5 against the fp64 oracle on N(0, 1) inputs (a score of 128
products is good to about 128 * 2^-24 = 8e-6 in the worst case and to a tenth of it in the mean).
"""

import math

import numpy as np
import pytest
import torch

import oracle
from oracle import attention_fp64 as oa
from paper_2507_16697_amd import ringx

from parity_util import TOL_F32, max_abs_err, random_case, to_device, to_host_f64

pytestmark = pytest.mark.gpu

# (H, Nq, Nk, d, R): ks = 1 needs 2048 blocks of 16 rows
CASES = [(1, 1, 1, 1, 1), (2, 15, 17, 3, 2), (1, 16, 64, 4, 1), (1, 17, 63, 16, 3),
         (2, 33, 129, 17, 4), (1, 64, 65, 20, 1), (1, 31, 128, 31, 2), (2, 48, 200, 47, 5),
         (1, 65, 511, 48, 1), (1, 40, 512, 60, 7), (1, 16, 513, 63, 2), (1, 80, 300, 64, 3),
         (2, 19, 90, 65, 2), (1, 50, 777, 79, 3), (1, 35, 260, 96, 1), (1, 100, 257, 100, 5),
         (1, 47, 144, 109, 2), (1, 18, 100, 112, 100), (1, 70, 150, 113, 3), (1, 66, 640, 127, 4),
         (2, 130, 190, 128, 3), (130, 257, 33, 24, 2), (64, 260, 70, 128, 1), (24, 300, 150, 37, 2)]


@pytest.mark.parametrize("H,Nq,Nk,d,R", CASES)
def test_tile_edges(H, Nq, Nk, d, R):
    t, x = random_case(61, 1, H, Nq, Nk, d, store="fp32")
    g = {key: to_device(val, "fp32") for key, val in t.items()}
    scale = float(np.float32(1 / math.sqrt(d)))
    out, lse = ringx.ringx_attn_fwd(g["q"], g["k"], g["v"], R, scale=scale)
    po, pl = ringx.ringx_attn_fwd_partials(g["q"], g["k"], g["v"], R, scale=scale)
    acc, acc_lse = torch.empty_like(out), torch.empty_like(lse)
    for r in range(R):
        lo, hi = ringx.ringx_chunk_bounds(Nk, R, r)
        if R <= 7:
            # clones: a chunk of one head is contiguous as it is, but rarely 16-byte aligned
            k_r, v_r = (g[n][:, :, lo:hi].clone(memory_format=torch.contiguous_format)
                        for n in ("k", "v"))
            ringx.ringx_attn_fwd_step(g["q"], k_r, v_r, acc, acc_lse, r == 0, scale=scale)
    dq, dk, dv = ringx.ringx_attn_bwd(g["q"], g["k"], g["v"], out, g["do"], lse, R, scale=scale)
    delta = ringx.ringx_bwd_preprocess(out, g["do"], lse)
    k2, v2 = ringx.ringx_attn_bwd_dkdv(g["q"], g["k"], g["v"], g["do"], lse, delta, R, scale=scale,
                                       dk=dk.clone(), dv=dv.clone(), accumulate_dkv=True)
    q2 = ringx.ringx_attn_bwd_dq(g["q"], g["k"], g["v"], g["do"], lse, delta, R, scale=scale)
    torch.cuda.synchronize()
    ro, rl = oracle.attention_chunked(x["q"], x["k"], x["v"], scale, R)
    rpo, rpl = oracle.attention_partials(x["q"], x["k"], x["v"], scale, R)
    rq, rk, rv = oracle.attention_bwd(x["q"], x["k"], x["v"], ro, x["do"], rl, scale)
    got = {"out": (out, ro), "lse": (lse, rl), "part_out": (po, rpo), "part_lse": (pl, rpl),
           "dq": (dq, rq), "dk": (dk, rk), "dv": (dv, rv), "dq alone": (q2, rq)}
    if R <= 7:
        got.update({"acc": (acc, ro), "acc_lse": (acc_lse, rl)})
    for name, (a, ref) in got.items():
        e = max_abs_err(to_host_f64(a), ref)
        assert e <= TOL_F32 * max(1.0, float(np.max(np.abs(ref)))), (name, e)
    # accumulating the same gradients once more doubles them, up to the addition's rounding
    for name, a, one in (("dk", k2, dk), ("dv", v2, dv)):
        assert max_abs_err(to_host_f64(a), 2 * to_host_f64(one)) <= \
            2.0 ** -22 * float(one.abs().max()) + 2 * TOL_F32, name


def test_rows_past_a_chunk_are_not_read_into_it():
    """An infinite V row and a NaN K row in one chunk leave the other chunks' partials finite and
    equal to those of clean inputs."""
    t, _ = random_case(62, 1, 2, 40, 150, 36, store="fp32")
    g = {key: to_device(val, "fp32") for key, val in t.items()}
    R = 3
    po, pl = ringx.ringx_attn_fwd_partials(g["q"], g["k"], g["v"], R)
    k, v = g["k"].clone(), g["v"].clone()
    v[:, :, 50] = math.inf       # first row of chunk 1, right after chunk 0's last block
    k[:, :, 99] = math.nan       # last row of chunk 1
    po2, pl2 = ringx.ringx_attn_fwd_partials(g["q"], k, v, R)
    torch.cuda.synchronize()
    for r in (0, 2):
        assert torch.equal(po[r], po2[r]) and torch.equal(pl[r], pl2[r])
    assert torch.isnan(po2[1]).all() and torch.isnan(pl2[1]).all()


@pytest.mark.parametrize("d", [24, 64, 128])
@pytest.mark.parametrize("Nq", [15, 16, 17, 40])
def test_gradients_of_masked_keys_are_zero(Nq, d):
    """Keys masked by a feature of -inf weigh nothing in any row (P = exp(-inf) = 0), so their dK and dV
    are exactly 0 and the other keys' those without them, at query counts that do and do not fill the
    last block of 16."""
    H, Nk, live = 2, 70, 50
    t, x = random_case(63, 1, H, Nq, Nk, d, store="fp32")
    g = {key: to_device(val, "fp32") for key, val in t.items()}
    q, k, v, do = g["q"], g["k"], g["v"], g["do"]
    q[..., 0], k[..., 0], k[:, :, live:, 0] = 1.0, 0.0, -math.inf
    x["q"][..., 0], x["k"][..., 0] = 1.0, 0.0
    scale = float(np.float32(d ** -0.5))
    out, lse = ringx.ringx_attn_fwd(q, k, v, 2, scale=scale)
    delta = ringx.ringx_bwd_preprocess(out, do, lse)
    new = dict(dtype=torch.float32, device="cuda")
    noalloc = [torch.empty((1, H, n, d), **new) for n in (Nq, Nk, Nk)]
    step = [torch.empty((1, H, n, d), **new) for n in (Nq, Nk, Nk)]
    got = {"bwd": ringx.ringx_attn_bwd(q, k, v, out, do, lse, 2, scale=scale)[1:],
           "gqa": ringx.ringx_attn_bwd_gqa(q, k, v, out, do, lse, 2, scale=scale)[1:],
           "dkdv": ringx.ringx_attn_bwd_dkdv(q, k, v, do, lse, delta, 2, scale=scale),
           "noalloc": ringx.ringx_attn_bwd_noalloc(q, k, v, out, do, lse, 2, *noalloc,
                                                   scale=scale)[1:],
           "step": ringx.ringx_attn_bwd_step(q, k, v, do, lse, delta, *step, accumulate_dq=False,
                                             scale=scale)[1:]}
    torch.cuda.synchronize()
    kl, vl = x["k"][:, :, :live], x["v"][:, :, :live]
    ro, rl = oracle.attention(x["q"], kl, vl, scale)
    _, rk, rv = oracle.attention_bwd(x["q"], kl, vl, ro, x["do"], rl, scale)
    for name, (dk, dv) in got.items():
        assert bool((dk[:, :, live:] == 0).all()) and bool((dv[:, :, live:] == 0).all()), name
        for a, ref in ((dk, rk), (dv, rv)):
            e = max_abs_err(to_host_f64(a)[:, :, :live], ref)
            assert e <= TOL_F32 * max(1.0, float(np.max(np.abs(ref)))), (name, e)


@pytest.mark.parametrize("H,Nq,Nk,d", [(3, 1531, 3001, 100), (1, 2000, 16, 8),
                                       (6, 40, 1500, 33), (4, 700, 1100, 64)])
def test_stages_compose_bitwise(H, Nq, Nk, d):
    """The whole backward is its stages bit for bit also where the number of 16-row blocks decides how
    many waves share one, and so the order of the sums: each half alone as in the common launch."""
    gen = torch.Generator(device="cuda").manual_seed(64)
    q, k, v, do = (torch.randn((1, H, n, d), generator=gen, device="cuda")
                   for n in (Nq, Nk, Nk, Nq))
    out, lse = ringx.ringx_attn_fwd(q, k, v, 1)
    delta = ringx.ringx_bwd_preprocess(out, do, lse)
    dq, dk, dv = ringx.ringx_attn_bwd(q, k, v, out, do, lse, 1)
    k2, v2 = ringx.ringx_attn_bwd_dkdv(q, k, v, do, lse, delta, 1)
    q2 = ringx.ringx_attn_bwd_dq(q, k, v, do, lse, delta, 1)
    step = [torch.empty_like(x) for x in (q, k, v)]
    ringx.ringx_attn_bwd_step(q, k, v, do, lse, delta, *step, accumulate_dq=False)
    torch.cuda.synchronize()
    for name, a, stage, one in zip(("dq", "dk", "dv"), (dq, dk, dv), (q2, k2, v2), step):
        assert torch.equal(a, stage) and torch.equal(a, one), name


def test_one_value_everywhere():
    """Equal scores: the output is the mean of V and lse = s + ln Nk at any magnitude."""
    for s in (0.0, 3e4, -3e4):
        q = torch.full((1, 1, 20, 8), 1.0, device="cuda")
        k = torch.full((1, 1, 333, 8), s / 8, device="cuda")
        v = torch.randn((1, 1, 333, 8), generator=torch.Generator().manual_seed(3)).cuda()
        out, lse = ringx.ringx_attn_fwd(q, k, v, 4, scale=1.0)
        ref = v.double().mean(2, keepdim=True).expand(1, 1, 20, 8)
        assert float((out.double() - ref).abs().max()) <= TOL_F32
        assert float((lse.double() - (s + math.log(333))).abs().max()) <= 1e-5 + 2.0 ** -23 * abs(s)


def test_no_keys_lost_between_waves():
    """Q = 0: every key weighs the same, so with V = (1, j) the output gives the count and the mean
    index of the keys that the waves visited, exactly placed for any split."""
    for Nk in (1, 15, 16, 17, 127, 128, 129, 255, 1023, 1025):
        q = torch.zeros((1, 1, 3, 2), device="cuda")
        k = torch.randn((1, 1, Nk, 2), generator=torch.Generator().manual_seed(Nk)).cuda()
        v = torch.stack([torch.ones(Nk), torch.arange(Nk, dtype=torch.float32)], -1)
        out, lse = ringx.ringx_attn_fwd(q, k, v.reshape(1, 1, Nk, 2).cuda(), 1)
        assert torch.allclose(out[..., 0].cpu(), torch.ones(1, 1, 3))
        assert abs(float(out[0, 0, 0, 1]) - (Nk - 1) / 2) <= 1e-4 * max(1, Nk)
        assert abs(float(lse[0, 0, 0]) - math.log(Nk)) <= 1e-5
    assert oa.chunk_bounds(10, 3, 2) == (6, 10)
