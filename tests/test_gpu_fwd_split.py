"""The bf16 forward's ways of cutting a launch (needs an MI355X): two and four key streams per
workgroup, half-size workgroups, and partials spread over chunk groups, at the edges of their
ranges (how many 256-query workgroups the problem makes decides) and at key counts that leave
streams empty, single tiles, or a ragged last round.

Bars: the outputs' element-wise rounding bound (P and the output are rounded to bf16), lse max abs
1e-4 (the row sums are fp32)."""

import numpy as np
import pytest
import torch

import oracle
from oracle import attention_fp64 as oa
from paper_2507_16697_amd import ringx

from parity_util import (TOL_BF16_REL_RMS, max_abs_err, random_case, rel_rms_err, to_device,
                         to_host_f64)

pytestmark = pytest.mark.gpu

# (H, Nq, Nk, R): n = H ceil(Nq / 256) workgroups of 256 queries
FOUR = [(1, 1, 1, 1), (2, 33, 64, 1), (1, 65, 255, 2), (3, 64, 256, 5), (2, 300, 257, 1),
        (1, 257, 700, 700), (64, 40, 300, 3)]
TWO = [(65, 70, 127, 1), (65, 70, 128, 4), (128, 129, 200, 3)]
WHOLE = [(129, 40, 100, 2), (256, 33, 65, 1)]
HALF = [(257, 70, 130, 3), (192, 300, 66, 1), (512, 20, 33, 2), (1025, 3, 65, 1)]
GROUPS = [(40, 300, 150, 20), (3, 90, 150, 150), (130, 20, 300, 9), (300, 20, 70, 3)]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,Nq,Nk,R", FOUR + TWO + WHOLE + HALF + GROUPS)
def test_every_cut(H, Nq, Nk, R, d):
    std = 0.5 if d == 64 else 2 ** -0.5
    t, x = random_case(71, 1, H, Nq, Nk, d, std=std)
    g = {key: to_device(val, "bf16") for key, val in t.items()}
    scale = float(np.float32(d ** -0.5))
    out, lse = ringx.ringx_attn_fwd(g["q"], g["k"], g["v"], R, scale=scale)
    po, pl = ringx.ringx_attn_fwd_partials(g["q"], g["k"], g["v"], R, scale=scale)
    acc = torch.full((1, H, Nq, d), float("nan"), device="cuda")
    acc_lse = torch.full((1, H, Nq), float("nan"), device="cuda")
    lo, hi = ringx.ringx_chunk_bounds(Nk, min(R, 2), 0)
    for i, s in enumerate((slice(0, hi), slice(hi, Nk))):
        if s.start < s.stop:
            ringx.ringx_attn_fwd_step(g["q"], g["k"][:, :, s].clone(), g["v"][:, :, s].clone(), acc,
                                      acc_lse, i == 0, scale=scale)
    torch.cuda.synchronize()
    rpo, rpl = oracle.attention_partials(x["q"], x["k"], x["v"], scale, R)
    ro, rl = oa.lse_merge(rpo, rpl)
    # element by element: P rounded to bf16 (relative 2^-8 of every term of the sum), and the bf16
    # output rounded once more, with the 1.5 margin of the other element-wise checks
    apo, _ = oracle.attention_partials(x["q"], x["k"], np.abs(x["v"]), scale, R)
    ao, _ = oa.lse_merge(apo, rpl)
    u = 1.5 * 2.0 ** -8
    for name, a, ref, bound in (("out", out, ro, ao + np.abs(ro)), ("part_out", po, rpo, apo),
                                ("acc", acc, ro, ao)):
        e = float(np.max(np.abs(to_host_f64(a) - ref) / (u * bound + 1e-6)))
        assert e <= 1.0, (name, e)
    for name, a, ref in (("lse", lse, rl), ("part_lse", pl, rpl), ("acc_lse", acc_lse, rl)):
        e = max_abs_err(to_host_f64(a), ref)
        assert e <= 1e-4, (name, e)


@pytest.mark.parametrize("d", [64, 128])
def test_streams_with_distant_references(d):
    """Scores that climb by 3000 along the keys: the key streams of a workgroup end with references
    far apart, and the last keys alone make the result."""
    Nk = 640
    q = torch.ones((1, 1, 70, d), device="cuda", dtype=torch.bfloat16)
    ramp = torch.arange(Nk, dtype=torch.float32).div(64).floor().mul(300 / d)
    k = ramp.reshape(1, 1, Nk, 1).expand(1, 1, Nk, d).contiguous().bfloat16().cuda()
    v = torch.randn((1, 1, Nk, d), generator=torch.Generator().manual_seed(5)).bfloat16().cuda()
    for sign in (1.0, -1.0):
        out, lse = ringx.ringx_attn_fwd(q, k * sign, v, 1, scale=1.0)
        s = (q.double() @ (k * sign).double().transpose(-1, -2).contiguous())
        ro = torch.softmax(s, -1) @ v.double()
        rl = torch.logsumexp(s, -1)
        assert rel_rms_err(to_host_f64(out), ro.cpu().numpy()) <= TOL_BF16_REL_RMS
        assert float((lse.double() - rl).abs().max()) <= 1e-3


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,Nq", [(2, 70), (65, 70)])
def test_streams_of_masked_keys(H, Nq, d):
    """Keys masked by a feature of -inf (scores of -inf): streams whose keys are all masked add
    nothing.  The first tile is not masked, so one stream over all keys needs no care."""
    gen = torch.Generator().manual_seed(6)
    q, k, v = (torch.randn((1, H, n, d), generator=gen).mul_(0.5) for n in (Nq, 700, 700))
    q[..., 0], k[..., 0] = 1.0, 0.0
    k[:, :, 64:] = 0.0
    k[:, :, 64:, 0] = -float("inf")
    q, k, v = (x.bfloat16().cuda() for x in (q, k, v))
    # one chunk: a chunk with no key at all has no local result
    out, lse = ringx.ringx_attn_fwd(q, k, v, 1, scale=d ** -0.5)
    s = (q.double() @ k[:, :, :64].double().transpose(-1, -2).contiguous()) * d ** -0.5
    ro = torch.softmax(s, -1) @ v[:, :, :64].double()
    assert rel_rms_err(to_host_f64(out), ro.cpu().numpy()) <= TOL_BF16_REL_RMS
    assert float((lse.double() - torch.logsumexp(s, -1)).abs().max()) <= 1e-4
