"""The bf16 backward's ways of cutting a launch (needs an MI355X), at the edges of their ranges and at
key and query counts that leave streams empty, single tiles, or a ragged last round.

Bar: the element-wise bound of the path's own roundings (P and dS rounded to bf16, the stored
output, D formed from it), with the margin of 1.5 that the other element-wise checks take."""

import numpy as np
import pytest
import torch

import oracle
from paper_2507_16697_amd import ringx

from parity_util import random_case, rounding_bounds, to_device, to_host_f64

pytestmark = pytest.mark.gpu

# (H, Nq, Nk, R): dQ is cut by n = H ceil(Nq / 256)
DQ = [(1, 1, 1, 1), (1, 65, 255, 2), (3, 64, 256, 5), (2, 300, 257, 1), (1, 257, 700, 700),
      (64, 40, 300, 3), (65, 70, 127, 1), (65, 70, 128, 4), (128, 129, 200, 3), (129, 40, 100, 2),
      (257, 70, 130, 3), (192, 300, 66, 1), (768, 5, 40, 2)]
# dK/dV at d = 64 is cut by n = H R ceil(ceil(Nk / R) / 128) 128-key tiles
DKDV = [(1, 63, 63, 1), (2, 64, 65, 1), (4, 129, 1000, 8), (65, 40, 200, 2), (128, 33, 129, 1),
        (130, 31, 260, 1), (129, 65, 128, 4), (300, 20, 300, 1)]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,Nq,Nk,R", DQ + DKDV)
def test_every_cut(H, Nq, Nk, R, d):
    std = 0.5 if d == 64 else 2 ** -0.5
    t, x = random_case(72, 1, H, Nq, Nk, d, std=std, do_std=std)
    g = {key: to_device(val, "bf16") for key, val in t.items()}
    scale = float(np.float32(d ** -0.5))
    ro, rl = oracle.attention(x["q"], x["k"], x["v"], scale)
    rq, rk, rv = oracle.attention_bwd(x["q"], x["k"], x["v"], ro, x["do"], rl, scale)
    _, bq, bk, bv = rounding_bounds(x, x["k"], x["v"], ro, rl, scale)
    out, lse = ringx.ringx_attn_fwd(g["q"], g["k"], g["v"], R, scale=scale)
    dq, dk, dv = ringx.ringx_attn_bwd(g["q"], g["k"], g["v"], out, g["do"], lse, R, scale=scale)
    again = ringx.ringx_attn_bwd(g["q"], g["k"], g["v"], out, g["do"], lse, R, scale=scale)
    delta = ringx.ringx_bwd_preprocess(out, g["do"], lse)
    acc = [dq.clone(), dk.clone(), dv.clone()]
    ringx.ringx_attn_bwd_step(g["q"], g["k"], g["v"], g["do"], lse, delta, acc[0], acc[1], acc[2],
                              accumulate_dq=True, accumulate_dkv=True, scale=scale)
    torch.cuda.synchronize()
    for name, a, b, twice, ref, bound in (("dq", dq, again[0], acc[0], rq, bq),
                                          ("dk", dk, again[1], acc[1], rk, bk),
                                          ("dv", dv, again[2], acc[2], rv, bv)):
        assert torch.equal(a, b), name
        e = float(np.max(np.abs(to_host_f64(a) - ref) / (1.5 * bound + 1e-6)))
        assert e <= 1.0, (name, e)
        e = float(np.max(np.abs(to_host_f64(twice) - 2 * ref) / (3.0 * bound + 2e-6)))
        assert e <= 1.0, (name, "accumulated", e)
