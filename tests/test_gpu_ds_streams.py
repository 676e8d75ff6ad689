"""dQ from stored dS through both of its kernels (needs an MI355X): the key-stream kernel (slabs of up
to 64 groups of 128 queries, and of up to 128 where it has enough keys) at the edges of its 32-key
blocks, 32-query blocks and four streams, in one round of workgroups and in two, and the 128-query
kernel for the others.  Held to the recompute backward: the two paths round the same
dS to bf16, so dQ differs by summation order and single roundings only (relative RMS 1e-4)."""

import math

import pytest
import torch

from paper_2507_16697_amd import ringx

pytestmark = pytest.mark.gpu

# (H, Hkv, Nq, Nk, R); groups of 128 queries = H ceil(Nq / 128)
CASES = [(1, 1, 1, 2, 1), (1, 1, 31, 31, 1), (1, 1, 33, 33, 3), (2, 1, 32, 96, 1),
         (2, 2, 127, 127, 2), (1, 1, 129, 128, 1), (3, 3, 160, 129, 4), (2, 1, 97, 640, 7),
         (128, 128, 20, 70, 2), (129, 129, 20, 70, 2), (129, 43, 33, 150, 1),
         (65, 65, 20, 255, 1), (65, 65, 20, 256, 1), (128, 64, 33, 300, 3), (70, 35, 101, 6200, 2)]


@pytest.mark.parametrize("H,Hkv,Nq,Nk,R", CASES)
def test_ds_streams(H, Hkv, Nq, Nk, R):
    gen = torch.Generator(device="cuda").manual_seed(91)

    def rand(h, n):
        return (torch.randn((1, h, n, 128), generator=gen, device="cuda") * 2 ** -0.5).bfloat16()

    q, k, v, do = rand(H, Nq), rand(Hkv, Nk), rand(Hkv, Nk), rand(H, Nq)
    out, lse = ringx.ringx_attn_fwd_gqa(q, k, v, R)
    ref = ringx.ringx_attn_bwd_gqa(q, k, v, out, do, lse, R)
    delta = ringx.ringx_bwd_preprocess(out, do, lse)
    ds = torch.empty(ringx.ringx_bwd_ds_bytes(H, Hkv, Nq, Nk, 128, R, Hkv), dtype=torch.uint8,
                     device="cuda")
    dk, dv = ringx.ringx_attn_bwd_dkdv_ds(q, k, v, do, lse, delta, R, ds, 0, Hkv)
    dq = torch.full((1, H, Nq, 128), math.nan, device="cuda")
    ringx.ringx_attn_bwd_dq_ds(ds, k, q.shape, R, 0, Hkv, dq=dq)
    again = ringx.ringx_attn_bwd_dq_ds(ds, k, q.shape, R, 0, Hkv)
    torch.cuda.synchronize()
    assert torch.equal(dk, ref[1]) and torch.equal(dv, ref[2])
    assert torch.equal(dq, again)
    diff = float((dq - ref[0]).double().pow(2).mean().sqrt())
    assert diff <= 1e-4 * float(ref[0].double().pow(2).mean().sqrt()), diff
