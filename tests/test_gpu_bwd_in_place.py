"""dK and dV written over K and V (either way round) by the backward that recomputes S and dP: the gradients are those of a call with
buffers of their own, bit for bit, since no tile reads K or V of another one while they are being replaced."""

import pytest
import torch

from paper_2407_17678_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("swap", [False, True])
@pytest.mark.parametrize("D,S,form", [(64, 64, "small"), (128, 64, "small"), (128, 16, "small"), (64, 64, "packed"), (128, 32, "packed"),
                                      (64, 64, "dense"), (128, 64, "dense")])
def test_gradients_in_place(D, S, form, swap):
    H, N, scale = 8, 2048, D ** -0.5
    print("in place", D, S, form, swap, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(D + S)
    q, k, v, g = (torch.randn((1, H, N, D), device="cuda", generator=gen).bfloat16() for _ in range(4))
    o, lse = torch.empty_like(q), torch.empty((1, H, N), dtype=torch.float32, device="cuda")
    lay = B.s2_layout_build(B.layout_params(H, N // S, S, max(1, 128 // S), 4))
    cu = torch.tensor([0, 700, N], dtype=torch.int32, device="cuda")
    if form == "packed":
        size = B.s2_attn_bwd_varlen_workspace_bytes(H, N, D)
        fwd = lambda: B.s2_attn_fwd_varlen(lay, q, k, v, o, lse[0], cu, N, scale)
        bwd = lambda k, v, *grads: B.s2_attn_bwd_varlen(lay, q, k, v, o, lse[0], g, *grads, cu, N, scale, ws)
    elif form == "dense":
        size = B.s2_dense_causal_bwd_workspace_bytes(1, H, N, D)
        fwd = lambda: B.s2_dense_causal_fwd(q, k, v, o, lse, scale)
        bwd = lambda k, v, *grads: B.s2_dense_causal_bwd(q, k, v, o, lse, g, *grads, scale, ws)
    else:
        size = B.s2_attn_bwd_workspace_bytes(1, H, N, D)
        fwd = lambda: B.s2_attn_fwd(lay, q, k, v, o, lse, scale)
        bwd = lambda k, v, *grads: B.s2_attn_bwd(lay, q, k, v, o, lse, g, *grads, scale, ws)
    ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")
    fwd()
    dq, dk, dv = (torch.empty_like(q) for _ in range(3))
    bwd(k, v, dq, dk, dv)
    dq2, k2, v2 = torch.empty_like(q), k.clone(), v.clone()
    bwd(k2, v2, dq2, *((v2, k2) if swap else (k2, v2)))
    torch.cuda.synchronize()
    dk2, dv2 = (v2, k2) if swap else (k2, v2)
    for name, a, b in zip(("dq", "dk", "dv"), (dq2, dk2, dv2), (dq, dk, dv)):
        assert torch.isfinite(b.float()).all(), name
        assert torch.equal(a, b), name
