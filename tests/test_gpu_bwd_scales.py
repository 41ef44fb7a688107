"""The dK/dV kernel starts its score accumulators at -lse / scale: gradients over softmax scales at which that is large
against the scores (small scales, down to the smallest that is accepted, where it would not be finite), of their size, and small
against them (large ones), for each form of the kernel."""

import numpy as np
import pytest
import torch

from oracle import s2_oracle as orc
from paper_2407_17678_amd import binding as B
from paper_2407_17678_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

GRAD_TOL = 2e-2  # relative L2 bound on gradients, as in test_gpu_bwd.py


@pytest.mark.parametrize("scale", [2.0 ** -149, 1e-38, 2e-38, 5e-38, 2.0 ** -121, 1e-30, 1e-4, 0.125, 2.0, 1e30])
@pytest.mark.parametrize("D,S,N,form", [(128, 64, 192, "small"), (128, 64, 320, "keep"), (64, 64, 192, "small"), (128, 16, 160, "small"),
                                        (64, 32, 224, "small"), (128, 64, 203, "packed"), (64, 16, 75, "packed"), (128, 64, 256, "dense")])
def test_scales(D, S, N, form, scale):
    print("scales case", D, S, N, form, scale, flush=True)
    H = 3
    rng = np.random.Generator(np.random.PCG64([synth.BASE_SEED, D, S, N]))
    # scores of about +-3 after scaling where the scale is large, so that rows are peaked but not of one key
    size = min(1.0, 3.0 / (scale * np.sqrt(D)))
    # gradients of about 1e-30 or more, which bf16 holds with all its bits
    grad = np.float32(max(1.0, 1e-30 / scale))
    bits = [synth.round_to_bf16_bits(rng.standard_normal((1, H, N, D)).astype(np.float32) * np.float32(f)) for f in (size, 1.0, 1.0, grad)]
    q, k, v, g = (G.to_dev(b) for b in bits)
    o, lse = torch.empty_like(q), torch.empty((1, H, N), dtype=torch.float32, device="cuda")
    grads = [torch.empty_like(q) for _ in range(3)]
    blocks = -(-N // S)
    blocks += blocks & 1 if S == 16 else 0
    ws = lambda n: torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")
    if form == "dense":
        M = orc.block_mask(H, blocks, blocks, 0, dense=True)
        B.s2_dense_causal_fwd(q, k, v, o, lse, scale)
        B.s2_dense_causal_bwd(q, k, v, o, lse, g, *grads, scale, ws(B.s2_attn_bwd_workspace_bytes(1, H, N, D)))
    else:
        lay = B.s2_layout_build(B.layout_params(H, blocks, S, 2, 3))
        M = orc.block_mask(H, blocks, 2, 3)
        if form == "packed":
            cu = torch.tensor([0, N], dtype=torch.int32, device="cuda")
            B.s2_attn_fwd_varlen(lay, q, k, v, o, lse[0], cu, blocks * S, scale)
            B.s2_attn_bwd_varlen(lay, q, k, v, o, lse[0], g, *grads, cu, blocks * S, scale,
                                 ws(B.s2_attn_bwd_varlen_workspace_bytes(H, N, D)))
        else:
            n = B.s2_attn_bwd_layout_workspace_bytes(lay, 1, H, N, D) if form == "keep" else B.s2_attn_bwd_workspace_bytes(1, H, N, D)
            B.s2_attn_fwd(lay, q, k, v, o, lse, scale)
            B.s2_attn_bwd(lay, q, k, v, o, lse, g, *grads, scale, ws(n))
    torch.cuda.synchronize()
    if form == "packed":
        want = orc.attention_backward_varlen(*(G.bits_f64(b)[0] for b in bits), [0, N], M, S, scale)[:3]
        want = [w[None] for w in want]
    else:
        want = orc.attention_backward(*(G.bits_f64(b) for b in bits), M, S, scale)[:3]
    for name, got, ref in zip(("dq", "dk", "dv"), grads, want):
        got = G.to_f64(got)
        assert np.isfinite(got).all(), name
        assert G.rel_l2(got, ref) <= GRAD_TOL, (name, G.rel_l2(got, ref))
