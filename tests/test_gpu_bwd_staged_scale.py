"""A call for dK/dV alone needs nothing of an earlier call but delta, which depends on neither the scale nor lse: both are its own."""

import pytest
import torch

from paper_2407_17678_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first", [B.BWD_DELTA, B.BWD_DQ])
@pytest.mark.parametrize("D,S,keep_ds", [(128, 64, False), (64, 64, False), (128, 16, False), (128, 128, True)])
def test_scale_of_the_dkdv_call(D, S, keep_ds, first):
    if keep_ds and first == B.BWD_DQ:
        pytest.skip("where dS is kept dQ comes last and leaves no delta")
    # (tiles are cut at this size, so the counters are cleared by the call for dK/dV)
    batch, H, N, scale = 1, 8, 4096, D ** -0.5
    print("staged backward", D, S, keep_ds, first, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(D + S + first)
    q, k, v, g = (torch.randn((batch, H, N, D), device="cuda", generator=gen).bfloat16() for _ in range(4))
    o, lse = torch.empty_like(q), torch.empty((batch, H, N), dtype=torch.float32, device="cuda")
    lay = B.s2_layout_build(B.layout_params(H, N // S, S, max(1, 128 // S), 4))
    B.s2_attn_fwd(lay, q, k, v, o, lse, scale)
    size = B.s2_attn_bwd_layout_workspace_bytes if keep_ds else lambda _, *shape: B.s2_attn_bwd_workspace_bytes(*shape)
    ws = torch.full((size(lay, batch, H, N, D),), 0xFF, dtype=torch.uint8, device="cuda")
    want = [torch.full_like(q, float("nan")) for _ in range(3)]
    B.s2_attn_bwd(lay, q, k, v, o, lse, g, *want, scale, ws)
    ws[:] = 0xFF
    got = [torch.full_like(q, float("nan")) for _ in range(3)]
    B.s2_attn_bwd_stages(lay, q, k, v, o, torch.zeros_like(lse), g, *got, 3.0, ws, first)
    B.s2_attn_bwd_stages(lay, q, k, v, o, lse, g, *got, scale, ws, B.BWD_DKDV)
    B.s2_attn_bwd_stages(lay, q, k, v, o, lse, g, *got, scale, ws, B.BWD_DQ)
    torch.cuda.synchronize()
    for name, a, b in zip(("dq", "dk", "dv"), got, want):
        assert torch.isfinite(a.float()).all(), name
        assert torch.equal(a, b), name
