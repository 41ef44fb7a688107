"""Long key tiles are also cut where the parts do not all start at once, if the longest tile is more than 2.4 times the length that
a part would best have: gradients of the cut and the uncut launch agree to the rounding of their sums."""

import pytest
import torch

from paper_2407_17678_amd import binding as B

pytestmark = pytest.mark.gpu


# an XCD's slots (64, and as many as 80 of head_dim 64) hold all tiles and no cut of them; longest tile / best length of a part
@pytest.mark.parametrize("D,batch,H,N,local,stride,keep_ds,cut", [
    (128, 4, 8, 2048, 2, 16, False, True), (128, 4, 8, 2048, 2, 16, True, True),   # 3.1
    (128, 3, 8, 2560, 4, 8, False, True), (128, 3, 8, 2560, 4, 8, True, True),     # 3.4
    (128, 3, 8, 2560, 16, 16, False, False),                                       # 2.36
    (64, 1, 8, 10240, 4, 8, False, True),                                          # 8.9
])
def test_cut_beyond_the_slots(D, batch, H, N, local, stride, keep_ds, cut):
    print("cut beyond the slots", D, batch, H, N, local, keep_ds, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(D + batch + N + local)
    q, k, v, g = (torch.randn((batch, H, N, D), device="cuda", generator=gen).bfloat16() for _ in range(4))
    lay = B.s2_layout_build(B.layout_params(H, N // 64, 64, local, stride))
    o, lse = torch.empty_like(q), torch.empty((batch, H, N), dtype=torch.float32, device="cuda")
    scale = D ** -0.5
    B.s2_attn_fwd(lay, q, k, v, o, lse, scale)
    full = B.s2_attn_bwd_workspace_bytes(batch, H, N, D)
    stats = 8 * batch * H * N   # two floats a row: all that a launch without cuts takes
    kept = B.s2_attn_bwd_layout_workspace_bytes(lay, batch, H, N, D) - full if keep_ds else 0
    out = []
    for size in (full + kept, stats + kept):
        ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")
        grads = [torch.full_like(q, float("nan")) for _ in range(3)]
        B.s2_attn_bwd(lay, q, k, v, o, lse, g, *grads, scale, ws)
        torch.cuda.synchronize()
        if size == full + kept:
            assert bool((ws[stats + kept:] != 0xFF).any()) == cut
        out.append(grads)
    for name, a, b in zip(("dq", "dk", "dv"), *out):
        a, b = a.float(), b.float()
        assert torch.isfinite(a).all(), name
        # the rounding to bf16 (one step at most), and float32 sums of up to N terms in another order
        bound = 2.0 ** -7 * b.abs() + N * 2.0 ** -24 * b.abs().max()
        assert ((a - b).abs() <= bound).all(), name
