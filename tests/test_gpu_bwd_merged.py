"""Up to 4096 workgroups in all a backward runs dQ and dK/dV in one launch after delta: its gradients are those of the two
launches, bit for bit, on both sides of that size, and so the kernels of either are held to the results of the other."""

import numpy as np
import pytest
import torch

from paper_2407_17678_amd import binding as B
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


# (batch, heads) x 128-row tiles of queries and of keys: 16 workgroups, some hundreds, 4096 and more
@pytest.mark.parametrize("batch,H,tiles", [(1, 1, 1), (1, 3, 5), (1, 8, 65), (4, 16, 32), (4, 16, 33)])
@pytest.mark.parametrize("D,S", [(128, 64), (64, 64), (128, 16), (64, 32), (128, 128)])
def test_one_launch_and_two(batch, H, tiles, D, S):
    N = 128 * tiles - (S if S < 128 and tiles > 1 else 0)
    N -= N % (2 * S) if S == 16 else 0
    print("backward", batch, H, N, D, S, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(batch + 10 * H + 100 * tiles + D + S)
    q, k, v, g = (torch.randn((batch, H, N, D), device="cuda", generator=gen).bfloat16() for _ in range(4))
    o, lse = torch.empty_like(q), torch.empty((batch, H, N), dtype=torch.float32, device="cuda")
    lay = B.s2_layout_build(B.layout_params(H, N // S, S, max(1, 128 // S), 4))
    scale = D ** -0.5
    B.s2_attn_fwd(lay, q, k, v, o, lse, scale)
    ws = torch.full((B.s2_attn_bwd_workspace_bytes(batch, H, N, D),), 0xFF, dtype=torch.uint8, device="cuda")
    one = [torch.full_like(q, float("nan")) for _ in range(3)]
    two = [torch.full_like(q, float("nan")) for _ in range(3)]
    B.s2_attn_bwd(lay, q, k, v, o, lse, g, *one, scale, ws)
    ws[:] = 0xFF
    for stage in (B.BWD_DQ, B.BWD_DKDV):
        B.s2_attn_bwd_stages(lay, q, k, v, o, lse, g, *two, scale, ws, stage)
    torch.cuda.synchronize()
    for name, a, b in zip(("dq", "dk", "dv"), one, two):
        assert torch.isfinite(a.float()).all(), name
        assert torch.equal(a, b), name


@pytest.mark.parametrize("D,S", [(128, 64), (64, 16)])
def test_packed_sequences_as_if_alone(D, S):
    # three sequences in one call against each in a call of its own: the same tiles, the same bits
    H, lens = 2, [200, 37, 512]
    total, scale = sum(lens), D ** -0.5
    gen = torch.Generator(device="cuda")
    gen.manual_seed(D + S)
    q, k, v, g = (torch.randn((1, H, total, D), device="cuda", generator=gen).bfloat16() for _ in range(4))
    lay = B.s2_layout_build(B.layout_params(H, 512 // S, S, 64 // S, 5))

    def run(q, k, v, g, lens):
        rows = sum(lens)
        cu = torch.tensor([0] + list(np.cumsum(lens)), dtype=torch.int32, device="cuda")
        o, lse = torch.empty_like(q), torch.empty((H, rows), dtype=torch.float32, device="cuda")
        grads = [torch.full_like(q, float("nan")) for _ in range(3)]
        ws = torch.full((B.s2_attn_bwd_varlen_workspace_bytes(H, rows, D),), 0xFF, dtype=torch.uint8, device="cuda")
        B.s2_attn_fwd_varlen(lay, q, k, v, o, lse, cu, 512, scale)
        B.s2_attn_bwd_varlen(lay, q, k, v, o, lse, g, *grads, cu, 512, scale, ws)
        torch.cuda.synchronize()
        return grads

    together = run(q, k, v, g, lens)
    lo = 0
    for n in lens:
        alone = run(*(x[:, :, lo:lo + n].contiguous() for x in (q, k, v, g)), [n])
        for name, a, b in zip(("dq", "dk", "dv"), together, alone):
            assert torch.isfinite(b.float()).all(), name
            assert torch.equal(a[:, :, lo:lo + n], b), (name, n)
        lo += n


@pytest.mark.parametrize("D", [64, 128])
def test_dense_in_one_launch_and_two(D):
    # 72 heads of 29 tiles of either kind are beyond 4096 workgroups, 36 of them are not
    H, N, scale = 72, 3712, D ** -0.5
    print("dense backward", H, N, D, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(D)
    q, k, v, g = (torch.randn((1, H, N, D), device="cuda", generator=gen).bfloat16() for _ in range(4))

    def run(q, k, v, g):
        heads = q.shape[1]
        o, lse = torch.empty_like(q), torch.empty((1, heads, N), dtype=torch.float32, device="cuda")
        grads = [torch.full_like(q, float("nan")) for _ in range(3)]
        ws = torch.full((B.s2_dense_causal_bwd_workspace_bytes(1, heads, N, D),), 0xFF, dtype=torch.uint8, device="cuda")
        B.s2_dense_causal_fwd(q, k, v, o, lse, scale)
        B.s2_dense_causal_bwd(q, k, v, o, lse, g, *grads, scale, ws)
        torch.cuda.synchronize()
        return grads

    whole = run(q, k, v, g)
    for lo in (0, 36):
        part = run(*(x[:, lo:lo + 36].contiguous() for x in (q, k, v, g)))
        for name, a, b in zip(("dq", "dk", "dv"), whole, part):
            assert torch.isfinite(a.float()).all(), name
            assert torch.equal(a[:, lo:lo + 36], b), (name, lo)


@pytest.mark.parametrize("S", [16, 32, 64, 128])
@pytest.mark.parametrize("D", [64, 128])
def test_packed_in_one_launch_and_two(D, S):
    # The grid goes by the layout (key tiles) and by the longest length allowed (query tiles): the same sequences with a small
    # and with a large one are 8 * (258 + 5) and 8 * (258 + 258) workgroups.
    H, lens, scale, long = 2, [200, 37, 600, 128], D ** -0.5, 258 * 128
    total = sum(lens)
    print("packed backward", D, S, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(D + S)
    q, k, v, g = (torch.randn((1, H, total, D), device="cuda", generator=gen).bfloat16() for _ in range(4))
    lay = B.s2_layout_build(B.layout_params(H, long // S, S, max(1, 64 // S), 5))
    assert B.s2_layout_get_tiles(lay, B.TILES_DKDV)["tiles_per_head"] == 258
    cu = torch.tensor([0] + list(np.cumsum(lens)), dtype=torch.int32, device="cuda")
    o, lse = torch.empty_like(q), torch.empty((H, total), dtype=torch.float32, device="cuda")
    B.s2_attn_fwd_varlen(lay, q, k, v, o, lse, cu, 640, scale)
    out = []
    for longest in (640, long):
        grads = [torch.full_like(q, float("nan")) for _ in range(3)]
        ws = torch.full((B.s2_attn_bwd_varlen_workspace_bytes(H, total, D),), 0xFF, dtype=torch.uint8, device="cuda")
        B.s2_attn_bwd_varlen(lay, q, k, v, o, lse, g, *grads, cu, longest, scale, ws)
        torch.cuda.synchronize()
        out.append(grads)
    for name, a, b in zip(("dq", "dk", "dv"), *out):
        assert torch.isfinite(a.float()).all(), name
        assert torch.equal(a, b), name
