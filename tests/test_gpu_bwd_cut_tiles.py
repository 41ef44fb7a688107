"""The dK/dV launch with its longest key tiles cut into parts that different workgroups walk (chosen when a
launch has few tiles, by the room in the workspace): against the fp64 oracle at the usual 2e-2 relative
L2, bit for bit repeatable though the parts finish in any order, the same through the stage calls when
the dK/dV launch runs several times on one delta, and close to the uncut result of the smallest workspace.
One pattern has a column that every row of one head attends while the other heads keep their diagonal
only, so that parts of their tiles are empty."""

import dataclasses

import numpy as np
import pytest
import torch

from oracle import s2_oracle as orc
from paper_2407_17678_amd import binding as B
from paper_2407_17678_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

CASES = [
    # D, S, heads, batch, blocks, local, stride (0: the one-column pattern), keep dS
    (64, 64, 4, 1, 8, 2, 4, False),       # parts of four steps
    (64, 16, 3, 1, 64, 2, 16, False),
    (64, 128, 2, 2, 12, 1, 4, False),
    (128, 64, 2, 1, 33, 2, 8, False),     # an odd number of blocks
    (128, 64, 3, 1, 32, 3, 8, True),
    (128, 32, 2, 2, 40, 2, 8, False),
    (128, 16, 9, 1, 66, 3, 16, False),    # the last step of a list not full
    (128, 128, 2, 1, 12, 1, 4, True),
    (128, 64, 3, 1, 32, 1, 0, False),
    (128, 64, 3, 1, 32, 1, 0, True),
    (64, 16, 3, 1, 128, 1, 0, False),
]


def _mask(H, Bk, B_l, stride):
    if stride:
        return orc.block_mask(H, Bk, B_l, stride)
    M = np.zeros((H, Bk, Bk), dtype=bool)
    M[:, np.arange(Bk), np.arange(Bk)] = True
    M[1, :, 0] = True
    return M


def _counters_and_sums(ws, lay, batch, H, N, D, keep_ds):
    """The part of the workspace that cut tiles use, behind the statistics and (kept) dS."""
    off = 2 * ((batch * H * N * 4 + 255) // 256 * 256)
    if keep_ds:
        off += B.s2_attn_bwd_layout_workspace_bytes(lay, batch, H, N, D) - B.s2_attn_bwd_workspace_bytes(batch, H, N, D)
    tiles = batch * H * (-(-N // 128))
    end = off + (4 * tiles + 255) // 256 * 256
    return ws[off:off + 4 * tiles].view(torch.int32), ws[end:]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "D%d_S%d_H%d_b%d_B%d_L%d_V%d_%s" % (c[:7] + ("keep" if c[7] else "again",)))
def test_cut_tiles(case):
    D, S, H, batch, Bk, B_l, stride, keep_ds = case
    N = Bk * S
    w = dataclasses.replace(synth.WORKLOADS["tiny" if D == 64 else "1p3b_8k"], block_size=S)
    print("cut tiles case", case, flush=True)
    bits = synth.train_inputs(w, heads=H, batch=batch, seqlen=N)
    q, k, v, g = (G.to_dev(x) for x in bits)
    M = _mask(H, Bk, B_l, stride)
    row_ptr, col_idx, _, _ = orc.compressed_layout(M)
    lay = B.s2_layout_from_csr(H, Bk, S, row_ptr, col_idx)
    o = torch.empty_like(q)
    lse = torch.empty((batch, H, N), dtype=torch.float32, device="cuda")
    B.s2_attn_fwd(lay, q, k, v, o, lse, w.scale)
    size = B.s2_attn_bwd_layout_workspace_bytes if keep_ds else lambda lay, *s: B.s2_attn_bwd_workspace_bytes(*s)
    ws = torch.full((size(lay, batch, H, N, D),), 0xFF, dtype=torch.uint8, device="cuda")
    runs = []
    for _ in range(3):
        grads = [torch.full_like(q, float("nan")) for _ in range(3)]
        ws[:] = 0xFF
        B.s2_attn_bwd(lay, q, k, v, o, lse, g, *grads, w.scale, ws)
        runs.append(grads)
        # the workspace shows that tiles were cut: a counter has counted parts, and sums have been written
        count, sums = _counters_and_sums(ws, lay, batch, H, N, D, keep_ds)
        assert 2 <= int(count.max()) <= 64 and int(count.min()) >= 0 and bool((sums != 0xFF).any())
    grads = [torch.full_like(q, float("nan")) for _ in range(3)]
    ws[:] = 0xFF
    # (delta comes from the launch that a whole backward takes it from, so that it is the same to the bit)
    for stage in (B.BWD_DELTA if keep_ds else B.BWD_DQ, B.BWD_DKDV, B.BWD_DKDV, B.BWD_DKDV):
        B.s2_attn_bwd_stages(lay, q, k, v, o, lse, g, *grads, w.scale, ws, stage)
    # two floats per row: nothing is cut
    small = [torch.full_like(q, float("nan")) for _ in range(3)]
    least = 2 * ((batch * H * N * 4 + 255) // 256 * 256)
    B.s2_attn_bwd(lay, q, k, v, o, lse, g, *small, w.scale, ws[:least])
    torch.cuda.synchronize()
    ref = orc.attention_backward(*(G.bits_f64(x) for x in bits), M, S, w.scale)
    for i, n in enumerate(("dq", "dk", "dv")):
        for b in range(batch):
            for h in range(H):
                assert G.rel_l2(G.to_f64(runs[0][i])[b, h], ref[i][b, h]) <= 2e-2, (n, b, h)
        assert all(torch.equal(runs[0][i], r[i]) for r in runs[1:]), n
        # (the sums differ in the order of their fp32 additions, dQ also in whether dS is formed twice: at
        # most bf16 roundings, 2^-9 of an element each way)
        assert G.rel_l2(G.to_f64(small[i]), G.to_f64(runs[0][i])) <= 5e-3, n
    assert torch.equal(grads[1], runs[0][1]) and torch.equal(grads[2], runs[0][2])


@pytest.mark.parametrize("keep_ds", [False, True])
def test_a_dkdv_call_clears_its_own_counters(keep_ds):
    # delta by a call whose workspace is too small for any tile to be cut, dK/dV by one with the room for it on
    # the same memory: the counters, which the first call does not know of, still hold what was there before
    D, S, H, batch, Bk = 128, 64, 3, 1, 32
    N = Bk * S
    w = dataclasses.replace(synth.WORKLOADS["1p3b_8k"], block_size=S)
    q, k, v, g = (G.to_dev(x) for x in synth.train_inputs(w, heads=H, batch=batch, seqlen=N))
    row_ptr, col_idx, _, _ = orc.compressed_layout(orc.block_mask(H, Bk, 3, 8))
    lay = B.s2_layout_from_csr(H, Bk, S, row_ptr, col_idx)
    o = torch.empty_like(q)
    lse = torch.empty((batch, H, N), dtype=torch.float32, device="cuda")
    B.s2_attn_fwd(lay, q, k, v, o, lse, w.scale)
    bytes_ = B.s2_attn_bwd_layout_workspace_bytes(lay, batch, H, N, D) if keep_ds else B.s2_attn_bwd_workspace_bytes(batch, H, N, D)
    least = 2 * ((batch * H * N * 4 + 255) // 256 * 256)
    stage = B.BWD_DELTA if keep_ds else B.BWD_DQ
    results = []
    for fill in (0xFF, 0x00, 0x01):
        for first in (least, bytes_):
            ws = torch.full((bytes_,), fill, dtype=torch.uint8, device="cuda")
            grads = [torch.full_like(q, float("nan")) for _ in range(3)]
            B.s2_attn_bwd_stages(lay, q, k, v, o, lse, g, *grads, w.scale, ws[:first], stage)
            B.s2_attn_bwd_stages(lay, q, k, v, o, lse, g, *grads, w.scale, ws, B.BWD_DKDV)
            results.append(grads[1:])
    torch.cuda.synchronize()
    for r in results:
        assert torch.equal(r[0], results[1][0]) and torch.equal(r[1], results[1][1])
    assert torch.isfinite(results[1][0].float()).all()


@pytest.mark.parametrize("D,S,H,N,local,cut", [
    (64, 64, 3, 1024, 1, False), (128, 32, 3, 1024, 1, False),     # a local window of one block: no key tile is long enough
    (128, 64, 60, 640, 10, False), (128, 64, 40, 640, 10, True),   # an XCD's 64 slots hold all 40 (25) tiles but not the 72 parts (but the 45)
])
def test_whether_tiles_are_cut(D, S, H, N, local, cut):
    # the room for the counters and sums of cut tiles stays untouched where none is
    w = dataclasses.replace(synth.WORKLOADS["tiny" if D == 64 else "1p3b_8k"], block_size=S)
    q, k, v, g = (G.to_dev(x) for x in synth.train_inputs(w, heads=H, batch=1, seqlen=N))
    lay = B.s2_layout_build(B.layout_params(H, N // S, S, local, 0))
    o, lse = torch.empty_like(q), torch.empty((1, H, N), dtype=torch.float32, device="cuda")
    B.s2_attn_fwd(lay, q, k, v, o, lse, w.scale)
    ws = torch.full((B.s2_attn_bwd_workspace_bytes(1, H, N, D),), 0xFF, dtype=torch.uint8, device="cuda")
    grads = [torch.empty_like(q) for _ in range(3)]
    B.s2_attn_bwd(lay, q, k, v, o, lse, g, *grads, w.scale, ws)
    count, sums = _counters_and_sums(ws, lay, 1, H, N, D, False)
    assert (int(count.max()) > 1) == cut and bool((sums != 0xFF).any()) == cut


@pytest.mark.parametrize("D,S,batch,H,N,local,stride,parts", [
    (128, 64, 1, 7, 8192, 4, 8, 8), (64, 64, 1, 2, 8192, 4, 8, 11), (128, 128, 3, 4, 3072, 3, 4, 3),   # pairs / 8 alone would give 3, 22 and 6 parts
    (128, 64, 4, 23, 768, 3, 7, 0), (128, 128, 4, 21, 512, 3, 5, 0),                                     # ... and two
    (64, 64, 1, 8, 8192, 4, 8, 4), (128, 32, 1, 16, 3584, 16, 16, 3),                                    # no pairs left over
])
def test_parts_of_the_longest_tile(D, S, batch, H, N, local, stride, parts):
    # pairs that are left over from a multiple of eight count as a whole one for whether tiles are cut, as most of one for how long parts are
    w = dataclasses.replace(synth.WORKLOADS["tiny" if D == 64 else "1p3b_8k"], block_size=S)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H + N)
    q, k, v, g = (torch.randn((batch, H, N, D), device="cuda", generator=gen).bfloat16() for _ in range(4))
    lay = B.s2_layout_build(B.layout_params(H, N // S, S, local, stride))
    o, lse = torch.empty_like(q), torch.empty((batch, H, N), dtype=torch.float32, device="cuda")
    B.s2_attn_fwd(lay, q, k, v, o, lse, w.scale)
    ws = torch.full((B.s2_attn_bwd_workspace_bytes(batch, H, N, D),), 0xFF, dtype=torch.uint8, device="cuda")
    grads = [torch.empty_like(q) for _ in range(3)]
    print("parts of the longest tile", D, S, batch, H, N, flush=True)
    B.s2_attn_bwd(lay, q, k, v, o, lse, g, *grads, w.scale, ws)
    count, sums = _counters_and_sums(ws, lay, batch, H, N, D, False)
    assert bool((sums != 0xFF).any()) == (parts > 0)
    assert parts == 0 or int(count.max()) == parts
