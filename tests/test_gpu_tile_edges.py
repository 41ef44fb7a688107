"""The row-tile kernels at the edges of their tiles: sequences that end inside a 128-row tile (whole
wavefronts without rows), lists whose blocks do not fill the last 64-key step, and mask rows of one
wavefront that keep different 16-key pieces of a step (random patterns), for both head sizes and every
block size below 128.  fp64 oracle; tolerances as everywhere (o: 1e-2 or half a bf16 ulp, LSE 1e-3,
gradients 2e-2 relative L2)."""

import dataclasses

import numpy as np
import pytest
import torch

from oracle import s2_oracle as orc
from paper_2407_17678_amd import binding as B
from paper_2407_17678_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def _random_mask(rng, H, Bk, density):
    M = np.tril(rng.random((H, Bk, Bk)) < density)
    M[:, np.arange(Bk), np.arange(Bk)] = True
    return M


@pytest.mark.parametrize("tokens", [32, 64, 96, 160, 320, 448])
@pytest.mark.parametrize("S", [16, 32, 64])
@pytest.mark.parametrize("D", [64, 128])
def test_forward_and_backward_at_tile_edges(D, S, tokens):
    if tokens % S:
        pytest.skip("not a whole number of blocks")
    H, batch, Bk = 3, 2, tokens // S
    w = dataclasses.replace(synth.WORKLOADS["tiny" if D == 64 else "1p3b_8k"], block_size=S)
    qb, kb, vb, gb = synth.train_inputs(w, heads=H, batch=batch, seqlen=tokens)
    rng = np.random.default_rng(1000 * D + 10 * S + tokens)
    for density in (0.15, 0.6):
        M = _random_mask(rng, H, Bk, density)
        row_ptr, col_idx, _, _ = orc.compressed_layout(M)
        lay = B.s2_layout_from_csr(H, Bk, S, row_ptr, col_idx)
        print("tile edge case D", D, "S", S, "tokens", tokens, "density", density, flush=True)
        q, k, v, g = (G.to_dev(x) for x in (qb, kb, vb, gb))
        o, dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(4))
        lse = torch.full((batch, H, tokens), float("nan"), dtype=torch.float32, device="cuda")
        ws = torch.full((B.s2_attn_bwd_workspace_bytes(batch, H, tokens, D),), 0xFF, dtype=torch.uint8, device="cuda")
        B.s2_attn_fwd(lay, q, k, v, o, lse, w.scale)
        B.s2_attn_bwd(lay, q, k, v, o, lse, g, dq, dk, dv, w.scale, ws)
        torch.cuda.synchronize()
        dQ, dK, dV, O, LSE = orc.attention_backward(G.bits_f64(qb), G.bits_f64(kb), G.bits_f64(vb), G.bits_f64(gb),
                                                    M, S, w.scale)
        assert G.o_excess(G.to_f64(o), O) <= 0
        assert np.abs(G.to_f64(lse) - LSE).max() <= 1e-3
        for n, t, ref in (("dq", dq, dQ), ("dk", dk, dK), ("dv", dv, dV)):
            assert G.rel_l2(G.to_f64(t), ref) <= 2e-2, n
