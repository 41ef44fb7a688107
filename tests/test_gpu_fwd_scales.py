"""The forward at softmax scales so small that no score matters (down to the smallest that is accepted): all of a row's keys weigh
the same and LSE is the logarithm of their number."""

import numpy as np
import pytest
import torch

from oracle import s2_oracle as orc
from paper_2407_17678_amd import binding as B
from paper_2407_17678_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [2.0 ** -149, 1e-38, 2e-38, 1e-30])
@pytest.mark.parametrize("D,S,N,form", [(128, 64, 256, "rows"), (128, 64, 256, "dense"), (128, 128, 203, "packed"), (64, 64, 192, "rows"),
                                        (128, 32, 224, "rows")])
def test_small_scales(D, S, N, form, scale):
    print("forward scales", D, S, N, form, scale, flush=True)
    H, blocks = 2, -(-N // S)
    rng = np.random.Generator(np.random.PCG64([synth.BASE_SEED, D, S, N]))
    bits = [synth.round_to_bf16_bits(rng.standard_normal((1, H, N, D)).astype(np.float32)) for _ in range(3)]
    q, k, v = (G.to_dev(b) for b in bits)
    o, lse = torch.empty_like(q), torch.empty((1, H, N), dtype=torch.float32, device="cuda")
    M = orc.block_mask(H, blocks, blocks if form == "dense" else 2, 3, dense=form == "dense")
    if form == "dense":
        B.s2_dense_causal_fwd(q, k, v, o, lse, scale)
    else:
        lay = B.s2_layout_build(B.layout_params(H, blocks, S, 2, 3))
        if form == "packed":
            cu = torch.tensor([0, N], dtype=torch.int32, device="cuda")
            B.s2_attn_fwd_varlen(lay, q, k, v, o, lse[0], cu, blocks * S, scale)
        else:
            B.s2_attn_fwd(lay, q, k, v, o, lse, scale)
    torch.cuda.synchronize()
    if form == "packed":
        O, LSE = (x[None] for x in orc.attention_forward_varlen(*(G.bits_f64(b)[0] for b in bits), [0, N], M, S, scale))
    else:
        O, LSE = orc.attention_forward(*(G.bits_f64(b) for b in bits), M, S, scale)
    assert G.o_excess(G.to_f64(o), O) <= 0
    assert np.abs(lse.double().cpu().numpy() - LSE).max() <= 1e-3  # as in test_gpu_fwd.py
