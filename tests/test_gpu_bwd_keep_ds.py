"""GPU parity of the backward that keeps dS (the larger workspace of s2_attn_bwd_layout_workspace_bytes:
delta, then dK/dV leaving dS, then dQ = scale * dS K) against the fp64 oracle, through the C ABI."""

import dataclasses

import numpy as np
import pytest
import torch

from oracle import s2_oracle as orc
from paper_2407_17678_amd import binding as B
from paper_2407_17678_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

GRAD_TOL = 2e-2   # relative L2 bound stated for this build


def _check(w, heads, batch, seqlen):
    qb, kb, vb, gb = synth.train_inputs(w, heads=heads, batch=batch, seqlen=seqlen)
    Bt, H, N, D = qb.shape
    print("bwd keeping dS", w.name, qb.shape, "S", w.block_size, flush=True)
    out = G.run_fwd_bwd(w, qb, kb, vb, gb, keep_ds=True)
    assert out["ws_bytes"] > B.s2_attn_bwd_workspace_bytes(Bt, H, N, D), "the case must take the path under test"
    M = G.oracle_mask(w, H, N)
    dQ, dK, dV, O, LSE = orc.attention_backward(G.bits_f64(qb), G.bits_f64(kb), G.bits_f64(vb),
                                                G.bits_f64(gb), M, w.block_size, w.scale)
    for n, ref in (("dq", dQ), ("dk", dK), ("dv", dV)):
        got = G.to_f64(out[n])
        assert np.isfinite(got).all(), n
        for b in range(Bt):
            for h in range(H):
                assert G.rel_l2(got[b, h], ref[b, h]) <= GRAD_TOL, (n, b, h)
    return (qb, kb, vb, gb), out


@pytest.mark.parametrize("name,heads,batch,seqlen", [
    ("1p3b_8k", 8, 2, 1024),
    ("7b_32k", 16, 1, 2048),
    ("7b_128k", 4, 1, 2048),     # 128-token blocks: a list entry is two chunks
    ("1p3b_8k", 3, 3, 384),      # odd head count, three tiles
    ("1p3b_8k", 2, 1, 128),      # one tile: only diagonal pieces
    ("7b_32k", 9, 1, 4096),      # more heads than one per XCD, long stripe tiles
])
def test_small_cases(name, heads, batch, seqlen):
    _check(synth.WORKLOADS[name], heads, batch, seqlen)


def test_variants_window_swa_and_sparse_rows():
    base = synth.WORKLOADS["1p3b_8k"]
    for kw in (dict(stride=0), dict(window_blocks=6), dict(local_blocks=1, stride=3), dict(local_blocks=1, stride=0)):
        _check(dataclasses.replace(base, **kw), 4, 1, 1024)


def test_agrees_with_the_recomputing_backward_and_repeats_bitwise():
    w = synth.WORKLOADS["1p3b_8k"]
    ins, a = _check(w, 8, 1, 1024)
    b = G.run_fwd_bwd(w, *ins, keep_ds=True)
    c = G.run_fwd_bwd(w, *ins)
    for n in ("dq", "dk", "dv"):
        assert torch.equal(a[n], b[n]), n
    # dV does not depend on delta: the two paths compute it with the same instructions
    assert torch.equal(a["dv"], c["dv"])
    # dK and dQ differ only through the order in which delta is summed and dS's rounding
    for n in ("dq", "dk"):
        assert G.rel_l2(G.to_f64(a[n]), G.to_f64(c[n])) <= 5e-3, n


def test_custom_pattern_and_sink():
    w = synth.WORKLOADS["1p3b_8k"]
    H, N = 3, 1024
    Bk = N // w.block_size
    M = orc.with_sink(orc.block_mask(H, Bk, 2, 5), 1)
    rng = np.random.default_rng(5)
    extra = np.tril(rng.random((H, Bk, Bk)) < 0.2)
    M = M | extra
    row_ptr, col_idx, _, _ = orc.compressed_layout(M)
    lay = B.s2_layout_from_csr(H, Bk, w.block_size, row_ptr, col_idx)
    qb, kb, vb, gb = synth.train_inputs(w, heads=H, batch=2, seqlen=N)
    q, k, v, g = (G.to_dev(x) for x in (qb, kb, vb, gb))
    o = torch.empty_like(q)
    lse = torch.empty((2, H, N), dtype=torch.float32, device="cuda")
    dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(3))
    ws = torch.full((B.s2_attn_bwd_layout_workspace_bytes(lay, 2, H, N, w.head_dim),), 0xFF, dtype=torch.uint8, device="cuda")
    B.s2_attn_fwd(lay, q, k, v, o, lse, w.scale)
    B.s2_attn_bwd(lay, q, k, v, o, lse, g, dq, dk, dv, w.scale, ws)
    torch.cuda.synchronize()
    ref = orc.attention_backward(G.bits_f64(qb), G.bits_f64(kb), G.bits_f64(vb), G.bits_f64(gb), M, w.block_size, w.scale)
    for got, want, n in zip((dq, dk, dv), ref[:3], ("dq", "dk", "dv")):
        gf = G.to_f64(got)
        for b in range(2):
            for h in range(H):
                assert G.rel_l2(gf[b, h], want[b, h]) <= GRAD_TOL, (n, b, h)


def test_stage_by_stage_and_strided_tensors():
    """delta, dK/dV and dQ as three calls on one workspace give what one call gives; tensors stored
    [batch, token, head, feature] and K / V rows longer than head_dim."""
    w = synth.WORKLOADS["1p3b_8k"]
    H, Bt, N, D = 3, 2, 768, w.head_dim
    qb, kb, vb, gb = synth.train_inputs(w, heads=H, batch=Bt, seqlen=N)

    def strided(bits, pad):
        base = torch.zeros((Bt, N, H, D + pad), dtype=torch.bfloat16, device="cuda")
        view = base[..., :D].permute(0, 2, 1, 3)
        view.copy_(G.to_dev(bits))
        return view

    q, g = strided(qb, 0), strided(gb, 0)
    k, v = strided(kb, 64), strided(vb, 64)
    o = torch.zeros((Bt, N, H, D), dtype=torch.bfloat16, device="cuda").permute(0, 2, 1, 3)
    lse = torch.empty((Bt, H, N), dtype=torch.float32, device="cuda")
    lay = B.s2_layout_build(B.layout_params(H, N // w.block_size, w.block_size, w.local_blocks, w.stride))
    B.s2_attn_fwd(lay, q, k, v, o, lse, w.scale)
    outs = []
    for staged in (False, True):
        dq = torch.zeros((Bt, N, H, D), dtype=torch.bfloat16, device="cuda").permute(0, 2, 1, 3)
        dk = torch.zeros((Bt, N, H, D + 64), dtype=torch.bfloat16, device="cuda")[..., :D].permute(0, 2, 1, 3)
        dv = torch.zeros((Bt, N, H, D + 64), dtype=torch.bfloat16, device="cuda")[..., :D].permute(0, 2, 1, 3)
        ws = torch.full((B.s2_attn_bwd_layout_workspace_bytes(lay, Bt, H, N, D),), 0xFF, dtype=torch.uint8, device="cuda")
        if staged:
            for st in (B.BWD_DELTA, B.BWD_DKDV, B.BWD_DQ):
                B.s2_attn_bwd_stages(lay, q, k, v, o, lse, g, dq, dk, dv, w.scale, ws, st)
        else:
            B.s2_attn_bwd(lay, q, k, v, o, lse, g, dq, dk, dv, w.scale, ws)
        torch.cuda.synchronize()
        outs.append((dq, dk, dv))
    for a, b in zip(*outs):
        assert torch.equal(a, b)
    M = G.oracle_mask(w, H, N)
    ref = orc.attention_backward(G.bits_f64(qb), G.bits_f64(kb), G.bits_f64(vb), G.bits_f64(gb), M, w.block_size, w.scale)
    for got, want in zip(outs[0], ref[:3]):
        assert G.rel_l2(G.to_f64(got), want) <= GRAD_TOL


def test_smaller_workspace_takes_the_other_path_and_one_byte_short_too():
    w = synth.WORKLOADS["1p3b_8k"]
    qb, kb, vb, gb = synth.train_inputs(w, heads=2, batch=1, seqlen=512)
    q, k, v, g = (G.to_dev(x) for x in (qb, kb, vb, gb))
    o = torch.empty_like(q)
    lse = torch.empty((1, 2, 512), dtype=torch.float32, device="cuda")
    lay = B.s2_layout_build(B.layout_params(2, 512 // w.block_size, w.block_size, w.local_blocks, w.stride))
    B.s2_attn_fwd(lay, q, k, v, o, lse, w.scale)
    big = B.s2_attn_bwd_layout_workspace_bytes(lay, 1, 2, 512, w.head_dim)
    res = []
    for nbytes in (B.s2_attn_bwd_workspace_bytes(1, 2, 512, w.head_dim), big - 1, big):
        dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(3))
        ws = torch.full((big,), 0xFF, dtype=torch.uint8, device="cuda")
        B.s2_attn_bwd(lay, q, k, v, o, lse, g, dq, dk, dv, w.scale, ws[:nbytes])
        torch.cuda.synchronize()
        res.append((dq, dk, dv))
    for a, b in zip(res[0], res[1]):
        assert torch.equal(a, b), "one byte short of the larger size: the recomputing path, bit for bit"
    for a, b in zip(res[0], res[2]):
        assert G.rel_l2(G.to_f64(b), G.to_f64(a)) <= 5e-3


def _sweep_cases(n, seed=20240719):
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(n):
        S = int(rng.choice([64, 128]))
        H = int(rng.integers(1, 10))
        batch = int(rng.integers(1, 4))
        Bk = int(rng.integers(1, 13 if S == 64 else 9)) * (2 if S == 64 else 1)   # whole 128-row tiles
        B_l = int(rng.integers(1, min(Bk, 6) + 2))          # may exceed the number of blocks
        stride = int(rng.choice([0, 1, 2, 3, 5, 8, 11]))
        base = int(rng.integers(0, 9))
        window = int(rng.choice([0, 0, 0, 4, 9]))
        out.append((S, H, batch, Bk, B_l, stride, base, window))
    return out


@pytest.mark.parametrize("case", _sweep_cases(20), ids=lambda c: "S%d_H%d_b%d_B%d_L%d_V%d_o%d_w%d" % c)
def test_random_case(case):
    """A seeded sweep over block size, heads, batch, length, window, stride, head index base and stripe
    window, each through the backward that keeps dS, against the fp64 oracle."""
    S, H, batch, Bk, B_l, stride, base, window = case
    N, D = Bk * S, 128
    w = dataclasses.replace(synth.WORKLOADS["1p3b_8k"], block_size=S, local_blocks=B_l, stride=stride,
                            window_blocks=window)
    print("keep-dS sweep case", case, flush=True)
    qb, kb, vb, gb = synth.train_inputs(w, heads=H, batch=batch, seqlen=N)
    lay = B.s2_layout_build(B.layout_params(H, Bk, S, B_l, stride, base, window, 0))
    M = orc.block_mask(H, Bk, B_l, stride, base, window)
    q, k, v, g = G.to_dev(qb), G.to_dev(kb), G.to_dev(vb), G.to_dev(gb)
    o = torch.empty_like(q)
    lse = torch.empty((batch, H, N), dtype=torch.float32, device="cuda")
    dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(3))
    nbytes = B.s2_attn_bwd_layout_workspace_bytes(lay, batch, H, N, D)
    assert nbytes > B.s2_attn_bwd_workspace_bytes(batch, H, N, D)
    ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")
    B.s2_attn_fwd(lay, q, k, v, o, lse, w.scale)
    B.s2_attn_bwd(lay, q, k, v, o, lse, g, dq, dk, dv, w.scale, ws)
    torch.cuda.synchronize()
    dQ, dK, dV, O, LSE = orc.attention_backward(G.bits_f64(qb), G.bits_f64(kb), G.bits_f64(vb), G.bits_f64(gb),
                                                M, S, w.scale)
    for n, got_t, ref in (("dq", dq, dQ), ("dk", dk, dK), ("dv", dv, dV)):
        got = G.to_f64(got_t)
        assert np.isfinite(got).all(), n
        for b in range(batch):
            for h in range(H):
                assert G.rel_l2(got[b, h], ref[b, h]) <= GRAD_TOL, (n, b, h)


@pytest.mark.parametrize("heads,seqlen,local", [(4, 1024, 2), (12, 4096, 16)])  # dS smaller and larger than the room to cut tiles
def test_room_for_ds_alone_keeps_it(heads, seqlen, local):
    w = dataclasses.replace(synth.WORKLOADS["1p3b_8k"], local_blocks=local)
    q, k, v, g = (G.to_dev(x) for x in synth.train_inputs(w, heads=heads, batch=1, seqlen=seqlen))
    lay = B.s2_layout_build(B.layout_params(heads, seqlen // w.block_size, w.block_size, local, w.stride))
    o, lse = torch.empty_like(q), torch.empty((1, heads, seqlen), dtype=torch.float32, device="cuda")
    B.s2_attn_fwd(lay, q, k, v, o, lse, w.scale)
    stats = 2 * ((heads * seqlen * 4 + 255) // 256 * 256)
    plain = B.s2_attn_bwd_workspace_bytes(1, heads, seqlen, 128)
    ds = B.s2_attn_bwd_layout_workspace_bytes(lay, 1, heads, seqlen, 128) - plain
    assert (ds > plain - stats) == (local == 16)

    def dq(size):
        ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")
        grads = [torch.full_like(q, float("nan")) for _ in range(3)]
        B.s2_attn_bwd(lay, q, k, v, o, lse, g, *grads, w.scale, ws)
        return grads[0], ws

    kept, _ = dq(plain + ds)
    again, _ = dq(stats)
    assert not torch.equal(kept, again)  # (dQ from the bf16 dS, or from scores formed a second time)
    for size in (stats + ds, stats + ds + 256):
        got, ws = dq(size)
        assert torch.equal(got, kept) and not (ws[stats:stats + 8192] == 0xFF).all()
    # the plain size, and what is no more than it, recomputes
    for size in (plain, stats + 256):
        assert torch.equal(dq(size)[0], again)
