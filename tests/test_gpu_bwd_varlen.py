"""GPU parity of the backward on packed variable-length batches (s2_attn_bwd_varlen) against the
fp64 oracle: ragged lengths, empty sequences, rows owned by no sequence, every block size, a custom
pattern, and bit-identity with the fixed-length backward."""

import dataclasses

import numpy as np
import pytest
import torch

from oracle import s2_oracle as orc
from paper_2407_17678_amd import binding as B
from paper_2407_17678_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

LSE_TOL, GRAD_TOL = 1e-3, 2e-2
SENTINEL = 0x4248  # bf16 50.0: what the outputs hold where the kernels must not write


def _run(w, H, lens, Bk, M=None, extra_rows=0):
    S, D = w.block_size, w.head_dim
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    total = int(cu[-1]) + extra_rows
    qb, kb, vb, gb = synth.train_inputs(w, heads=H, batch=1, seqlen=total)
    if M is None:
        M = orc.block_mask(H, Bk, w.local_blocks, w.stride)
        lay = B.s2_layout_build(B.layout_params(H, Bk, S, w.local_blocks, w.stride))
    else:
        row_ptr, col_idx, _, _ = orc.compressed_layout(M)
        lay = B.s2_layout_from_csr(H, Bk, S, row_ptr, col_idx)
    q, k, v, g = G.to_dev(qb), G.to_dev(kb), G.to_dev(vb), G.to_dev(gb)
    sent = lambda: torch.full_like(q.view(torch.int16), SENTINEL).view(q.dtype)
    o, dq, dk, dv = sent(), sent(), sent(), sent()
    lse = torch.full((H, total), 77.0, dtype=torch.float32, device="cuda")
    cud = torch.from_numpy(cu).cuda()
    # the workspace starts out as NaN: the slack the kernels read past a sequence's end must not matter
    ws = torch.full((B.s2_attn_bwd_varlen_workspace_bytes(H, total, D) // 4,), float("nan"), dtype=torch.float32,
                    device="cuda")
    B.s2_attn_fwd_varlen(lay, q, k, v, o, lse, cud, Bk * S, w.scale)
    B.s2_attn_bwd_varlen(lay, q, k, v, o, lse, g, dq, dk, dv, cud, Bk * S, w.scale, ws)
    torch.cuda.synchronize()
    return (qb, kb, vb, gb), cu, M, dict(o=o, lse=lse, dq=dq, dk=dk, dv=dv)


def _check(bits, cu, M, S, scale, out, end):
    f = G.bits_f64
    qb, kb, vb, gb = bits
    dQ, dK, dV, O, LSE = orc.attention_backward_varlen(f(qb)[0], f(kb)[0], f(vb)[0], f(gb)[0], cu, M, S, scale)
    assert G.o_excess(G.to_f64(out["o"])[0, :, :end], O[:, :end]) <= 0
    assert np.abs(G.to_f64(out["lse"])[:, :end] - LSE[:, :end]).max() <= LSE_TOL
    for n, ref in (("dq", dQ), ("dk", dK), ("dv", dV)):
        got = G.to_f64(out[n])[0, :, :end]
        assert np.isfinite(got).all(), n
        # per sequence, so that a short sequence is not drowned by a long one
        # (a one-token sequence has dQ = dK = 0 exactly: the relative bound gets an absolute floor of
        # 1e-3 rms, far below the gradients' own scale of about 1)
        for lo, hi in zip(cu[:-1], cu[1:]):
            if hi > lo:
                a, b = got[:, lo:hi], ref[:, lo:hi]
                err = np.linalg.norm(a - b)
                assert err <= GRAD_TOL * max(np.linalg.norm(b), 1e-3 * np.sqrt(b.size)), (n, int(lo), int(hi), err)
        assert (out[n].view(torch.int16)[0, :, end:] == SENTINEL).all(), n


CASES = {
    # name: (workload for D / seed, S, heads, layout blocks, B_l, stride, lengths)
    "S64_D128": ("1p3b_8k", 64, 3, 16, 2, 3, [1, 127, 128, 129, 700, 64, 0, 333, 1024]),
    "S16_D64": ("tiny", 16, 4, 16, 2, 5, [5, 16, 17, 31, 100, 250, 256, 33]),
    "S128_D128": ("7b_128k", 128, 2, 8, 2, 3, [130, 384, 1, 1000, 257]),
    "S32_D128": ("1p3b_8k", 32, 3, 20, 3, 4, [31, 32, 33, 95, 640, 2, 161]),
    "S64_D64_many_short": ("tiny", 64, 2, 4, 1, 2, [3, 9, 1, 64, 65, 12, 200, 7, 130, 256, 40, 99, 128, 5]),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_varlen_backward_against_the_oracle(case):
    wname, S, H, Bk, B_l, s, lens = CASES[case]
    w = dataclasses.replace(synth.WORKLOADS[wname], block_size=S, local_blocks=B_l, stride=s)
    print("varlen backward case", case, "H", H, "S", S, "B", Bk, "lens", lens, flush=True)
    bits, cu, M, out = _run(w, H, lens, Bk, extra_rows=70)
    _check(bits, cu, M, S, w.scale, out, int(cu[-1]))


def test_varlen_backward_custom_pattern():
    w = dataclasses.replace(synth.WORKLOADS["1p3b_8k"], block_size=32)
    H, Bk, S = 2, 24, 32
    rng = np.random.default_rng(17)
    M = np.tril(rng.random((H, Bk, Bk)) < 0.3)
    i = np.arange(Bk)
    M[:, i, i] = True
    bits, cu, M, out = _run(w, H, [700, 45, 768, 129], Bk, M=M)
    _check(bits, cu, M, S, w.scale, out, int(cu[-1]))


def test_varlen_backward_agrees_with_the_fixed_length_backward():
    # differently scheduled kernels may run behind the two entry points: agreement to rounding (the
    # gradients are bf16: relative L2 of the difference well below the 2e-2 either is held to)
    # each sequence on its own through s2_attn_fwd / s2_attn_bwd (lengths they accept: whole blocks)
    w = dataclasses.replace(synth.WORKLOADS["1p3b_8k"], block_size=64, local_blocks=2, stride=3)
    H, Bk, S, D = 3, 12, 64, 128
    lens = [768, 64, 320, 128]
    bits, cu, M, out = _run(w, H, lens, Bk)
    q, k, v, g = (G.to_dev(x) for x in bits)
    for sq, L in enumerate(lens):
        lo = int(cu[sq])
        lay = B.s2_layout_build(B.layout_params(H, L // S, S, w.local_blocks, w.stride))
        qs, ks, vs, gs = (x[:, :, lo:lo + L].contiguous() for x in (q, k, v, g))
        o1 = torch.empty_like(qs)
        lse1 = torch.empty((1, H, L), dtype=torch.float32, device="cuda")
        d1 = [torch.empty_like(qs) for _ in range(3)]
        ws = torch.empty(B.s2_attn_bwd_workspace_bytes(1, H, L, D), dtype=torch.uint8, device="cuda")
        B.s2_attn_fwd(lay, qs, ks, vs, o1, lse1, w.scale)
        B.s2_attn_bwd(lay, qs, ks, vs, o1, lse1, gs, d1[0], d1[1], d1[2], w.scale, ws)
        torch.cuda.synchronize()
        for n, t in zip(("dq", "dk", "dv"), d1):
            assert G.rel_l2(G.to_f64(t), G.to_f64(out[n][:, :, lo:lo + L])) <= 5e-3, (sq, n)


def test_varlen_seeded_sweep_around_the_tile_size():
    """Random packed batches for head_dim 128 and blocks of 64 and 128 tokens, lengths drawn around the
    multiples of 128, where a sequence's partial last tile begins: lengths of exactly k * 128, one more, one
    less, below 128 and zero all occur, with random local-window and stride parameters."""
    rng = np.random.default_rng(2024)
    for case in range(10):
        S = int(rng.choice([64, 128]))
        H = int(rng.integers(1, 4))
        Bk = int(rng.integers(2, 9)) * (2 if S == 64 else 1)
        max_len = Bk * S
        lens = []
        for _ in range(int(rng.integers(2, 7))):
            base = int(rng.integers(0, max_len // 128 + 1)) * 128
            lens.append(int(np.clip(base + int(rng.choice([-1, 0, 0, 1, 5, -37, 64])), 0, max_len)))
        lens.append(int(rng.integers(0, 128)))
        w = dataclasses.replace(synth.WORKLOADS["1p3b_8k"], block_size=S, local_blocks=int(rng.integers(1, 4)),
                                stride=int(rng.integers(0, 5)))
        print("varlen sweep case", case, "S", S, "H", H, "B", Bk, "local", w.local_blocks, "stride", w.stride, "lens", lens,
              flush=True)
        bits, cu, M, out = _run(w, H, lens, Bk, extra_rows=int(rng.integers(0, 70)))
        _check(bits, cu, M, S, w.scale, out, int(cu[-1]))


@pytest.mark.parametrize("D,S", [(64, 16), (64, 32), (64, 128), (128, 16), (128, 32)])
def test_varlen_short_sequences_in_a_long_layout(D, S):
    """Sequences from one token to the whole of a layout whose lists are longer than the 64 entries held at a time
    (16- and 32-token blocks), so that the entries after a short sequence's end, which its key tiles skip, are in other
    batches of 64 than the ones they use, and a wavefront's columns lie far apart, one of them past the end."""
    rng = np.random.default_rng(100 * D + S)
    H, Bk = 2, 2560 // S
    M = np.tril(rng.random((H, Bk, Bk)) < 0.7)
    M[:, np.arange(Bk), np.arange(Bk)] = True
    w = dataclasses.replace(synth.WORKLOADS["tiny" if D == 64 else "1p3b_8k"], block_size=S)
    lens = [2560, 1, S, 2 * S + 1, 700, 0, 129, 1290]
    print("varlen long layout case D", D, "S", S, flush=True)
    bits, cu, M, out = _run(w, H, lens, Bk, M=M, extra_rows=3)
    _check(bits, cu, M, S, w.scale, out, int(cu[-1]))


def test_varlen_the_longest_sequence_of_16_token_blocks():
    # 65536 blocks, the most a layout takes: partner indices use all sixteen bits
    S, Bk, D = 16, 65536, 64
    N = S * Bk
    lay = B.s2_layout_build(B.layout_params(1, Bk, S, 2, 0))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    q, k, v, g = (torch.empty((1, 1, N, D), dtype=torch.bfloat16, device="cuda").normal_(generator=gen) for _ in range(4))
    o, dq, dk, dv = (torch.full_like(q, float("nan")) for _ in range(4))
    lse = torch.empty((1, N), dtype=torch.float32, device="cuda")
    cu = torch.tensor([0, N], dtype=torch.int32, device="cuda")
    ws = torch.empty(B.s2_attn_bwd_varlen_workspace_bytes(1, N, D), dtype=torch.uint8, device="cuda")
    B.s2_attn_fwd_varlen(lay, q, k, v, o, lse, cu, N, D ** -0.5)
    B.s2_attn_bwd_varlen(lay, q, k, v, o, lse, g, dq, dk, dv, cu, N, D ** -0.5, ws)
    # a local window of two blocks: the first and the last 320 rows but their margins, as sequences of their own
    M = orc.block_mask(1, 20, 2, 0)
    for lo in (0, N - 320):
        f = lambda x: G.to_f64(x[0, :, lo:lo + 320])[None]
        ref = orc.attention_backward(f(q), f(k), f(v), f(g), M, S, D ** -0.5)
        rows = slice(0, 288) if lo == 0 else slice(32, 320)
        assert G.o_excess(f(o)[0, :, rows], ref[3][0, :, rows]) <= 0
        for n, t, want in zip(("dq", "dk", "dv"), (dq, dk, dv), ref):
            assert G.rel_l2(f(t)[0, :, rows], want[0, :, rows]) <= GRAD_TOL, (n, lo)


def test_varlen_row_offsets_that_make_no_sense_stay_inside_the_tensors():
    """cu_seqlens is a device array the host cannot check: negative entries, entries far beyond the tensors,
    decreasing ones.  The kernels cut every sequence to the rows that exist and to max_seqlen, so such a call
    must complete, leave the rows no (cut) sequence owns alone, and still compute the sequences that are in
    order and overlap nothing - forward and backward."""
    w = dataclasses.replace(synth.WORKLOADS["1p3b_8k"], local_blocks=2, stride=3)
    H, Bk, S, D = 2, 8, w.block_size, w.head_dim
    total, max_len = 1600, Bk * S
    big = 2_000_000_000
    cu = np.array([-big, -3, 600, 900, big, 1450, 1500, 1600], dtype=np.int32)
    # as the kernels read it: rows 0..511 (twice), 600..899, 900..1411, nothing, 1450..1499, 1500..1599
    valid = [(600, 300), (1450, 50), (1500, 100)]
    qb, kb, vb, gb = synth.train_inputs(w, heads=H, batch=1, seqlen=total)
    M = orc.block_mask(H, Bk, w.local_blocks, w.stride)
    lay = B.s2_layout_build(B.layout_params(H, Bk, S, w.local_blocks, w.stride))
    q, k, v, g = G.to_dev(qb), G.to_dev(kb), G.to_dev(vb), G.to_dev(gb)
    sent = lambda: torch.full_like(q.view(torch.int16), SENTINEL).view(q.dtype)
    o, dq, dk, dv = sent(), sent(), sent(), sent()
    lse = torch.full((H, total), 77.0, dtype=torch.float32, device="cuda")
    cud = torch.from_numpy(cu).cuda()
    ws = torch.zeros(B.s2_attn_bwd_varlen_workspace_bytes(H, total, D), dtype=torch.uint8, device="cuda")
    print("varlen case with senseless row offsets", cu.tolist(), flush=True)
    B.s2_attn_fwd_varlen(lay, q, k, v, o, lse, cud, max_len, w.scale)
    B.s2_attn_bwd_varlen(lay, q, k, v, o, lse, g, dq, dk, dv, cud, max_len, w.scale, ws)
    torch.cuda.synchronize()
    f = G.bits_f64
    for lo, L in valid:
        for h in range(H):
            sl = lambda x: f(x)[0, h, lo:lo + L]
            dQ, dK, dV, O, LSE = orc.attention_backward_head(sl(qb), sl(kb), sl(vb), sl(gb), M[h], S, w.scale)
            assert G.o_excess(G.to_f64(o)[0, h, lo:lo + L], O) <= 0, (lo, h)
            assert np.abs(G.to_f64(lse)[h, lo:lo + L] - LSE).max() <= LSE_TOL, (lo, h)
            for n, got, ref in (("dq", dq, dQ), ("dk", dk, dK), ("dv", dv, dV)):
                assert G.rel_l2(G.to_f64(got)[0, h, lo:lo + L], ref) <= GRAD_TOL, (n, lo, h)
    for t in (o, dq, dk, dv):
        # rows 512..599 and 1412..1449 belong to no sequence as the kernels cut them
        assert (t.view(torch.int16)[0, :, 512:600] == SENTINEL).all()
        assert (t.view(torch.int16)[0, :, 1412:1450] == SENTINEL).all()
        assert torch.isfinite(t[0, :, :512].float()).all() and torch.isfinite(t[0, :, 900:1412].float()).all()


def test_more_key_tiles_than_a_grid_holds_are_refused():
    # 129 tiles of each of 16647159 pairs are dealt out in runs of four: fewer than 2^31 tiles, more than 2^31 workgroups
    seqs, rows, D = 16647159, 128, 64
    lay = B.s2_layout_build(B.layout_params(1, 129, 128, 1, 2))
    t = [torch.zeros((1, 1, rows, D), dtype=torch.bfloat16, device="cuda") for _ in range(8)]
    lse = torch.zeros((1, rows), dtype=torch.float32, device="cuda")
    cu = torch.full((seqs + 1,), rows, dtype=torch.int32, device="cuda")
    cu[0] = 0                                                   # one sequence of all rows, the others empty
    ws = torch.empty(B.s2_attn_bwd_varlen_workspace_bytes(1, rows, D), dtype=torch.uint8, device="cuda")
    with pytest.raises(B.S2Error) as e:
        B.s2_attn_bwd_varlen(lay, *t[:4], lse, *t[4:], cu, rows, 1.0, ws)
    assert e.value.status == -3
