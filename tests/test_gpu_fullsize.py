"""Parity at the full workload sizes, in the launch configuration bench.py times.

The oracle cannot afford every output at these sizes, so: forward rows are independent and are
sampled (each sampled row is computed by the oracle from all N keys); the backward is checked on
whole heads (one head of the 32K workload costs the oracle about ten seconds)."""

import numpy as np
import pytest
import torch

from oracle import s2_oracle as orc
from paper_2407_17678_amd import binding as B
from paper_2407_17678_amd import synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def _sample_rows(N, S, B_l, rng, n_random=24):
    fixed = [0, 1, S - 1, S, S * B_l - 1, S * B_l, S * B_l + 1, N // 2, N - S - 1, N - S, N - 1]
    rows = sorted(set(fixed) | set(int(x) for x in rng.integers(0, N, size=n_random)))
    return np.array(rows)


def _check_forward_rows(w, o, lse, bits, heads, rng):
    qb, kb, vb = bits
    N, S = w.seqlen, w.block_size
    M = orc.block_mask(w.heads, N // S, w.local_blocks, w.stride)
    for (b, h) in heads:
        rows = _sample_rows(N, S, w.local_blocks, rng)
        f = lambda x: G.bits_f64(x[b, h])
        O, LSE = orc.forward_rows(f(qb)[rows], rows, f(kb), f(vb), M[h], S, w.scale)
        go = G.to_f64(o[b, h][torch.from_numpy(rows).cuda()])
        gl = G.to_f64(lse[b, h][torch.from_numpy(rows).cuda()])
        assert G.o_excess(go, O) <= 0, (b, h)
        assert np.abs(gl - LSE).max() <= 1e-3, (b, h)


def _check_backward_head(w, outs, bits, b, h, stripe_columns=False):
    """`outs`: results of the two forms of the backward (small workspace: the dQ launch recomputes S
    and dP; larger workspace: dS kept between the launches), both held to the oracle's one result."""
    qb, kb, vb, gb = bits
    S = w.block_size
    M = orc.block_mask(w.heads, w.seqlen // S, w.local_blocks, w.stride)
    f = lambda x: G.bits_f64(x[b, h])
    dQ, dK, dV, O, LSE = orc.attention_backward_head(f(qb), f(kb), f(vb), f(gb), M[h], S, w.scale)
    for which, out in outs.items():
        assert G.o_excess(G.to_f64(out["o"][b, h]), O) <= 0
        assert np.abs(G.to_f64(out["lse"][b, h]) - LSE).max() <= 1e-3
        for n, ref in (("dq", dQ), ("dk", dK), ("dv", dV)):
            e = G.rel_l2(G.to_f64(out[n][b, h]), ref)
            print("   %s head (%d,%d) %s rel-L2 %.3e" % (n, b, h, which, e), flush=True)
            assert e <= 2e-2, (which, n, b, h, e)
        if stripe_columns and w.stride > 0:
            # The key blocks on this head's stripes are attended by every later query block: their dK / dV
            # rows come from the longest key tiles (hundreds of steps) and are a small part of the head's
            # norm, so they are held to the bound on their own as well.
            nb = w.seqlen // S
            cols = np.arange(h % w.stride, nb, w.stride)
            rows = (cols[:, None] * S + np.arange(S)[None, :]).ravel()
            for n, ref in (("dk", dK), ("dv", dV)):
                e = G.rel_l2(G.to_f64(out[n][b, h])[rows], ref[rows])
                print("   %s head (%d,%d) %s stripe columns rel-L2 %.3e" % (n, b, h, which, e), flush=True)
                assert e <= 2e-2, (which, n, b, h, e)


def _both_backwards(w, bits):
    outs = {"recomputing": G.run_fwd_bwd(w, *bits), "keeping dS": G.run_fwd_bwd(w, *bits, keep_ds=True)}
    assert outs["keeping dS"]["ws_bytes"] > outs["recomputing"]["ws_bytes"]
    return outs


def test_1p3b_8k_full():
    w = synth.WORKLOADS["1p3b_8k"]
    print("full-size case", w.name, flush=True)
    bits = synth.train_inputs(w)
    outs = _both_backwards(w, bits)
    out = outs["recomputing"]
    rng = np.random.default_rng(1)
    _check_forward_rows(w, out["o"], out["lse"], bits[:3], [(b, (5 * b + 2 * k) % w.heads) for b in range(w.batch) for k in range(2)], rng)
    for b in range(w.batch):          # every (batch, head) pair: under a second of oracle each
        for h in range(w.heads):
            _check_backward_head(w, outs, bits, b, h, stripe_columns=(h % 5 == 0))
    # every output finite and nothing left unwritten
    for out in outs.values():
        for n in ("o", "dq", "dk", "dv"):
            assert torch.isfinite(out[n].float()).all()


def test_7b_32k_full():
    w = synth.WORKLOADS["7b_32k"]
    print("full-size case", w.name, flush=True)
    bits = synth.train_inputs(w)
    outs = _both_backwards(w, bits)
    out = outs["recomputing"]
    rng = np.random.default_rng(2)
    _check_forward_rows(w, out["o"], out["lse"], bits[:3], [(0, h) for h in (0, 3, 5, 10, 15, 16, 21, 26, 31)], rng)
    for h in (0, 5, 15, 16, 21, 31):   # both ends of the stripe offsets and between; about ten seconds of oracle each
        _check_backward_head(w, outs, bits, 0, h, stripe_columns=True)
    for out in outs.values():
        for n in ("o", "dq", "dk", "dv"):
            assert torch.isfinite(out[n].float()).all()


def test_7b_32k_backward_repeats_bitwise_at_full_size():
    """Both forms of the backward, ten launches each on the full 7b_32k tensors with the workspace
    scribbled over in between: every launch must reproduce the first bit for bit (the kernels leave
    stores in flight across their waits for the next chunk and read dS back through a second launch; an
    ordering mistake there would show as results that differ from run to run)."""
    w = synth.WORKLOADS["7b_32k"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(77)
    shape = (w.batch, w.heads, w.seqlen, w.head_dim)
    q, k, v, g = (torch.randn(shape, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(4))
    o = torch.empty_like(q)
    lse = torch.empty(shape[:3], dtype=torch.float32, device="cuda")
    lay = B.s2_layout_build(B.layout_params(w.heads, w.seqlen // w.block_size, w.block_size, w.local_blocks, w.stride))
    B.s2_attn_fwd(lay, q, k, v, o, lse, w.scale)
    sizes = (B.s2_attn_bwd_workspace_bytes(*shape), B.s2_attn_bwd_layout_workspace_bytes(lay, *shape))
    assert sizes[1] > sizes[0]
    for nbytes in sizes:
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        first = None
        for rep in range(10):
            ws.random_(0, 255)
            outs = [torch.full_like(q, float("nan")) for _ in range(3)]
            B.s2_attn_bwd(lay, q, k, v, o, lse, g, outs[0], outs[1], outs[2], w.scale, ws)
            torch.cuda.synchronize()
            if first is None:
                first = outs
                assert all(torch.isfinite(t.float()).all() for t in first)
            else:
                for a, b_ in zip(first, outs):
                    assert torch.equal(a, b_), (nbytes, rep)
        del ws


def test_7b_128k_forward_full():
    w = synth.WORKLOADS["7b_128k"]
    print("full-size case", w.name, flush=True)
    rngs = synth.rng_for(w.index)
    shape = (w.batch, w.heads, w.seqlen, w.head_dim)
    qb, kb, vb = (synth.normal_bf16(rngs, shape) for _ in range(3))
    o, lse, _, _ = G.run_fwd(w, qb, kb, vb)
    rng = np.random.default_rng(3)
    _check_forward_rows(w, o, lse, (qb, kb, vb), [(0, h) for h in (0, 4, 7, 13, 18, 22, 27, 31)], rng)
    assert torch.isfinite(o.float()).all()


def test_7b_decode_full():
    """64 sequences x 32 heads against a 34 GB cache filled on the device; the oracle checks a
    sample of (sequence, head) pairs from slices copied back."""
    w = synth.WORKLOADS["7b_decode"]
    print("full-size case", w.name, flush=True)
    nseq, H, D, max_len = w.batch, w.heads, w.head_dim, w.max_len
    lens = synth.decode_lengths(w)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(synth.BASE_SEED + w.index)
    q = torch.randn((nseq, H, D), device="cuda", generator=gen).to(torch.bfloat16)
    kc = torch.empty((nseq, H, max_len, D), dtype=torch.bfloat16, device="cuda")
    vc = torch.empty_like(kc)
    for b in range(nseq):
        kc[b] = torch.randn((H, max_len, D), device="cuda", generator=gen).to(torch.bfloat16)
        vc[b] = torch.randn((H, max_len, D), device="cuda", generator=gen).to(torch.bfloat16)
    sl = torch.from_numpy(lens).cuda()
    o = torch.empty_like(q)
    lse = torch.empty((nseq, H), dtype=torch.float32, device="cuda")
    p = B.layout_params(H, 1, w.block_size, w.local_blocks, w.stride)
    splits = B.s2_attn_decode_default_splits(nseq, H, max_len)
    ws = torch.empty(B.s2_attn_decode_workspace_bytes(nseq, H, D, max_len, splits), dtype=torch.uint8,
                     device="cuda")
    B.s2_attn_decode(p, q, kc, vc, sl, o, lse, w.scale, ws, max_len, num_splits=splits)
    torch.cuda.synchronize()
    assert torch.isfinite(o.float()).all()
    rng = np.random.default_rng(4)
    pairs = {(int(np.argmin(lens)), 0), (int(np.argmax(lens)), 31)}
    while len(pairs) < 24:
        pairs.add((int(rng.integers(0, nseq)), int(rng.integers(0, H))))
    for (b, h) in sorted(pairs):
        L = int(lens[b])
        ref, ref_lse = orc.decode_row(G.to_f64(q[b, h]), G.to_f64(kc[b, h, :L]), G.to_f64(vc[b, h, :L]), L, h,
                                      w.block_size, w.local_blocks, w.stride, w.scale)
        assert G.o_excess(G.to_f64(o[b, h]), ref) <= 0, (b, h)
        assert abs(float(lse[b, h]) - ref_lse) <= 1e-3, (b, h)


def test_7b_decode_paged_full():
    """The same 64 x 32 decode step with the cache as pages: each head holds only the blocks it can
    still attend (about 1/9 of a contiguous cache).  The oracle checks a sample of (sequence, head)
    pairs on their own pages copied back."""
    w = synth.WORKLOADS["7b_decode"]
    print("full-size case", w.name, "paged", flush=True)
    nseq, H, D, max_len, S = w.batch, w.heads, w.head_dim, w.max_len, w.block_size
    lens = synth.decode_lengths(w)
    resident = [[orc.resident_blocks(int(L), h, S, w.local_blocks, w.stride) for h in range(H)] for L in lens]
    max_blocks = max_len // S
    table, num_pages = synth.page_table(resident, max_blocks, index=w.index)
    assert num_pages * S < 0.13 * nseq * H * max_len
    gen = torch.Generator(device="cuda")
    gen.manual_seed(synth.BASE_SEED + w.index)
    q = torch.randn((nseq, H, D), device="cuda", generator=gen).to(torch.bfloat16)
    kp = torch.empty((num_pages, S, D), dtype=torch.bfloat16, device="cuda")
    vp = torch.empty_like(kp)
    for lo in range(0, num_pages, 4096):
        n = min(4096, num_pages - lo)
        kp[lo:lo + n] = torch.randn((n, S, D), device="cuda", generator=gen).to(torch.bfloat16)
        vp[lo:lo + n] = torch.randn((n, S, D), device="cuda", generator=gen).to(torch.bfloat16)
    tb = torch.from_numpy(table).cuda()
    sl = torch.from_numpy(lens).cuda()
    o = torch.empty_like(q)
    lse = torch.empty((nseq, H), dtype=torch.float32, device="cuda")
    missing = torch.zeros(1, dtype=torch.int32, device="cuda")
    p = B.layout_params(H, 1, S, w.local_blocks, w.stride)
    splits = B.s2_attn_decode_default_splits(nseq, H, max_len)
    ws = torch.empty(B.s2_attn_decode_workspace_bytes(nseq, H, D, max_len, splits), dtype=torch.uint8,
                     device="cuda")
    B.s2_attn_decode_paged(p, q, kp, vp, tb, sl, o, lse, w.scale, ws, missing=missing, num_splits=splits)
    torch.cuda.synchronize()
    assert int(missing.item()) == 0
    assert torch.isfinite(o.float()).all()
    rng = np.random.default_rng(4)
    pairs = {(int(np.argmin(lens)), 0), (int(np.argmax(lens)), 31)}
    while len(pairs) < 24:
        pairs.add((int(rng.integers(0, nseq)), int(rng.integers(0, H))))
    for (b, h) in sorted(pairs):
        L = int(lens[b])
        # this pair's pages, renumbered 0..n-1
        held = resident[b][h]
        idx = torch.from_numpy(table[b, h, held].astype(np.int64)).cuda()
        kpool, vpool = G.to_f64(kp[idx]), G.to_f64(vp[idx])
        row = np.full(max_blocks, -1, dtype=np.int32)
        row[held] = np.arange(len(held))
        ref, ref_lse = orc.paged_decode_row(G.to_f64(q[b, h]), kpool, vpool, row, L, h, S, w.local_blocks,
                                            w.stride, w.scale)
        assert G.o_excess(G.to_f64(o[b, h]), ref) <= 0, (b, h)
        assert abs(float(lse[b, h]) - ref_lse) <= 1e-3, (b, h)


def test_7b_prefill_varlen_full():
    # the packed prefill batch bench.py times (12 prompts, 87 418 tokens): sampled rows of every
    # prompt, the ragged last rows among them, each computed by the oracle from that prompt's keys
    w = synth.WORKLOADS["7b_32k"]
    H, D, S = w.heads, w.head_dim, w.block_size
    lens = synth.prefill_lengths(w, 12, 1024)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    total = int(cu[-1])
    print("full-size case 7b_prefill_varlen", lens.tolist(), flush=True)
    qb, kb, vb, _ = synth.train_inputs(w, heads=H, batch=1, seqlen=total)
    lay = B.s2_layout_build(B.layout_params(H, w.num_blocks, S, w.local_blocks, w.stride))
    q, k, v = G.to_dev(qb), G.to_dev(kb), G.to_dev(vb)
    o = torch.empty_like(q)
    lse = torch.empty((H, total), dtype=torch.float32, device="cuda")
    B.s2_attn_fwd_varlen(lay, q, k, v, o, lse, torch.from_numpy(cu).cuda(), w.seqlen, w.scale)
    torch.cuda.synchronize()
    assert torch.isfinite(o.float()).all() and torch.isfinite(lse).all()
    M = orc.block_mask(H, w.num_blocks, w.local_blocks, w.stride)
    rng = np.random.default_rng(4)
    for sq, L in enumerate(lens.tolist()):
        lo = int(cu[sq])
        # (both sides of the line between the whole 128-row tiles and the partial last one are in the sample)
        rows = sorted({0, S - 1, S, L // 2, (L // S) * S - 1, min((L // S) * S, L - 1), L - 2, L - 1,
                       (L // 128) * 128 - 1, min((L // 128) * 128, L - 1)} |
                      set(int(x) for x in rng.integers(0, L, size=6)))
        rows = np.array([r for r in rows if 0 <= r < L])
        for h in (int(rng.integers(0, H)), (5 * sq + 3) % H):
            f = lambda x: G.bits_f64(x[0, h, lo:lo + L])
            O, LSE = orc.forward_rows(f(qb)[rows], rows, f(kb), f(vb), M[h], S, w.scale)
            idx = torch.from_numpy(rows + lo).cuda()
            assert G.o_excess(G.to_f64(o[0, h][idx]), O) <= 0, (sq, h)
            assert np.abs(G.to_f64(lse[h][idx]) - LSE).max() <= 1e-3, (sq, h)
    # the backward of the same packed batch: whole (sequence, head) pairs against the oracle
    gb = synth.train_inputs(w, heads=H, batch=1, seqlen=total)[3]
    g = G.to_dev(gb)
    dq, dk, dv = torch.empty_like(q), torch.empty_like(q), torch.empty_like(q)
    ws = torch.empty(B.s2_attn_bwd_varlen_workspace_bytes(H, total, D), dtype=torch.uint8, device="cuda")
    B.s2_attn_bwd_varlen(lay, q, k, v, o, lse, g, dq, dk, dv, torch.from_numpy(cu).cuda(), w.seqlen, w.scale, ws)
    torch.cuda.synchronize()
    for t in (dq, dk, dv):
        assert torch.isfinite(t.float()).all()
    for sq, h in ((10, 3), (8, 30), (1, 17)):    # 8553, 1966 and 13231 tokens, ragged ends
        lo, L = int(cu[sq]), int(lens[sq])
        f = lambda x: G.bits_f64(x[0, h, lo:lo + L])
        dQ, dK, dV, _, _ = orc.attention_backward_head(f(qb), f(kb), f(vb), f(gb), M[h], S, w.scale)
        for n, got, ref in (("dq", dq, dQ), ("dk", dk, dK), ("dv", dv, dV)):
            e = G.rel_l2(G.to_f64(got[0, h, lo:lo + L]), ref)
            print("   varlen %s seq %d head %d rel-L2 %.3e" % (n, sq, h, e), flush=True)
            assert e <= 2e-2, (n, sq, h, e)
