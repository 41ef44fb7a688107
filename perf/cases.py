"""Performance cases: the calls a program makes of this library, over the sizes it makes them at.

A training step is s2_attn_fwd + s2_attn_bwd (fixed length), s2_attn_fwd_varlen + s2_attn_bwd_varlen
(packed sequences) or the dense pair (the dense layers of a hybrid stack); serving is a whole-prompt or
chunked prefill and one decode step against a contiguous or a paged cache.  Every case keeps what such a
program keeps between calls (layout handle, workspace, output buffers) and passes fresh inputs.
"""

import math

import numpy as np
import torch

from paper_2407_17678_amd import binding as B
from paper_2407_17678_amd import synth

# ------------------------------------------------------------------------------------ cases


def _mask(block_size, local_blocks, stride):
    return {"block_size": block_size, "local_blocks": local_blocks, "stride": stride}


def listed():
    return [
        # the repository's smallest workload: a unit-test sized model, all launch latency
        dict(name="train_tiny", kind="train", batch=1, heads=4, seqlen=512, head_dim=64, keep_ds=False, **_mask(64, 2, 4)),
        # a small model with 64-wide heads at an ordinary context
        dict(name="train_d64_4k", kind="train", batch=2, heads=16, seqlen=4096, head_dim=64, keep_ds=False, **_mask(64, 4, 8)),
        # a context that is not a multiple of the kernels' 128-row tiles (61 blocks)
        dict(name="train_odd", kind="train", batch=2, heads=16, seqlen=3904, head_dim=128, keep_ds=True, **_mask(64, 4, 8)),
        # the 1.3B training shape
        dict(name="train_1p3b_8k", kind="train", batch=4, heads=16, seqlen=8192, head_dim=128, keep_ds=True, **_mask(64, 4, 8)),
        # the 7B long-context training shape (the default benchmark)
        dict(name="train_7b_32k", kind="train", batch=1, heads=32, seqlen=32768, head_dim=128, keep_ds=True, **_mask(64, 16, 16)),
        # the finest shards the mask allows, 256 local tokens and a stripe every 512
        dict(name="train_fine_8k", kind="train", batch=1, heads=16, seqlen=8192, head_dim=128, keep_ds=False, **_mask(16, 16, 32)),
        # a training batch of packed documents of any length
        dict(name="train_packed", kind="train_packed", nseq=8, heads=32, min_len=200, max_len=8192, head_dim=128, len_seed=11,
             **_mask(64, 16, 16)),
        # one of the dense layers of a hybrid stack
        dict(name="train_dense_8k", kind="train_dense", batch=1, heads=32, seqlen=8192, head_dim=128),
        # a whole 128K prompt
        dict(name="prefill_7b_128k", kind="prefill", batch=1, heads=32, seqlen=131072, head_dim=128, **_mask(128, 8, 32)),
        # one chunk of a long prompt against what is cached of it so far
        dict(name="prefill_chunk", kind="prefill_chunk", batch=1, heads=32, context=30720, rows=2048, head_dim=128,
             **_mask(64, 16, 16)),
        # a single user's decode step
        dict(name="decode_one_32k", kind="decode", nseq=1, heads=32, min_len=32768, max_len=32768, head_dim=128, len_seed=5,
             **_mask(64, 16, 16)),
        # a serving batch's decode step against a paged cache of 16-token blocks
        dict(name="decode_paged_64", kind="decode_paged", nseq=64, heads=32, min_len=8192, max_len=32768, head_dim=128, len_seed=5,
             **_mask(16, 64, 64)),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_mask(rng):
    S = rng.choice([16, 32, 64, 64, 64, 128])
    local = max(1, round(_log_uniform(rng, 64, 1024) / S))
    stride = max(2, round(_log_uniform(rng, 256, 2048) / S))
    return _mask(S, local, stride)


def draw(rng):
    while True:
        kind = rng.choice(["train", "train", "train", "train_packed", "train_dense", "prefill", "prefill_chunk", "decode",
                           "decode_paged"])
        case = dict(kind=kind, head_dim=rng.choice([64, 128, 128]))
        if kind in ("train", "prefill", "train_dense"):
            case.update(batch=rng.randint(1, 4), heads=rng.randint(2, 40))
            tokens = _log_uniform(rng, 512, 32768 if kind != "prefill" else 131072)
            if kind == "train_dense":
                case.update(seqlen=128 * max(1, round(tokens / 128)))
            else:
                case.update(_draw_mask(rng))
                unit = max(32, case["block_size"])
                case.update(seqlen=unit * max(1, round(tokens / unit)))
            if kind == "train":
                case.update(keep_ds=rng.random() < 0.5)
        elif kind == "train_packed":
            case.update(nseq=rng.randint(2, 24), heads=rng.randint(2, 40), min_len=rng.randint(1, 512),
                        max_len=128 * rng.randint(8, 128), len_seed=rng.randrange(1 << 20), **_draw_mask(rng))
        elif kind == "prefill_chunk":
            case.update(batch=rng.randint(1, 4), heads=rng.randint(2, 40), context=128 * rng.randint(0, 500),
                        rows=128 * round(_log_uniform(rng, 1, 64)), **_draw_mask(rng))
        else:
            lo = round(_log_uniform(rng, 64, 16384))
            case.update(nseq=round(_log_uniform(rng, 1, 96)), heads=rng.randint(2, 40), min_len=lo,
                        max_len=128 * math.ceil(lo * rng.uniform(1.0, 4.0) / 128), len_seed=rng.randrange(1 << 20),
                        **_draw_mask(rng))
        w = work(case)
        if w["flops"] < 1e12 and w["bytes"] < 1.5e9 and _cache_bytes(case) < 16e9:
            return case


# ------------------------------------------------------------------------------------ what a case holds


def _lengths(case):
    """Sequence lengths of a packed batch (log-uniform) or of a decode batch (uniform): part of the case."""
    rng = np.random.Generator(np.random.PCG64([synth.BASE_SEED, case["len_seed"]]))
    lo, hi, n = case["min_len"], case["max_len"], case["nseq"]
    if case["kind"] == "train_packed":
        return np.exp(rng.uniform(np.log(lo), np.log(hi + 1), size=n)).astype(np.int64).clip(1, hi).astype(np.int32)
    return rng.integers(lo, hi + 1, size=n).astype(np.int32)


def _cache_bytes(case):
    if case["kind"] != "decode":
        return 0
    return case["nseq"] * case["heads"] * case["max_len"] * case["head_dim"] * 4


def _scale(case):
    return 1.0 / math.sqrt(case["head_dim"])


def _params(case, num_blocks):
    return B.layout_params(case["heads"], num_blocks, case["block_size"], case["local_blocks"], case["stride"])


def _layout(case, tokens):
    S = case["block_size"]
    n = -(-tokens // S)
    return B.s2_layout_build(_params(case, n + (n & 1 if S == 16 else 0)))


def _normal(gen, *shape):
    return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind, H, D = case["kind"], case["heads"], case["head_dim"]
    st = {"case": case, "scale": _scale(case)}
    f32 = lambda *shape: torch.empty(shape, dtype=torch.float32, device="cuda")
    u8 = lambda n: torch.empty(n, dtype=torch.uint8, device="cuda")
    if kind in ("train", "train_dense", "prefill"):
        Bt, N = case["batch"], case["seqlen"]
        st["qkv"] = [_normal(gen, Bt, H, N, D) for _ in range(3)]
        st["o"], st["lse"] = torch.empty_like(st["qkv"][0]), f32(Bt, H, N)
        if kind != "train_dense":
            st["layout"] = _layout(case, N)
        if kind != "prefill":
            st["do"] = _normal(gen, Bt, H, N, D)
            st["grads"] = [torch.empty_like(st["do"]) for _ in range(3)]
            # with the workspace to spare the backward may keep dS; without, it takes the small one
            if kind == "train" and case["keep_ds"]:
                st["ws"] = u8(B.s2_attn_bwd_layout_workspace_bytes(st["layout"], Bt, H, N, D))
            else:
                st["ws"] = u8(B.s2_attn_bwd_workspace_bytes(Bt, H, N, D))
    elif kind == "train_packed":
        lens = _lengths(case)
        total = int(lens.sum())
        st["qkv"] = [_normal(gen, 1, H, total, D) for _ in range(3)]
        st["o"], st["lse"] = torch.empty_like(st["qkv"][0]), f32(H, total)
        st["layout"] = _layout(case, case["max_len"])
        st["cu"] = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).cuda()
        st["do"] = _normal(gen, 1, H, total, D)
        st["grads"] = [torch.empty_like(st["do"]) for _ in range(3)]
        st["ws"] = u8(B.s2_attn_bwd_varlen_workspace_bytes(H, total, D))
    elif kind == "prefill_chunk":
        Bt, rows, N = case["batch"], case["rows"], case["context"] + case["rows"]
        st["q"] = _normal(gen, Bt, H, rows, D)
        st["k"], st["v"] = _normal(gen, Bt, H, N, D), _normal(gen, Bt, H, N, D)
        st["o"], st["lse"] = torch.empty_like(st["q"]), f32(Bt, H, rows)
        st["layout"] = _layout(case, N)
    else:
        n, S, lens = case["nseq"], case["block_size"], _lengths(case)
        st["params"] = _params(case, 1)
        st["q"] = _normal(gen, n, H, D)
        st["o"], st["lse"] = torch.empty_like(st["q"]), f32(n, H)
        st["lens"] = torch.from_numpy(lens).cuda()
        st["ws"] = u8(B.s2_attn_decode_workspace_bytes(n, H, D, case["max_len"]))
        if kind == "decode":
            st["k"], st["v"] = (_normal(gen, n, H, case["max_len"], D) for _ in range(2))
        else:
            # only the blocks a later query can still attend are held, in pages placed at random
            table = np.full((n, H, case["max_len"] // S), -1, dtype=np.int32)
            rows, cols = [], []
            for b in range(n):
                for h in range(H):
                    held = B.s2_kv_resident_blocks(st["params"], h, int(lens[b]))
                    rows.append(np.full(len(held), b * H + h))
                    cols.append(held)
            rows, cols = np.concatenate(rows), np.concatenate(cols)
            order = np.random.Generator(np.random.PCG64(seed)).permutation(len(rows)).astype(np.int32)
            table.reshape(n * H, -1)[rows, cols] = order
            st["table"] = torch.from_numpy(table).cuda()
            st["k"], st["v"] = (_normal(gen, len(rows), S, D) for _ in range(2))
    return st


def run(st):
    kind, scale = st["case"]["kind"], st["scale"]
    if kind in ("train", "prefill"):
        q, k, v = st["qkv"]
        B.s2_attn_fwd(st["layout"], q, k, v, st["o"], st["lse"], scale)
        if kind == "train":
            B.s2_attn_bwd(st["layout"], q, k, v, st["o"], st["lse"], st["do"], *st["grads"], scale, st["ws"])
            return [st["o"], st["lse"]] + st["grads"]
    elif kind == "train_dense":
        q, k, v = st["qkv"]
        B.s2_dense_causal_fwd(q, k, v, st["o"], st["lse"], scale)
        B.s2_dense_causal_bwd(q, k, v, st["o"], st["lse"], st["do"], *st["grads"], scale, st["ws"])
        return [st["o"], st["lse"]] + st["grads"]
    elif kind == "train_packed":
        q, k, v = st["qkv"]
        longest = st["case"]["max_len"]
        B.s2_attn_fwd_varlen(st["layout"], q, k, v, st["o"], st["lse"], st["cu"], longest, scale)
        B.s2_attn_bwd_varlen(st["layout"], q, k, v, st["o"], st["lse"], st["do"], *st["grads"], st["cu"], longest, scale,
                             st["ws"])
        return [st["o"], st["lse"]] + st["grads"]
    elif kind == "prefill_chunk":
        B.s2_attn_fwd_rows(st["layout"], st["q"], st["k"], st["v"], st["o"], st["lse"], st["case"]["context"], scale)
    elif kind == "decode":
        B.s2_attn_decode(st["params"], st["q"], st["k"], st["v"], st["lens"], st["o"], st["lse"], scale, st["ws"],
                         st["case"]["max_len"])
    else:
        B.s2_attn_decode_paged(st["params"], st["q"], st["k"], st["v"], st["table"], st["lens"], st["o"], st["lse"], scale,
                               st["ws"])
    return [st["o"], st["lse"]]


# ------------------------------------------------------------------------------------ work and tolerance


def _row_blocks(case, head, rows):
    """Kept blocks of the block rows `rows` (array) of a head: local window plus stripe columns before it."""
    local = np.minimum(rows + 1, case["local_blocks"])
    s = case["stride"]
    before = rows + 1 - local - head % s  # columns from the head's first stripe to the window
    return local + np.where(before > 0, (before + s - 1) // s, 0)


def _pairs(case, first, tokens):
    """Unmasked (query, key) pairs of the queries first .. tokens-1 of one sequence, summed over heads."""
    S = case["block_size"]
    t = np.arange(first, tokens, dtype=np.int64)
    rows, per_row = np.unique(t // S, return_counts=True)
    diagonal = int((t % S + 1).sum())
    return sum(int(((_row_blocks(case, h, rows) - 1) * S * per_row).sum()) + diagonal for h in range(case["heads"]))


def work(case):
    kind, H, D = case["kind"], case["heads"], case["head_dim"]
    if kind in ("train", "prefill", "train_dense"):
        Bt, N = case["batch"], case["seqlen"]
        pairs = Bt * (H * (N * (N + 1) // 2) if kind == "train_dense" else _pairs(case, 0, N))
        rows = Bt * H * N
        if kind == "prefill":
            return {"bytes": rows * (4 * D * 2 + 4), "flops": 4 * D * pairs}
        return {"bytes": rows * (8 * D * 2 + 4), "flops": 14 * D * pairs}
    lens = None if kind == "prefill_chunk" else _lengths(case)
    if kind == "train_packed":
        pairs = sum(_pairs(case, 0, int(n)) for n in lens)
        return {"bytes": int(lens.sum()) * H * (8 * D * 2 + 4), "flops": 14 * D * pairs}
    if kind == "prefill_chunk":
        Bt, c, r = case["batch"], case["context"], case["rows"]
        S, s = case["block_size"], case["stride"]
        # keys some query of the chunk attends: the window of its first row on, and each head's stripes before
        lo = max(0, c // S - case["local_blocks"] + 1)
        stripes = sum(max(0, -(-(lo - h % s) // s)) for h in range(H))
        keys = stripes * S + H * (c + r - lo * S)
        return {"bytes": Bt * (H * r * (2 * D * 2 + 4) + keys * D * 4), "flops": 4 * D * Bt * _pairs(case, c, c + r)}
    tokens = sum(_pairs(case, int(n) - 1, int(n)) for n in lens)
    return {"bytes": tokens * D * 4 + len(lens) * H * (D * 4 + 4), "flops": 4 * D * tokens}


def tolerance(case):
    # bf16 results of bf16 contractions (the probabilities and dS rounded to bf16 between them) against the
    # same in 64 bits: 2.0e-3 to 2.5e-3 measured for o and the gradients, times four
    return {"rel": 1e-2}
