"""What a mask row does not keep does not reach its results, whatever it holds: blocks of K and V (for dK and dV: of
q and dO) are overwritten with NaN and infinities, and the rows that keep none of them come out bit for bit as with
the clean tensors.  With 16-token blocks a wavefront's 32 rows are two mask rows, which share this: the rows that
count are those of pairs of which neither keeps a poisoned block (dK and dV: see _clean_columns)."""

import numpy as np
import pytest
import torch

from oracle import s2_oracle as orc
from paper_2407_17678_amd import binding as B

pytestmark = pytest.mark.gpu

NEG, POS, NAN = -float("inf"), float("inf"), float("nan")


def _mask(rng, H, Bk, density):
    M = np.tril(rng.random((H, Bk, Bk)) < density)
    M[:, np.arange(Bk), np.arange(Bk)] = True
    return M


def _setup(D, S, H, Bk, density, seed):
    rng = np.random.default_rng(seed)
    M = _mask(rng, H, Bk, density)
    row_ptr, col_idx, _, _ = orc.compressed_layout(M)
    lay = B.s2_layout_from_csr(H, Bk, S, row_ptr, col_idx)
    bad = rng.choice(np.arange(1, Bk - 1), size=max(1, Bk // 8), replace=False)
    return M, lay, bad, D ** -0.5


def _poison(x, blocks, S, values):
    y = x.clone()
    for n, j in enumerate(blocks):
        y[..., j * S:(j + 1) * S, :] = values[n % len(values)]
    return y


def _clean_rows(M, bad, S):
    """[H, rows]: rows of wavefronts (32 rows) of whose mask rows none keeps a poisoned block."""
    keeps = M[:, :, bad].any(2)
    per_row = np.repeat(keeps, S, axis=1)
    H, N = per_row.shape
    pad = np.pad(per_row, ((0, 0), (0, -N % 32)))
    return torch.from_numpy(~np.repeat(pad.reshape(H, -1, 32).any(2), 32, axis=1)[:, :N])


def _rand(*shape):
    return torch.randn(*shape, device="cuda", generator=_gen).bfloat16()


_gen = None


@pytest.fixture(autouse=True)
def _seeded():
    global _gen
    _gen = torch.Generator(device="cuda")
    _gen.manual_seed(5)


FORMS = [(64, 16), (64, 32), (64, 64), (64, 128), (128, 16), (128, 32), (128, 64), (128, 128)]


@pytest.mark.parametrize("D,S", FORMS)
@pytest.mark.parametrize("density", [0.15, 0.5])
def test_forward(D, S, density):
    H, Bk = 3, 12 if S == 128 else 1152 // S + (S == 64)
    M, lay, bad, scale = _setup(D, S, H, Bk, density, 10 * D + S)
    N = Bk * S
    q, k, v = _rand(1, H, N, D), _rand(1, H, N, D), _rand(1, H, N, D)
    clean = _clean_rows(M, bad, S)
    assert clean.any()

    def fwd(k, v):
        o, lse = torch.empty_like(q), torch.empty((1, H, N), dtype=torch.float32, device="cuda")
        B.s2_attn_fwd(lay, q, k, v, o, lse, scale)
        return o[0].cpu(), lse[0].cpu()

    o, lse = fwd(k, v)
    for values in ((NAN,), (POS, NEG)):
        o1, lse1 = fwd(_poison(k, bad, S, values), _poison(v, bad, S, values))
        assert torch.equal(o1[clean], o[clean]) and torch.equal(lse1[clean], lse[clean])


@pytest.mark.parametrize("D,S", FORMS)
def test_forward_packed(D, S):
    H, Bk = 2, 768 // S
    M, lay, bad, scale = _setup(D, S, H, Bk, 0.3, 11 * D + S)
    lens = [768, 700, 39, 333]
    total = sum(lens)
    cu = torch.tensor([0] + list(np.cumsum(lens)), dtype=torch.int32, device="cuda")
    q, k, v = _rand(1, H, total, D), _rand(1, H, total, D), _rand(1, H, total, D)
    rows = _clean_rows(M, bad, S)
    clean = torch.cat([rows[:, :n] for n in lens], 1)
    where = torch.cat([torch.arange(n) for n in lens])
    hit = torch.zeros(total, dtype=torch.bool)
    for j in bad:
        hit |= where // S == int(j)

    def fwd(k, v):
        o, lse = torch.empty_like(q), torch.empty((H, total), dtype=torch.float32, device="cuda")
        B.s2_attn_fwd_varlen(lay, q, k, v, o, lse, cu, 768, scale)
        return o[0].cpu(), lse.cpu()

    o, lse = fwd(k, v)
    for value in (NAN, POS):
        k1, v1 = k.clone(), v.clone()
        k1[:, :, hit.cuda()] = value
        v1[:, :, hit.cuda()] = value
        o1, lse1 = fwd(k1, v1)
        assert torch.equal(o1[clean], o[clean]) and torch.equal(lse1[clean], lse[clean])


def _forward(lay, q, k, v, scale):
    o, lse = torch.empty_like(q), torch.empty(q.shape[:3], dtype=torch.float32, device="cuda")
    B.s2_attn_fwd(lay, q, k, v, o, lse, scale)
    return o, lse


@pytest.mark.parametrize("D,S", FORMS)
@pytest.mark.parametrize("density", [0.15, 0.5])
def test_dq(D, S, density):
    H, Bk = 3, 12 if S == 128 else 1152 // S + (S == 64)
    M, lay, bad, scale = _setup(D, S, H, Bk, density, 12 * D + S)
    N = Bk * S
    q, k, v, g = (_rand(1, H, N, D) for _ in range(4))
    clean = _clean_rows(M, bad, S)
    o, lse = _forward(lay, q, k, v, scale)
    ws = torch.empty(B.s2_attn_bwd_workspace_bytes(1, H, N, D), dtype=torch.uint8, device="cuda")

    def dq(k, v):
        grads = [torch.empty_like(q) for _ in range(3)]
        B.s2_attn_bwd(lay, q, k, v, o, lse, g, *grads, scale, ws)
        return grads[0][0].cpu()

    want = dq(k, v)
    for values in ((NAN,), (POS, NEG)):
        assert torch.equal(dq(_poison(k, bad, S, values), _poison(v, bad, S, values))[clean], want[clean])


@pytest.mark.parametrize("D,S", FORMS)
def test_dq_packed(D, S):
    H, Bk = 2, 768 // S
    M, lay, bad, scale = _setup(D, S, H, Bk, 0.3, 13 * D + S)
    lens = [768, 700, 39, 333]
    total = sum(lens)
    cu = torch.tensor([0] + list(np.cumsum(lens)), dtype=torch.int32, device="cuda")
    q, k, v, g = (_rand(1, H, total, D) for _ in range(4))
    rows = _clean_rows(M, bad, S)
    clean = torch.cat([rows[:, :n] for n in lens], 1)
    where = torch.cat([torch.arange(n) for n in lens])
    hit = torch.isin(where // S, torch.from_numpy(np.asarray(bad))).cuda()
    o, lse = torch.empty_like(q), torch.empty((H, total), dtype=torch.float32, device="cuda")
    B.s2_attn_fwd_varlen(lay, q, k, v, o, lse, cu, 768, scale)
    ws = torch.empty(B.s2_attn_bwd_varlen_workspace_bytes(H, total, D), dtype=torch.uint8, device="cuda")

    def dq(k, v):
        grads = [torch.empty_like(q) for _ in range(3)]
        B.s2_attn_bwd_varlen(lay, q, k, v, o, lse, g, *grads, cu, 768, scale, ws)
        return grads[0][0].cpu()

    want = dq(k, v)
    for value in (NAN, POS):
        k1, v1 = k.clone(), v.clone()
        k1[:, :, hit] = value
        v1[:, :, hit] = value
        assert torch.equal(dq(k1, v1)[clean], want[clean])


def _clean_columns(lay, M, bad, S):
    """[H, keys]: keys that no poisoned query block attends.  With 16-token blocks dK and dV are formed for two columns
    of a key tile and from two blocks of its list at a time, which share this."""
    H, Bk, _ = M.shape
    hit = M[:, bad, :].any(1)
    if S == 16:
        kv = B.s2_layout_get_tiles(lay, B.TILES_DKDV)
        T = kv["tiles_per_head"]
        for h in range(H):
            for t in range(T):
                ent = np.asarray(kv["ent"][kv["ptr"][h * T + t]:kv["ptr"][h * T + t + 1]]).view(np.uint32)
                mem = np.asarray(kv["members"][(h * T + t) * 8:(h * T + t + 1) * 8])
                for i in range(0, len(ent), 2):
                    half = ent[i:i + 2]
                    if not np.isin(half >> 16, bad).any():
                        continue
                    bits = int(np.bitwise_or.reduce(half)) & 0xFF
                    for w in range(4):
                        if (bits >> (2 * w)) & 3:
                            hit[h, [m for m in mem[2 * w:2 * w + 2] if m >= 0]] = True
    return torch.from_numpy(~np.repeat(hit, S, axis=1))


@pytest.mark.parametrize("D,S,keep_ds", [f + (False,) for f in FORMS] + [(128, 64, True), (128, 128, True)])
@pytest.mark.parametrize("density", [0.1, 0.5])
def test_dk_dv(D, S, keep_ds, density):
    H, Bk = 3, 12 if S == 128 else 1152 // S
    M, lay, bad, scale = _setup(D, S, H, Bk, density, 14 * D + S)
    N = Bk * S
    q, k, v, g = (_rand(1, H, N, D) for _ in range(4))
    clean = _clean_columns(lay, M, bad, S)
    assert clean.any()
    o, lse = _forward(lay, q, k, v, scale)
    ws = torch.empty(B.s2_attn_bwd_layout_workspace_bytes(lay, 1, H, N, D) if keep_ds else B.s2_attn_bwd_workspace_bytes(1, H, N, D),
                     dtype=torch.uint8, device="cuda")

    def bwd(q, g):
        grads = [torch.empty_like(q) for _ in range(3)]
        B.s2_attn_bwd(lay, q, k, v, o, lse, g, *grads, scale, ws)
        return grads[1][0].cpu(), grads[2][0].cpu()

    want = bwd(q, g)
    for values in ((NAN,), (POS, NEG)):
        got = bwd(_poison(q, bad, S, values), _poison(g, bad, S, values))
        for a, b in zip(got, want):
            assert torch.equal(a[clean], b[clean])


@pytest.mark.parametrize("D,S", FORMS)
def test_dk_dv_packed(D, S):
    H, Bk = 2, 768 // S
    M, lay, bad, scale = _setup(D, S, H, Bk, 0.15, 15 * D + S)
    lens = [768, 700, 39, 333]
    total = sum(lens)
    cu = torch.tensor([0] + list(np.cumsum(lens)), dtype=torch.int32, device="cuda")
    q, k, v, g = (_rand(1, H, total, D) for _ in range(4))
    keys = _clean_columns(lay, M, bad, S)
    clean = torch.cat([keys[:, :n] for n in lens], 1)
    assert clean.any()
    where = torch.cat([torch.arange(n) for n in lens])
    hit = torch.isin(where // S, torch.from_numpy(np.asarray(bad))).cuda()
    o, lse = torch.empty_like(q), torch.empty((H, total), dtype=torch.float32, device="cuda")
    B.s2_attn_fwd_varlen(lay, q, k, v, o, lse, cu, 768, scale)
    ws = torch.empty(B.s2_attn_bwd_varlen_workspace_bytes(H, total, D), dtype=torch.uint8, device="cuda")

    def bwd(q, g):
        grads = [torch.empty_like(q) for _ in range(3)]
        B.s2_attn_bwd_varlen(lay, q, k, v, o, lse, g, *grads, cu, 768, scale, ws)
        return grads[1][0].cpu(), grads[2][0].cpu()

    want = bwd(q, g)
    for value in (NAN, POS):
        q1, g1 = q.clone(), g.clone()
        q1[:, :, hit] = value
        g1[:, :, hit] = value
        for a, b in zip(bwd(q1, g1), want):
            assert torch.equal(a[clean], b[clean])
