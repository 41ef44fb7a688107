"""CPU tests of the extension that makes the compute calls (csrc/marshal.cpp): what arrives at a C entry point for given tensors, put
there by callbacks in the entry points' place, and that what the binding refuses is refused."""

import ctypes as C

import pytest
import torch

from paper_2407_17678_amd import binding as B

P, I, F, Z = C.c_void_p, C.c_int32, C.c_float, C.c_size_t
T, D, G, LP = C.POINTER(B.Tensors), C.POINTER(B.DecodeArgs), C.POINTER(B.PagedDecodeArgs), C.POINTER(B.LayoutParams)
SIGNATURES = {
    "s2_attn_fwd": (P, T, F, P), "s2_attn_fwd_rows": (P, T, I, I, F, P), "s2_attn_fwd_varlen": (P, T, P, I, I, F, P),
    "s2_attn_bwd_stages": (P, T, F, P, Z, I, P), "s2_attn_bwd_varlen": (P, T, P, I, I, F, P, Z, P), "s2_dense_causal_fwd": (T, F, P),
    "s2_dense_causal_bwd": (T, F, P, Z, P), "s2_attn_decode": (LP, D, F, P, Z, P), "s2_attn_decode_static": (LP, D, F, P),
    "s2_attn_decode_layout": (P, D, F, P, Z, P), "s2_attn_decode_paged": (LP, G, F, P, Z, P), "s2_attn_decode_paged_layout": (P, G, F, P, Z, P),
}


class Stream:
    cuda_stream = 0x5000


class Handle:
    handle = C.c_void_p(0x7000)


@pytest.fixture()
def seen():
    """Binds callbacks that keep their arguments (structures as dicts); gives the list they are kept in."""
    calls, got = B._marshal(), []

    def callback(name, types):
        def f(*args):
            flat = []
            for a in args:
                if hasattr(a, "contents"):
                    a = {n: getattr(a.contents, n) for n, *_ in a.contents._fields_}
                flat.append(a)
            got.append((name, flat))
            return 0
        return C.CFUNCTYPE(C.c_int, *types)(f)

    kept = [callback(n, SIGNATURES[n]) for n in B._MARSHALLED]
    calls.bind(*(C.cast(f, C.c_void_p).value for f in kept))
    yield got
    calls.bind(*(C.cast(getattr(B.lib(), n), C.c_void_p).value for n in B._MARSHALLED))


def _bf16(*shape):
    return torch.zeros(shape, dtype=torch.bfloat16)


def _training(pad=0, rows=24):
    """Nine tensors, q-like ones [batch, token, head, feature] in memory, k-like ones with longer rows; lse."""
    q, o, g, dq = (_bf16(2, rows, 3, 64).permute(0, 2, 1, 3) for _ in range(4))
    k, v, dk, dv = (_bf16(2, 3, rows, 64 + pad)[..., :64] for _ in range(4))
    return q, k, v, o, torch.zeros(2, 3, rows), g, dq, dk, dv


def _check_tensors(s, t, backward, seqlen=24):
    for name, x in zip(("q", "k", "v", "o", "lse") + (("d_o", "dq", "dk", "dv") if backward else ()), t):
        assert s[name] == x.data_ptr(), name
    if not backward:
        assert not any(s[n] for n in ("d_o", "dq", "dk", "dv"))
    assert (s["batch"], s["heads"], s["seqlen"], s["head_dim"]) == (2, 3, seqlen, 64)
    assert (s["q_stride_b"], s["q_stride_h"], s["q_stride_t"]) == t[0].stride()[:3]
    assert (s["kv_stride_b"], s["kv_stride_h"], s["kv_stride_t"]) == t[1].stride()[:3]


@pytest.mark.parametrize("pad", [0, 8])
def test_training_calls(seen, pad):
    t, ws, lay, st = _training(pad), torch.zeros(100, dtype=torch.float32), Handle(), Stream()
    B.s2_attn_fwd(lay, *t[:5], 0.5, stream=st)
    B.s2_attn_bwd(lay, *t, 0.5, ws, stream=st)
    B.s2_attn_bwd_stages(lay, *t, 0.5, ws, 5, stream=st)
    B.s2_dense_causal_fwd(*t[:5], 0.5, stream=st)
    B.s2_dense_causal_bwd(*t, 0.5, ws, stream=st)
    fwd, bwd, stages, dfwd, dbwd = (a for _, a in seen)
    assert [n for n, _ in seen] == ["s2_attn_fwd", "s2_attn_bwd_stages", "s2_attn_bwd_stages", "s2_dense_causal_fwd", "s2_dense_causal_bwd"]
    for a, back in ((fwd[1], False), (bwd[1], True), (stages[1], True), (dfwd[0], False), (dbwd[0], True)):
        _check_tensors(a, t, back)
    assert fwd[0] == bwd[0] == stages[0] == 0x7000
    assert fwd[2:] == [0.5, 0x5000] and dfwd[1:] == [0.5, 0x5000]
    assert bwd[2:] == [0.5, ws.data_ptr(), 400, 7, 0x5000] and stages[2:] == [0.5, ws.data_ptr(), 400, 5, 0x5000]
    assert dbwd[1:] == [0.5, ws.data_ptr(), 400, 0x5000]


def test_rows_and_packed_calls(seen):
    t, lay, st = _training(rows=24), Handle(), Stream()
    longer = _training(rows=40)
    B.s2_attn_fwd_rows(lay, t[0], longer[1], longer[2], t[3], t[4], 16, 0.5, stream=st)
    a = seen[0][1]
    assert (a[1]["seqlen"], a[2], a[3], a[4], a[5]) == (40, 16, 24, 0.5, 0x5000)
    assert a[1]["k"] == longer[1].data_ptr() and a[1]["kv_stride_b"] == longer[1].stride(0)
    one = [x[:1] for x in t[:4]] + [t[4][0]] + [x[:1] for x in t[5:]]
    cu, ws = torch.tensor([0, 3, 24], dtype=torch.int32), torch.zeros(64, dtype=torch.uint8)
    B.s2_attn_fwd_varlen(lay, *one[:5], cu, 21, 0.25, stream=st)
    B.s2_attn_bwd_varlen(lay, *one, cu, 21, 0.25, ws, stream=st)
    f, b = seen[1][1], seen[2][1]
    assert f[2:] == [cu.data_ptr(), 2, 21, 0.25, 0x5000] and b[2:] == [cu.data_ptr(), 2, 21, 0.25, ws.data_ptr(), 64, 0x5000]
    for bad in (cu[:1], cu[::2]):  # one offset; not contiguous
        with pytest.raises(AssertionError):
            B.s2_attn_fwd_varlen(lay, *one[:5], bad, 21, 0.25, stream=st)
    with pytest.raises(AssertionError):
        B.s2_attn_bwd_varlen(lay, *t, cu, 21, 0.25, ws, stream=st)  # two batch elements
    assert len(seen) == 3


@pytest.mark.parametrize("lse", [False, True])
def test_decode_calls(seen, lse):
    q, o, k, v = _bf16(2, 3, 64), _bf16(2, 3, 64), _bf16(2, 3, 40, 72)[..., :64], _bf16(2, 3, 40, 72)[..., :64]
    lens, ws, par, lay, st = torch.ones(2, dtype=torch.int32), torch.zeros(64, dtype=torch.uint8), B.layout_params(3, 1, 16, 2, 3), Handle(), Stream()
    l = torch.zeros(2, 3) if lse else None
    B.s2_attn_decode(par, q, k, v, lens, o, l, 0.5, ws, 40, num_splits=3, stream=st)
    B.s2_attn_decode_static(par, q, k, v, lens, o, l, 0.5, 40, stream=st)
    B.s2_attn_decode_layout(lay, q, k, v, lens, o, l, 0.5, ws, 40, stream=st)
    want = dict(q=q.data_ptr(), k_cache=k.data_ptr(), v_cache=v.data_ptr(), seq_lens=lens.data_ptr(), o=o.data_ptr(),
                lse=l.data_ptr() if lse else None, nseq=2, heads=3, head_dim=64, max_len=40, num_splits=3, kv_stride_seq=3 * 40 * 72,
                kv_stride_head=40 * 72, kv_stride_tok=72)
    (_, a), (_, s), (_, c) = seen
    assert a[0]["num_heads"] == s[0]["num_heads"] == 3 and c[0] == 0x7000
    assert a[1] == want and s[1] == c[1] == dict(want, num_splits=0)
    assert a[2:] == c[2:] == [0.5, ws.data_ptr(), 64, 0x5000] and s[2:] == [0.5, 0x5000]
    kp, vp = _bf16(5, 16, 72)[..., :64], _bf16(5, 16, 72)[..., :64]
    table, miss = torch.zeros(2, 3, 7, dtype=torch.int32), torch.zeros(1, dtype=torch.int32)
    B.s2_attn_decode_paged(par, q, kp, vp, table, lens, o, l, 0.5, ws, missing=miss, stream=st)
    B.s2_attn_decode_paged_layout(lay, q, kp, vp, table, lens, o, l, 0.5, ws, num_splits=2, stream=st)
    (_, a), (_, c) = seen[3:]
    want = dict(q=q.data_ptr(), k_pages=kp.data_ptr(), v_pages=vp.data_ptr(), block_table=table.data_ptr(), seq_lens=lens.data_ptr(), o=o.data_ptr(),
                lse=l.data_ptr() if lse else None, missing=miss.data_ptr(), nseq=2, heads=3, head_dim=64, max_blocks=7, num_pages=5, num_splits=0,
                page_stride=16 * 72, tok_stride=72)
    assert a[1] == want and c[1] == dict(want, missing=None, num_splits=2) and c[0] == 0x7000
    assert a[2:] == c[2:] == [0.5, ws.data_ptr(), 64, 0x5000]


def test_what_is_refused(seen):
    t, lay, st = list(_training()), Handle(), Stream()

    def refused(error, i, x, n=5):
        bad = list(t)
        bad[i] = x
        with pytest.raises(error):
            if n == 5:
                B.s2_attn_fwd(lay, *bad[:5], 0.5, stream=st)
            else:
                B.s2_attn_bwd(lay, *bad, 0.5, torch.zeros(4), stream=st)

    refused(AssertionError, 1, t[0])                                         # k and v of different strides
    refused(AssertionError, 3, t[1])                                         # q and o
    refused(AssertionError, 4, torch.zeros(2, 3, 48)[..., ::2])              # lse not contiguous
    refused(AssertionError, 0, _bf16(2, 3, 24, 128)[..., ::2])               # features not side by side
    refused(ValueError, 0, _bf16(3, 24, 64))                                 # three sizes
    refused(AttributeError, 2, None)
    for i, x in ((5, t[1]), (6, t[1]), (7, t[0]), (8, t[0])):
        refused(AssertionError, i, x, 9)
    with pytest.raises(TypeError):
        B.s2_attn_fwd(lay, *t[:5], "1", stream=st)
    with pytest.raises(TypeError):
        B.s2_attn_bwd_stages(lay, *t, 0.5, torch.zeros(4), 7.5, stream=st)
    with pytest.raises(AttributeError):
        B.s2_attn_bwd(lay, *t, 0.5, None, stream=st)
    q, k, lens, ws = _bf16(2, 3, 64), _bf16(2, 3, 40, 64), torch.ones(2, dtype=torch.int32), torch.zeros(64, dtype=torch.uint8)
    par = B.layout_params(3, 1, 16, 2, 3)
    for bad in (B.DecodeArgs(), 5, None):
        with pytest.raises((TypeError, C.ArgumentError)):
            B.s2_attn_decode(bad, q, k, k, lens, q, None, 0.5, ws, 40, stream=st)
    for a, b, c, o in ((q.transpose(0, 1), k, k, q), (q, k, k, q.transpose(0, 1)), (q, k, _bf16(2, 3, 41, 64), q), (q, k.transpose(2, 3), k.transpose(2, 3), q)):
        with pytest.raises(AssertionError):
            B.s2_attn_decode(par, a, b, c, lens, o, None, 0.5, ws, 40, stream=st)
    kp = _bf16(5, 16, 64)
    for table in (torch.zeros(3, 2, 7), torch.zeros(2), torch.zeros(2, 3, 14)[..., ::2]):
        with pytest.raises(AssertionError):
            B.s2_attn_decode_paged(par, q, kp, kp, table, lens, q, None, 0.5, ws, stream=st)
    assert not seen


def test_a_destroyed_layout_is_a_null_handle():
    t = _training()
    gone = Handle()
    gone.handle = None
    with pytest.raises(B.S2Error) as e:
        B.s2_attn_fwd(gone, *t[:5], 0.5, stream=Stream())
    assert e.value.status == -1


def test_an_extension_of_other_sources_is_refused(monkeypatch):
    # (its functions call by position)
    B._marshal()
    monkeypatch.setattr(B, "_calls", None)
    monkeypatch.setattr(B, "_MARSHALLED", B._MARSHALLED[::-1])
    with pytest.raises(ImportError):
        B._marshal()
