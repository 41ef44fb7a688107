"""A packed backward forms the row statistics up to the last row that a sequence owns and of none after it: tensors may hold many
more rows than are in use (a buffer of fixed capacity), and the time of a call goes by the rows in use."""

import pytest
import torch

from paper_2407_17678_amd import binding as B

pytestmark = pytest.mark.gpu


# Row offsets; the sequences as they are cut at 512 rows.  The last two have their last rows beyond as many sequences of that length
# (1024 rows, 3072), and 300 sequences are more than a workgroup has lanes.
CASES = {
    "in_order": ([0, 200, 200, 500, 501], [(0, 200), (200, 500), (500, 501)]),
    "nothing": ([0, 0, 0], []),
    "cut": ([0, 1300, 1365], [(0, 512), (1300, 1365)]),
    "not_ascending": ([0, 70, 2600, 2900, 40, 90, 80], [(0, 70), (70, 582), (2600, 2900), (40, 90)]),
    "many": (list(range(0, 2101, 7)), [(0, 2100)]),
}


@pytest.mark.parametrize("case", sorted(CASES))
@pytest.mark.parametrize("D,S", [(64, 64), (64, 16), (128, 64), (128, 32)])
def test_statistics_of_rows_in_use_only(D, S, case):
    H, rows, max_len, scale = 3, 3000, 512, D ** -0.5
    offsets, bounds = CASES[case]
    cu = torch.tensor(offsets, dtype=torch.int32, device="cuda")
    print("statistics of packed rows", D, S, case, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(D + S)
    q, k, v, g = (torch.randn((1, H, rows, D), device="cuda", generator=gen).bfloat16() for _ in range(4))
    lay = B.s2_layout_build(B.layout_params(H, max_len // S, S, max(1, 64 // S), 5))
    o, lse = torch.zeros_like(q), torch.zeros((H, rows), dtype=torch.float32, device="cuda")
    grads = [torch.zeros_like(q) for _ in range(3)]
    size = B.s2_attn_bwd_varlen_workspace_bytes(H, rows, D)
    ws = torch.full((size // 4,), -1, dtype=torch.int32, device="cuda")
    B.s2_attn_fwd_varlen(lay, q, k, v, o, lse, cu, max_len, scale)
    B.s2_attn_bwd_varlen(lay, q, k, v, o, lse, g, *grads, cu, max_len, scale, ws)
    torch.cuda.synchronize()
    owned = torch.zeros(rows, dtype=torch.bool, device="cuda")
    for lo, hi in bounds:
        owned[lo:hi] = True
    end = max([hi for _, hi in bounds], default=0)
    delta = (g.double() * o.double()).sum(-1)[0]
    halves = ws.view(2, -1)  # two arrays of [heads, rows], each at the start of a half
    for half in halves:
        written = half[:H * rows].view(H, rows) != -1
        assert written[:, owned].all()
        assert not written[:, end:].any()
        assert (half[H * rows:] == -1).all()
    got = [half[:H * rows].view(H, rows).view(torch.float32)[:, owned].double() for half in halves]
    # D products of bf16 values in float32, and one product
    assert ((got[0] + delta[:, owned]).abs() <= D * 2.0 ** -24 * (g.double() * o.double()).abs().sum(-1)[0][:, owned]).all()
    assert ((got[1] + lse[:, owned].double() / scale).abs() <= 2.0 ** -22 * (lse[:, owned].double() / scale).abs()).all()
