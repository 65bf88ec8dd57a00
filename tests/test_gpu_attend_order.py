"""Compressed attention of more heads than workgroups start at once: every head is served once, whichever way their order is found."""
import pytest
import torch

from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,B,H,n,kind", [
    (128, 1, 257, 96, "ragged"), (64, 3, 85, 300, "ragged"), (128, 2, 128, 300, "equal"), (128, 1, 300, 130, "long"), (64, 4, 100, 260, "empty"),
    (64, 8, 64, 200, "ragged"), (64, 1, 512, 129, "equal"), (64, 1, 513, 129, "ragged"), (128, 9, 64, 96, "ragged"),
    # up to 256 heads, whose order the kernel's workgroups find
    (128, 1, 200, 300, "long"), (64, 1, 255, 300, "long"), (128, 4, 50, 300, "empty"), (128, 4, 64, 300, "ragged"), (64, 1, 256, 300, "some empty"),
    (128, 1, 130, 600, "cut"), (64, 2, 128, 300, "cut"), (128, 1, 300, 300, "cut")])
def test_every_head_is_served_once(d, B, H, n, kind):
    m = hp.mk()
    gen = torch.Generator(device="cuda").manual_seed(B * H)
    rnd = lambda *shape: torch.randn(shape, generator=gen, device="cuda").bfloat16()
    heads = B * H
    if kind == "equal":
        keep = torch.full((heads,), 70)
    elif kind == "empty":
        keep = torch.zeros(heads, dtype=torch.int64)
    else:
        keep = torch.randint(0, 300, (heads,), generator=torch.Generator().manual_seed(3))
        if kind == "long":
            keep[heads // 2] = 70000  # more 64-key tiles than the order tells apart
            keep[heads - 1] = 69000
        elif kind == "some empty":
            keep[::3] = 0
    cu = torch.cat([torch.zeros(1, dtype=torch.int64), keep.cumsum(0)]).to(torch.int32)
    total = int(cu[-1])
    if kind == "cut":                # rows from there on were not written: they count as not kept
        total = int(cu[heads * 2 // 3]) + 5
    Q, K, V = rnd(B, H, n, d), rnd(B, H, n, d), rnd(B, H, n, d)
    Kc, Vc = rnd(max(total, 1), d), rnd(max(total, 1), d)
    O = torch.full((B, H, n, d), float("nan"), device="cuda").bfloat16()
    desc = m.Desc(B=B, H=H, d=d, dtype=m.MASKKV_BF16, n_resp=n, P_max=int(max(keep.max(), 1)), prompt_len=None if B == 1 else [int(max(keep.max(), 1))] * B)
    m.maskkv_attend(desc, Q, Kc, Vc, cu.cuda(), total, K, V, 0.0, O, None, hp.workspace(max(1, m.maskkv_attend_workspace_bytes(desc, False))))
    for i in range(heads):
        rows = slice(min(int(cu[i]), total), min(int(cu[i + 1]), total))
        k, v = torch.cat([Kc[rows], K[i // H, i % H]]).double(), torch.cat([Vc[rows], V[i // H, i % H]]).double()
        p = torch.softmax(Q[i // H, i % H].double() @ k.T / d ** 0.5, dim=1)
        # probabilities and results are rounded to bf16's 8 significant bits (2^-8 each)
        assert ((O[i // H, i % H].double() - p @ v).abs() <= 2.0 ** -7 * (p @ v.abs())).all(), i
