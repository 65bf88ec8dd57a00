"""The gather on either side of the number of heads whose ends a wave holds: rows of one wave that belong to many heads, and to none."""
import pytest
import torch

from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H", [(1, 1), (1, 63), (2, 32), (3, 43), (1, 256), (8, 32), (1, 257), (5, 60)])
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 128)])
@pytest.mark.parametrize("spare", [0, 100, -3])
def test_rows_of_every_head(B, H, dtype, d, spare):
    m = hp.mk()
    dt, code = (torch.bfloat16, m.MASKKV_BF16) if dtype == "bf16" else (torch.float32, m.MASKKV_F32)
    heads, P_max = B * H, 40
    P = [P_max] if B == 1 else [P_max - 5 * b for b in range(B)]
    keep = [(0, 0, 1, 0, 3, 0, 0, 0, 7, 19)[(i * 7) % 10] for i in range(heads)]
    if sum(keep) == 0:
        keep[0] = 5
    cu = [sum(keep[:i]) for i in range(heads + 1)]
    total, cap = cu[-1], cu[-1] + spare
    gen = torch.Generator(device="cuda").manual_seed(heads)
    K, V = (torch.randn((B, H, P_max + 2, d), generator=gen, device="cuda").to(dt) for _ in range(2))
    idx = torch.randint(0, min(P), (total,), generator=torch.Generator().manual_seed(1), dtype=torch.int32)
    idx[0], idx[-1] = -4, P_max + 9  # (clamped to the prompt)
    Kc, Vc = (torch.full((max(total, cap), d), 7.0, device="cuda").to(dt) for _ in range(2))
    desc = m.Desc(B=B, H=H, d=d, dtype=code, n_resp=2, P_max=P_max, prompt_len=None if B == 1 else P)
    m.maskkv_compact(desc, K, V, idx.cuda(), torch.tensor(cu, dtype=torch.int32, device="cuda"), cap, Kc, Vc)
    head = torch.repeat_interleave(torch.arange(heads), torch.tensor(keep))
    row = torch.minimum(idx.clamp(min=0).long(), torch.tensor(P)[head // H] - 1)
    rows = min(total, cap)
    for src, packed in ((K, Kc), (V, Vc)):
        want = src.cpu()[head // H, head % H, row]
        assert torch.equal(packed[:rows].cpu(), want[:rows]) and (packed[rows:] == 7).all()
