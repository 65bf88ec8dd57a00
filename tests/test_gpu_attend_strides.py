"""The tiled bf16 attention's transfers go on from tile to tile by the segment's own stride: response rows whose K and V have different
strides and starts give what packed ones give, bit for bit, wherever the packed cache ends (needs an MI355X)."""
import pytest
import torch

from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [264, 520])  # 128 and 256 queries a workgroup
@pytest.mark.parametrize("lo", [0, 57])
def test_strided_response_rows(d, n, lo):
    m = hp.mk()
    B, H = 2, 48
    gen = torch.Generator(device="cuda").manual_seed(d + n + lo)
    rnd = lambda *shape: torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
    budgets = torch.tensor([lo + i * 5 % 79 for i in range(B * H)])  # ends at every place of the rows that a wave moves
    cu = torch.cat([torch.zeros(1, dtype=torch.int64), budgets.cumsum(0)]).to(torch.int32).cuda()
    cap = int(budgets.sum())
    Q, Kc, Vc = rnd(B, H, n, d), rnd(cap, d), rnd(cap, d)
    K, V = rnd(B, 3 + n, H, d), rnd(B, 2 * H, 8 + n, 3 * d)  # tokens before heads; rows and heads apart
    views = m.tensor_view(K.transpose(1, 2), seq_start=[3, 1]), m.tensor_view(V[:, ::2, :, d:2 * d], seq_start=[8, 0])
    packed = [torch.stack([K.transpose(1, 2)[b, :, s:s + n] for b, s in enumerate((3, 1))]).contiguous(),
              torch.stack([V[b, ::2, s:s + n, d:2 * d] for b, s in enumerate((8, 0))]).contiguous()]
    desc = m.Desc(B=B, H=H, d=d, dtype=m.MASKKV_BF16, n_resp=n, P_max=256, prompt_len=[256, 256])
    out = []
    for Kr, Vr in (packed, views):
        O = torch.full((B, H, n, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        m.maskkv_attend(desc, Q, Kc, Vc, cu, cap, Kr, Vr, 0.0, O, None, hp.workspace(m.maskkv_attend_workspace_bytes(desc, False)))
        out.append(O)
    assert torch.isfinite(out[0].float()).all() and torch.equal(out[0], out[1])
