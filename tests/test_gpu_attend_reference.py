"""Compressed bf16 attention of few query tiles: a row's largest probability loses nothing, also where it comes from a kept row that a
wave meets after response rows with somewhat smaller logits (needs an MI355X).

One kept row holds nearly all weight and the values of all other rows are zero, so the result is that row's value times its share, which
fp32 sums give to 2^-20 or better: correctly rounded to bf16, but for results that close to the middle of two.
"""
import pytest
import torch

from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("n,keep,at", [(256, 40, 0), (256, 40, 39), (300, 33, 5), (512, 70, 64)])
def test_a_dominant_kept_row_is_not_rounded(d, n, keep, at):
    m = hp.mk()
    H = 3
    gen = torch.Generator(device="cuda").manual_seed(n + at)
    e = lambda x: torch.nn.functional.one_hot(torch.zeros_like(x, dtype=torch.int64), d) * x[..., None]
    # logits are products along the first element: queries 4 .. 8, one key in 32 of the response span 0, the others far below
    Q = e(4 + 4 * torch.rand((1, H, n), generator=gen, device="cuda")).bfloat16()
    Kr = torch.full((1, H, n), -64.0, device="cuda")
    Kr[:, :, 7::32] = 0.0
    Kc = torch.full((H, keep), -64.0, device="cuda")
    Kc[:, at] = 5.0 / 8 * d ** 0.5                       # 2.5 .. 5 more than those: 2^3.6 .. 2^7.2
    Kr, Kc = e(Kr).bfloat16(), e(Kc).bfloat16()
    Vr, Vc = torch.zeros((1, H, n, d), device="cuda").bfloat16(), torch.zeros((H, keep, d), device="cuda").bfloat16()
    Vc[:, at] = torch.randn((H, d), generator=gen, device="cuda").bfloat16()
    O = torch.full((1, H, n, d), float("nan"), device="cuda").bfloat16()
    cu = (torch.arange(H + 1, device="cuda") * keep).to(torch.int32)
    desc = m.Desc(B=1, H=H, d=d, dtype=m.MASKKV_BF16, n_resp=n, P_max=keep)
    m.maskkv_attend(desc, Q, Kc.view(-1, d), Vc.view(-1, d), cu, H * keep, Kr, Vr, 0.0, O, None,
                    hp.workspace(max(1, m.maskkv_attend_workspace_bytes(desc, False))))
    k, v = torch.cat([Kc, Kr[0]], 1).double(), torch.cat([Vc, Vr[0]], 1).double()
    want = torch.softmax(Q[0].double() @ k.transpose(1, 2).contiguous() / d ** 0.5, dim=2) @ v
    half_ulp = 2.0 ** (torch.floor(torch.log2(want.abs().clamp(min=1e-30))) - 8)
    assert ((O[0].double() - want).abs() <= half_ulp + 2.0 ** -20 * want.abs()).all()
