"""fp32 scoring of short prompts with many rows, whose column sums and masses are added up over 2 ... 128 parts: around the sixteen parts
that are asked for at once and the sixty-four masses that a wave holds (needs an MI355X).

Reference: float64 on the same inputs.  fp32 logits of up to 2^4 are off by 2^-20 or less, an exponential and a sum of them by as
much relative to themselves; a mass is a sum of shares, each off by as much.
"""
import pytest
import torch

from tests import helpers as hp

pytestmark = pytest.mark.gpu

RTOL = 2.0 ** -19


@pytest.mark.parametrize("n,g", [(8, 4), (12, 4), (16, 4), (20, 4), (24, 4), (64, 4), (68, 4), (69, 4), (132, 4), (136, 4), (137, 4), (63, 16),
                                 (64, 16), (65, 16), (130, 16), (130, 32)])
def test_against_float64(n, g):
    m = hp.mk()
    gen = torch.Generator(device="cuda").manual_seed(n + g)
    H, d, Ps, P_max = 2, 64, (60, 41), 60
    Q = torch.randn((2, H * g, n, d), generator=gen, device="cuda")
    K = torch.randn((2, H, P_max + n, d), generator=gen, device="cuda")
    desc = m.Desc(B=2, H=H, d=d, dtype=m.MASKKV_F32, n_resp=n, P_max=P_max, prompt_len=list(Ps), q_per_kv=g)
    scores, mass = torch.full((2 * H, P_max), float("nan"), device="cuda"), torch.full((2 * H,), float("nan"), device="cuda")
    m.maskkv_score(desc, Q, K, 0.0, scores, P_max, mass, hp.workspace(m.maskkv_score_workspace_bytes(desc)))
    for b, P in enumerate(Ps):
        for h in range(H):
            q = Q[b, h * g:(h + 1) * g].reshape(g * n, d).double()
            want = torch.softmax(q @ K[b, h, :P + n].double().T / d ** 0.5, dim=1)[:, :P].sum(0)
            assert torch.allclose(scores[b * H + h, :P].double(), want, rtol=RTOL, atol=0)
            assert torch.isnan(scores[b * H + h, P:]).all()
            assert abs(float(mass[b * H + h]) - float(want.sum())) <= RTOL * float(want.sum())
