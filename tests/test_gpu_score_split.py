"""Scoring of short fp32 prompts whose rows and keys are both dealt out over workgroups: edges of the parts of 64, 128 and 256 keys, of the
groups of 16 rows and of the tiles that a workgroup sums up, several rounds of groups, more than 16 parts, empty prompts, grouped queries
and strides (needs an MI355X).

Reference: float64 on the same inputs.  fp32 logits of up to 2^4 are off by 2^-20 or less, an exponential and a sum of them by as
much relative to themselves; a mass is a sum of shares, each off by as much.
"""
import pytest
import torch

from tests import helpers as hp

pytestmark = pytest.mark.gpu

RTOL = 2.0 ** -19


@pytest.mark.parametrize("d,n,H,g,Ps,split", [
    # parts of 64 keys, one group of rows a workgroup
    (64, 17, 3, 1, (366, 367, 368, 0), (1, 64, 7)), (128, 17, 3, 1, (111, 112, 175), (1, 64, 3)), (64, 64, 4, 1, (512,), (1, 64, 9)),
    (128, 36, 4, 1, (544,), (1, 64, 10)), (64, 33, 2, 1, (991,), (1, 64, 16)),
    # of 128
    (64, 33, 2, 1, (992,), (1, 128, 9)), (128, 32, 4, 1, (2500, 100), (1, 128, 20)), (128, 31, 1, 4, (3041,), (1, 128, 24)),
    (64, 130, 2, 1, (1150,), (1, 128, 10)), (64, 47, 16, 1, (1233, 0), (1, 128, 10)), (128, 64, 8, 1, (1984, 0), (1, 128, 16)),
    # of 256, two groups of rows: whole parts and a key more, an odd group, grouped queries, short and empty prompts beside the long one
    (64, 100, 8, 1, (1180,), (2, 256, 5)), (64, 128, 4, 1, (2500,), (2, 256, 11)), (64, 40, 4, 7, (2499,), (2, 256, 10)),
    (64, 130, 4, 1, (1918, 0), (2, 256, 8)), (64, 130, 4, 1, (1917, 200), (2, 256, 8)), (64, 64, 8, 1, (1985, 0), (2, 256, 9)),
    (128, 128, 4, 1, (2500,), (2, 256, 11)), (128, 64, 8, 1, (2000,), (2, 256, 9)), (128, 130, 4, 1, (1918, 0), (2, 256, 8)),
    (128, 130, 4, 1, (1919, 0), (2, 256, 9)), (128, 130, 6, 1, (1917, 3, 0), (2, 256, 8)), (128, 77, 3, 4, (1740, 0, 300), (2, 256, 8))])
def test_against_float64(d, n, H, g, Ps, split):
    m = hp.mk()
    gen = torch.Generator(device="cuda").manual_seed(d + n + H)
    B, P_max = len(Ps), max(Ps)
    Q = torch.randn((B, H * g, n, d), generator=gen, device="cuda")
    K = torch.randn((B, P_max + n, H, d), generator=gen, device="cuda").transpose(1, 2)   # (rows of a head are H * d apart)
    desc = m.Desc(B=B, H=H, d=d, dtype=m.MASKKV_F32, n_resp=n, P_max=P_max, prompt_len=None if B == 1 else list(Ps), q_per_kv=0 if g == 1 else g)
    from paper_2510_09309_amd import bench_binding as bb
    assert bb.maskkv_bench_score_split(desc) == split      # (a change of the cost model could take a case past what it is here for)
    scores, mass = torch.full((B * H, P_max + 3), float("nan"), device="cuda"), torch.full((B * H,), float("nan"), device="cuda")
    ws = hp.workspace(m.maskkv_score_workspace_bytes(desc))
    m.maskkv_score(desc, Q, K, 0.0, scores, P_max + 3, mass, ws)
    for b, P in enumerate(Ps):
        for h in range(H):
            q = Q[b, h * g:(h + 1) * g].reshape(g * n, d).double()
            want = torch.softmax(q @ K[b, h, :P + n].double().T / d ** 0.5, dim=1)[:, :P].sum(0)
            assert torch.allclose(scores[b * H + h, :P].double(), want, rtol=RTOL, atol=0), (b, h)
            assert torch.isnan(scores[b * H + h, P:]).all()
            assert abs(float(mass[b * H + h]) - float(want.sum())) <= RTOL * float(want.sum()), (b, h)
    again, mass2 = torch.full_like(scores, float("nan")), torch.empty_like(mass)
    m.maskkv_score(desc, Q, K, 0.0, again, P_max + 3, mass2, ws)
    assert torch.equal(mass, mass2) and torch.equal(again.nan_to_num(-1.0), scores.nan_to_num(-1.0))


def test_logits_far_apart():
    """Rows whose parts' maxima differ by more than an exponential's range, and a key that outweighs all others."""
    m = hp.mk()
    gen = torch.Generator(device="cuda").manual_seed(3)
    H, n, d, P = 2, 20, 64, 700
    Q, K = torch.randn((1, H, n, d), generator=gen, device="cuda"), torch.randn((1, H, P + n, d), generator=gen, device="cuda")
    K[:, :, 64:128] *= 40
    K[:, 0, 333] = 0
    desc = m.Desc(B=1, H=H, d=d, dtype=m.MASKKV_F32, n_resp=n, P_max=P)
    from paper_2510_09309_amd import bench_binding as bb
    assert bb.maskkv_bench_score_split(desc).parts > 0
    scores, mass = torch.empty((H, P), device="cuda"), torch.empty((H,), device="cuda")
    m.maskkv_score(desc, Q, K, 0.0, scores, P, mass, hp.workspace(m.maskkv_score_workspace_bytes(desc)))
    s = Q[0].double() @ K[0].double().transpose(1, 2).contiguous() / d ** 0.5
    want = torch.softmax(s, dim=2)[:, :, :P].sum(1)
    # logits of up to 2^9 are off by 2^-15 (their products' sums), and so are exponentials, relative to themselves; below fp32's range they are 0
    assert torch.allclose(scores.double(), want, rtol=2.0 ** -13, atol=1e-37)
    assert torch.allclose(mass.double(), want.sum(1), rtol=2.0 ** -13, atol=0)
