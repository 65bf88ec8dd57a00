"""The kernels that put parts together: the un-evicted call's splits of the keys, two to sixty-four of them and around the numbers that are
asked for at once, and the rows' statistics of the two scoring passes with one group of rows to several, empty prompts among them (needs an
MI355X)."""
import pytest
import torch

from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("splits", [2, 3, 4, 5, 7, 8, 9, 16, 17, 64])
@pytest.mark.parametrize("d,dtype", [(128, "bf16"), (64, "bf16"), (128, "f32"), (64, "f32")])
def test_splits_of_the_keys(d, dtype, splits):
    """(A split is 512 keys or more, and the last one is short.  Fewer than ten are a narrow kernel's, which has none.)"""
    m = hp.mk()
    gen = torch.Generator(device="cuda").manual_seed(splits + d)
    H, n, P = 2, 37, 512 * splits - 100
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    Q, K, V = (torch.randn((1, H, x, d), generator=gen, device="cuda").to(t) for x in (n, P + n, P + n))
    Q[0, 1] *= 4                                                    # (weights far apart)
    O, lse = torch.full((1, H, n, d), float("nan"), device="cuda").to(t), torch.full((H, n), float("nan"), device="cuda")
    desc = m.Desc(B=1, H=H, d=d, dtype=m.MASKKV_BF16 if dtype == "bf16" else m.MASKKV_F32, n_resp=n, P_max=P)
    m.maskkv_attend_full(desc, Q, K, V, 0.0, O, lse, hp.workspace(m.maskkv_attend_workspace_bytes(desc, True)))
    for h in range(H):
        s = Q[0, h].double() @ K[0, h].double().T / d ** 0.5
        p, v = torch.softmax(s, dim=1), V[0, h].double()
        # a logit is a sum of d products, each addition off by up to 2^-24 of the terms' magnitudes; an exponential is off by as much
        # relative to itself, a weight by twice that, and sums of them by less than 2^-17.  bf16: a probability and the result are
        # rounded as well, by up to 2^-8 of themselves each (and the products are exact)
        off = d * 2.0 ** -24 * (Q[0, h].double().abs() @ K[0, h].double().abs().T / d ** 0.5).amax(1)
        weights = 2.0 ** -7 if dtype == "bf16" else (2 * off + 2.0 ** -17)[:, None]
        assert ((O[0, h].double() - p @ v).abs() <= weights * (p @ v.abs())).all()
        assert ((lse[h].double() - torch.logsumexp(s, dim=1)).abs() <= off + 2.0 ** -17).all()


# heads of 250 queries, each a workgroup's, that leave every compute unit a workgroup with so many splits
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("dtype,H,splits", [("bf16", 90, 2), ("bf16", 80, 3), ("bf16", 60, 4), ("bf16", 50, 5), ("bf16", 30, 8), ("bf16", 28, 9),
                                            ("f32", 128, 2), ("f32", 90, 3), ("f32", 80, 4), ("f32", 52, 5), ("f32", 32, 8), ("f32", 30, 9)])
def test_few_splits_of_many_heads(d, dtype, H, splits):
    """Two, four and eight splits, which are asked for at once, and one more; too many keys or groups of 32 queries for the narrow kernels,
    which leave nothing in the workspace."""
    m = hp.mk()
    gen = torch.Generator(device="cuda").manual_seed(H + d)
    n, P = 250, 1800 if H > 73 else 9000
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    Q, K, V = (torch.randn((1, H, x, d), generator=gen, device="cuda").to(t) for x in (n, P + n, P + n))
    Q[0, H // 2] *= 4                                               # (weights far apart)
    O, lse = torch.full((1, H, n, d), float("nan"), device="cuda").to(t), torch.full((H, n), float("nan"), device="cuda")
    desc = m.Desc(B=1, H=H, d=d, dtype=m.MASKKV_BF16 if dtype == "bf16" else m.MASKKV_F32, n_resp=n, P_max=P)
    rows = H * splits * n
    at = (rows * d * 4 + 255) // 256 * 256                          # (references and sums, behind the partial outputs)
    ws = torch.full((m.maskkv_attend_workspace_bytes(desc, True),), 0xFF, dtype=torch.uint8, device="cuda")
    assert ws.numel() == at + rows * 8
    m.maskkv_attend_full(desc, Q, K, V, 0.0, O, lse, ws)
    assert torch.isfinite(ws[at:].view(torch.float32)).all() and torch.isfinite(ws[:rows * d * 4].view(torch.float32)).all()
    for h in (0, H // 2, H - 1):
        s = Q[0, h].double() @ K[0, h].double().T / d ** 0.5
        p, v = torch.softmax(s, dim=1), V[0, h].double()
        off = d * 2.0 ** -24 * (Q[0, h].double().abs() @ K[0, h].double().abs().T / d ** 0.5).amax(1)     # (see above)
        weights = 2.0 ** -7 if dtype == "bf16" else (2 * off + 2.0 ** -17)[:, None]
        assert ((O[0, h].double() - p @ v).abs() <= weights * (p @ v.abs())).all()
        assert ((lse[h].double() - torch.logsumexp(s, dim=1)).abs() <= off + 2.0 ** -17).all()


@pytest.mark.parametrize("n,g", [(100, 1), (256, 1), (257, 1), (300, 2), (130, 7)])
@pytest.mark.parametrize("Ps", [(6000, 0, 5000), (0, 0, 0)])
def test_statistics_of_many_rows(n, g, Ps):
    """fp32 and prompts beyond the one pass's, so that the two passes serve the call.  fp32 logits of up to 2^4 are off by 2^-20 or less, an
    exponential and a sum of them by as much relative to themselves, the two passes' one after the other; a mass is a sum of shares."""
    m = hp.mk()
    gen = torch.Generator(device="cuda").manual_seed(n + g)
    B, H, d, P_max = 3, 2, 64, 6000
    Q = torch.randn((B, H * g, n, d), generator=gen, device="cuda")
    K = torch.randn((B, H, P_max + n, d), generator=gen, device="cuda")
    desc = m.Desc(B=B, H=H, d=d, dtype=m.MASKKV_F32, n_resp=n, P_max=P_max, prompt_len=list(Ps), q_per_kv=0 if g == 1 else g)
    scores, mass = torch.full((B * H, P_max), float("nan"), device="cuda"), torch.full((B * H,), float("nan"), device="cuda")
    m.maskkv_score(desc, Q, K, 0.0, scores, P_max, mass, hp.workspace(m.maskkv_score_workspace_bytes(desc)))
    for b, P in enumerate(Ps):
        for h in range(H):
            q = Q[b, h * g:(h + 1) * g].reshape(g * n, d).double()
            want = torch.softmax(q @ K[b, h, :P + n].double().T / d ** 0.5, dim=1)[:, :P].sum(0)
            assert torch.allclose(scores[b * H + h, :P].double(), want, rtol=2.0 ** -18, atol=0)
            assert abs(float(mass[b * H + h]) - float(want.sum())) <= 2.0 ** -18 * float(want.sum())
