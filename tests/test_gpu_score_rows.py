"""The one-pass scoring kernel of short fp32 prompts: edges of its tiles of 16 keys and of its groups of 16 rows, several groups of
a workgroup, grouped queries, empty prompts, strides, its longest prompts and the first ones that are too long (needs an MI355X).

Reference: float64 on the same inputs.  fp32 logits of up to 2^4 are off by 2^-20 or less, an exponential and a sum of them by as
much relative to themselves.
"""
import pytest
import torch

from tests import helpers as hp

pytestmark = pytest.mark.gpu

RTOL = 2.0 ** -19
# The two passes accumulate logits from minus the row's normaliser over scale * log2(e), a number of up to 2^7: eight times the rounding.
RTOL_TWO_PASSES = 2.0 ** -16


def way(desc):
    """(workgroups a head of the one pass, parts of the keys where rows and keys are both dealt out instead)"""
    from paper_2510_09309_amd import bench_binding as bb
    return bb.maskkv_bench_score_plan(desc).parts, bb.maskkv_bench_score_split(desc).parts


@pytest.mark.parametrize("d,n,H,g,Ps,ways", [
    (64, 1, 1, 1, (1,), (1, 0)), (128, 15, 2, 1, (15, 16, 17, 0), (1, 0)), (64, 48, 5, 4, (640, 463), (12, 0)),
    # (few workgroups' worth of rows: dealt out)
    (64, 17, 3, 1, (128, 367, 368, 95), (2, 7)), (128, 33, 2, 1, (351, 352, 607), (3, 10)), (128, 16, 2, 7, (1008, 1009, 1500), (7, 12)),
    (64, 60, 100, 1, (300, 20), (2, 0)), (128, 40, 130, 1, (200, 333, 64, 1), (1, 0)),       # several groups of rows a workgroup, or all of them
    (128, 100, 12, 1, (2972,), (7, 0)), (128, 100, 12, 1, (2973,), (0, 0))])                 # the most keys, and one more (two passes)
def test_against_float64(d, n, H, g, Ps, ways):
    m = hp.mk()
    gen = torch.Generator(device="cuda").manual_seed(d + n + H)
    B, P_max = len(Ps), max(Ps)
    Q = torch.randn((B, H * g, n, d), generator=gen, device="cuda")
    K = torch.randn((B, P_max + n, H, d), generator=gen, device="cuda").transpose(1, 2)   # (rows of a head are H * d apart)
    desc = m.Desc(B=B, H=H, d=d, dtype=m.MASKKV_F32, n_resp=n, P_max=P_max, prompt_len=None if B == 1 else list(Ps), q_per_kv=0 if g == 1 else g)
    scores, mass = torch.full((B * H, P_max + 3), float("nan"), device="cuda"), torch.full((B * H,), float("nan"), device="cuda")
    ws = hp.workspace(m.maskkv_score_workspace_bytes(desc))
    m.maskkv_score(desc, Q, K, 0.0, scores, P_max + 3, mass, ws)
    assert way(desc) == ways and (ways[0] > 0) == (P_max + n <= 3072)
    rtol = RTOL if P_max + n <= 3072 else RTOL_TWO_PASSES
    for b, P in enumerate(Ps):
        for h in range(0, H, 1 + H // 8):
            q = Q[b, h * g:(h + 1) * g].reshape(g * n, d).double()
            want = torch.softmax(q @ K[b, h, :P + n].double().T / d ** 0.5, dim=1)[:, :P].sum(0)
            assert torch.allclose(scores[b * H + h, :P].double(), want, rtol=rtol, atol=0), (b, h)
            assert torch.isnan(scores[b * H + h, P:]).all()
            assert abs(float(mass[b * H + h]) - float(want.sum())) <= rtol * float(want.sum()), (b, h)
    again, mass2 = torch.empty_like(scores), torch.empty_like(mass)
    m.maskkv_score(desc, Q, K, 0.0, again, P_max + 3, mass2, ws)
    assert torch.equal(mass, mass2)
    for b, P in enumerate(Ps):
        assert torch.equal(again[b * H:(b + 1) * H, :P], scores[b * H:(b + 1) * H, :P])


# as many tiles of 128 keys a wave as each form of the kernel holds, and one key more
@pytest.mark.parametrize("keys", [384, 385, 640, 641, 1024, 1025, 1536, 1537, 2048, 2049, 3072])
@pytest.mark.parametrize("H,short,parts", [(64, (), 2), (130, (1, 47), 1)])   # a workgroup a group of rows; two groups a workgroup
@pytest.mark.parametrize("d", [64, 128])
def test_every_number_of_tiles(d, H, short, parts, keys):
    """Two groups of 16 rows (one and a row more), a prompt that ends on a tile of 16 keys and one beside it."""
    m = hp.mk()
    n = 17
    Ps = [keys - n] + [keys - n - 1 if s == 1 else s for s in short]
    B, P_max = len(Ps), Ps[0]
    gen = torch.Generator(device="cuda").manual_seed(d + keys)
    Q = torch.randn((B, H, n, d), generator=gen, device="cuda")
    K = torch.randn((B, H, P_max + n, d), generator=gen, device="cuda")
    desc = m.Desc(B=B, H=H, d=d, dtype=m.MASKKV_F32, n_resp=n, P_max=P_max, prompt_len=None if B == 1 else Ps)
    assert way(desc) == (parts, 0)
    scores, mass = torch.full((B * H, P_max), float("nan"), device="cuda"), torch.full((B * H,), float("nan"), device="cuda")
    m.maskkv_score(desc, Q, K, 0.0, scores, P_max, mass, hp.workspace(m.maskkv_score_workspace_bytes(desc)))
    for b, P in enumerate(Ps):
        for h in range(b, H, 9):
            want = torch.softmax(Q[b, h].double() @ K[b, h, :P + n].double().T / d ** 0.5, dim=1)[:, :P].sum(0)
            # Of a million columns some have one row's largest logits for their sum, of 5 or 6: a sum of d products that grows to 64 is rounded
            # by some 2^-24 / sqrt(3) of it d times at random, the logit by 64 / sqrt(3) * 2^-24 / sqrt(3) = 2^-19.6, and four times that is 2^-17.6
            worst = float((scores[b * H + h, :P].double() / want - 1).abs().max())
            assert worst <= 2.0 ** -17, (b, h, worst)
            assert torch.isnan(scores[b * H + h, P:]).all()
            assert abs(float(mass[b * H + h]) - float(want.sum())) <= RTOL * float(want.sum()), (b, h)


@pytest.mark.parametrize("d,n,H,g,B,P,parts", [(64, 64, 2, 64, 1, 300, 256), (128, 96, 2, 32, 1, 300, 192), (64, 60, 32, 4, 16, 60, 1)])
def test_masses_of_many_groups_of_rows(d, n, H, g, B, P, parts):
    """256 and 192 workgroups a head, and 15 groups of a head in one: adding their masses loses less than rounding the result does."""
    m = hp.mk()
    gen = torch.Generator(device="cuda").manual_seed(d + n)
    Q = torch.randn((B, H * g, n, d), generator=gen, device="cuda")
    K = torch.randn((B, H, P + n, d), generator=gen, device="cuda")
    desc = m.Desc(B=B, H=H, d=d, dtype=m.MASKKV_F32, n_resp=n, P_max=P, q_per_kv=g)
    assert way(desc) == (parts, 0)
    scores, mass = torch.empty((B * H, P), device="cuda"), torch.empty((B * H,), device="cuda")
    m.maskkv_score(desc, Q, K, 0.0, scores, P, mass, hp.workspace(m.maskkv_score_workspace_bytes(desc)))
    A = torch.softmax(Q.double().view(B * H, g * n, d) @ K.double().view(B * H, P + n, d).transpose(1, 2).contiguous() / d ** 0.5, dim=2)
    want = A[:, :, :P].sum((1, 2))
    # a row's share is off by some 2^-22, at random, so the mean of a thousand rows or more by 2^-26; the quarters of 16 rows are added
    # and stored in fp32 (once, or 192 times at random), and the result is rounded by up to 2^-24
    rms = ((mass.double() / want - 1) ** 2).mean().sqrt()
    assert float(rms) <= 2.0 ** -24
