"""Attention of few query tiles over [packed rows ; response]: a wave takes blocks of 32 keys (bf16) or 16 (fp32), and each segment has a
last block of its own."""
import pytest
import torch

from tests import helpers as hp

pytestmark = pytest.mark.gpu


def attend(d, n, g, budgets, capacity=None, spoil=None, dtype=torch.bfloat16):
    """One sequence; K and V of the response are views into longer rows.  Result, the float64 reference and its sum of absolute terms."""
    m = hp.mk()
    H, total = len(budgets), sum(budgets)
    gen = torch.Generator(device="cuda").manual_seed(7)
    rnd = lambda *shape: torch.randn(shape, generator=gen, device="cuda").to(dtype)
    Q, Kc, Vc = rnd(1, H * g, n, d), rnd(max(total, 1), d), rnd(max(total, 1), d)
    K, V = rnd(1, H, 5 + n, d)[:, :, 5:], rnd(1, H, 3 + n, d)[:, :, 3:]
    if spoil:
        spoil(Kc, Vc, K, V)
    cu = torch.tensor([sum(budgets[:h]) for h in range(H + 1)], dtype=torch.int32, device="cuda")
    O, lse = torch.full((1, H * g, n, d), float("nan"), device="cuda").to(dtype), torch.zeros(H, g * n, device="cuda")
    desc = m.Desc(B=1, H=H, d=d, dtype=m.MASKKV_BF16 if dtype == torch.bfloat16 else m.MASKKV_F32, n_resp=n, P_max=max(max(budgets), 1), q_per_kv=0 if g == 1 else g)
    ws = hp.workspace(max(1, m.maskkv_attend_workspace_bytes(desc, False)))
    m.maskkv_attend(desc, Q, Kc, Vc, cu, total if capacity is None else capacity, K, V, 0.0, O, lse, ws)
    for h in range(H):
        rows = slice(sum(budgets[:h]), sum(budgets[:h + 1]))
        q = Q[0, h * g:(h + 1) * g].reshape(g * n, d).double()
        k, v = torch.cat([Kc[rows], K[0, h]]).double(), torch.cat([Vc[rows], V[0, h]]).double()
        s = q @ k.T / d ** 0.5
        p = torch.softmax(s, dim=1)
        yield O[0, h * g:(h + 1) * g].reshape(g * n, d).double(), p @ v, p @ v.abs(), lse[h].double(), torch.logsumexp(s, dim=1)


def check(results, bound=2.0 ** -8, atol=32 * 2.0 ** -24):
    # bf16: probabilities and results are rounded (2^-9 each); what fp32 adds is far below
    for out, want, terms, lse, want_lse in results:
        assert ((out - want).abs() <= bound * terms).all()
        assert torch.allclose(lse, want_lse, rtol=0, atol=atol)


@pytest.mark.parametrize("d,n,g,budgets", [
    (128, 1, 1, (0, 1, 31, 32, 33, 700)), (64, 1, 1, (0, 1, 31, 32, 33, 700)), (128, 33, 1, (223, 224, 225, 0)), (64, 255, 1, (1, 256, 600)),
    (128, 256, 1, (300,)), (128, 257, 1, (17, 2049)), (64, 100, 7, (64, 5)), (128, 37, 4, (0, 96)), (64, 640, 1, (130,) * 32),
    (128, 384, 1, (130, 7) * 16)])
def test_edges_of_segments_blocks_and_query_tiles(d, n, g, budgets):
    check(attend(d, n, g, budgets))


@pytest.mark.parametrize("d,n,g,budgets", [
    (128, 1, 1, (0, 1, 15, 16, 17, 700)), (64, 1, 1, (0, 1, 15, 16, 17, 700)), (64, 17, 1, (111, 112, 113, 0)), (128, 100, 7, (64, 5)),
    (64, 255, 1, (30,) * 16), (64, 257, 1, (30,) * 16)])  # (the last two: either side of a workgroup of 16 queries per compute unit)
def test_edges_in_fp32(d, n, g, budgets):
    # logits of up to 2^4 are rounded (2^-21) once for every four products, twice over for a probability and its sum
    check(attend(d, n, g, budgets, dtype=torch.float32), bound=d / 2 * 2.0 ** -21, atol=d / 4 * 2.0 ** -21)


@pytest.mark.parametrize("spare", [0, 20000])
def test_either_side_of_the_capacity_that_the_choice_of_kernel_looks_at(spare):
    budgets = (100, 0, 333) * 3
    check(attend(128, 1024, 1, budgets, sum(budgets) + spare))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d", [64, 128])
def test_an_infinite_value_in_a_segments_last_row(d, dtype):
    """The last rows are read again in place of the rows that fill their blocks, which must not show."""
    def spoil(Kc, Vc, K, V):
        Vc[39, 3] = float("inf")
        V[0, 0, 32, 5] = float("-inf")
    (out, want, _, _, _), = attend(d, 33, 1, (40,), spoil=spoil, dtype=dtype)
    finite = torch.isfinite(want)
    assert (out[:, 3] == float("inf")).all() and (out[:, 5] == float("-inf")).all()
    assert finite.sum() == want.numel() - 2 * 33 and torch.isfinite(out[finite]).all()
