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


def check(results, bound=2.0 ** -7, atol=32 * 2.0 ** -24):
    # bf16 has 8 significant bits: rounding to nearest is off by up to 2^-8 of the value, once for a probability and once for the
    # result (with two keys both can be nearly that: nothing averages); what fp32 adds is far below
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


@pytest.mark.parametrize("dtype,B,H,d,n,g,P", [
    ("bf16", 1, 3, 128, 1, 1, [1]), ("bf16", 3, 2, 64, 33, 1, [0, 700, 255]), ("bf16", 2, 4, 128, 100, 7, [300, 29]), ("bf16", 1, 9, 128, 1000, 1, [500]),
    ("bf16", 1, 4, 128, 64, 1, [2716]), ("bf16", 1, 4, 128, 64, 1, [2717]), ("bf16", 2, 2, 64, 70, 1, [4100, 5]), ("bf16", 1, 9, 64, 1000, 1, [4100]),
    ("f32", 1, 3, 128, 1, 1, [1]), ("f32", 3, 2, 64, 17, 1, [0, 700, 255]), ("f32", 2, 4, 128, 20, 7, [300, 29]), ("f32", 1, 2, 64, 40, 1, [4961]),
    ("f32", 1, 17, 64, 256, 1, [700]), ("f32", 1, 9, 128, 1000, 1, [600])])
def test_un_evicted(dtype, B, H, d, n, g, P):
    """Whichever kernel serves the call: prompts of few keys and none, either side of the lengths at which it changes."""
    m = hp.mk()
    dt, code = (torch.bfloat16, m.MASKKV_BF16) if dtype == "bf16" else (torch.float32, m.MASKKV_F32)
    gen = torch.Generator(device="cuda").manual_seed(11)
    Q, K, V = (torch.randn(s, generator=gen, device="cuda").to(dt) for s in ((B, H * g, n, d), (B, H, max(P) + n, d), (B, H, max(P) + n, d)))
    O, lse = torch.full((B, H * g, n, d), float("nan"), device="cuda").to(dt), torch.zeros(B * H, g * n, device="cuda")
    desc = m.Desc(B=B, H=H, d=d, dtype=code, n_resp=n, P_max=max(max(P), 1), prompt_len=None if B == 1 else P, q_per_kv=0 if g == 1 else g)
    m.maskkv_attend_full(desc, Q, K, V, 0.0, O, lse, hp.workspace(max(1, m.maskkv_attend_workspace_bytes(desc, True))))

    def results():
        for i in range(B * H):
            b, h = divmod(i, H)
            q = Q[b, h * g:(h + 1) * g].reshape(g * n, d).double()
            s = q @ K[b, h, :P[b] + n].double().T / d ** 0.5
            p, v = torch.softmax(s, dim=1), V[b, h, :P[b] + n].double()
            yield O[b, h * g:(h + 1) * g].reshape(g * n, d).double(), p @ v, p @ v.abs(), lse[i].double(), torch.logsumexp(s, dim=1)
    if dtype == "bf16":
        check(results())
    else:
        check(results(), bound=d / 2 * 2.0 ** -21, atol=d / 4 * 2.0 ** -21)
