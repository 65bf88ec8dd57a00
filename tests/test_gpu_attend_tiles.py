"""The tiled bf16 attention at the sizes where its schedule can go wrong, against the oracle (needs an MI355X): key axes of one
tile, of an odd number of tiles, ending inside a tile; the border of the packed cache and the strided rows at every place
of a wave's eight or sixteen rows; empty heads; query tiles that are partly or wholly without queries; both forms
(256 queries a workgroup, and 128 with the tiles dealt to the two groups of waves) and both launch orders."""
import numpy as np
import pytest
import torch

from oracle import maskkv_oracle as orc
from tests import helpers as hp

pytestmark = pytest.mark.gpu


def run(B, H, d, n, budgets, seed):
    m = hp.mk()
    rng = np.random.default_rng(seed)
    P = max(int(max(budgets)), 1)
    desc = m.Desc(B=B, H=H, d=d, dtype=m.MASKKV_BF16, n_resp=n, P_max=P, prompt_len=None if B == 1 else [P] * B)
    cu = np.concatenate([[0], np.cumsum(budgets)]).astype(np.int32)

    def draw(*shape):
        t = torch.from_numpy(rng.standard_normal(shape, dtype=np.float32)).to(torch.bfloat16)
        return t.cuda(), t.float().numpy()

    cap = int(cu[-1])
    Kc, Kc_h = draw(cap, d)
    Vc, Vc_h = draw(cap, d)
    Q, Q_h = draw(B, H, n, d)
    Kr, Kr_h = draw(B, H, n, d)
    Vr, Vr_h = draw(B, H, n, d)
    O = torch.full((B, H, n, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B * H * n,), float("nan"), dtype=torch.float32, device="cuda")
    ws = hp.workspace(m.maskkv_attend_workspace_bytes(desc, False))
    m.maskkv_attend(desc, Q, Kc, Vc, torch.from_numpy(cu).cuda(), cap, Kr, Vr, 0.0, O, lse, ws)
    torch.cuda.synchronize()
    O_h, lse_h = O.float().cpu().numpy(), lse.cpu().numpy().reshape(B * H, n)
    assert np.isfinite(O_h).all()
    for bh in sorted(set(np.linspace(0, B * H - 1, 24).astype(int)) | set(range(min(B * H, 4)))):
        b, h = divmod(bh, H)
        rows = slice(cu[bh], cu[bh + 1])
        ref, rl = orc.attend(Q_h[b, h], Kc_h[rows], Vc_h[rows], Kr_h[b, h], Vr_h[b, h], return_lse=True)
        err = np.abs(O_h[b, h] - ref).max()
        # values of order one: probabilities and outputs rounded to bf16 (2^-9 each, relative to sums of |p v| below about 5)
        assert err <= hp.ATTEND_ATOL_BF16, f"head {bh} budget {budgets[bh]}: {err:.3e}"
        assert np.abs(lse_h[bh] - rl).max() <= 1e-3


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,H,n,lo,hi", [
    (8, 32, 33, 0, 31),       # one tile, or one and a few keys of a second; 128 queries a workgroup, most waves without any
    (4, 48, 100, 1, 180),     # one to five tiles, odd and even, 128 a workgroup
    (2, 60, 257, 0, 70),      # a third tile of queries with one row
    (8, 32, 129, 0, 200),     # 256 a workgroup, unordered
    (8, 40, 260, 3, 300),     # 256 a workgroup, ordered, the second tile of queries nearly empty
])
def test_tiles(B, H, n, lo, hi, d):
    budgets = [lo + (i * 37) % (hi - lo + 1) for i in range(B * H)]
    run(B, H, d, n, budgets, seed=B * 1000 + n + d)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("P,n", [(1, 5), (63, 64), (700, 130), (1500, 256), (2049, 127)])
def test_tiles_full_sequence(P, n, d):
    """The un-evicted call: splits that end inside a tile, one split, fewer queries than a workgroup serves."""
    m = hp.mk()
    rng = np.random.default_rng(P + d)
    H, N = 4, P + n
    desc = m.Desc(B=1, H=H, d=d, dtype=m.MASKKV_BF16, n_resp=n, P_max=P)
    t = [torch.from_numpy(rng.standard_normal((1, H, x, d), dtype=np.float32)).to(torch.bfloat16) for x in (n, N, N)]
    Q, K, V = [x.cuda() for x in t]
    O = torch.full((1, H, n, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((H * n,), float("nan"), dtype=torch.float32, device="cuda")
    m.maskkv_attend_full(desc, Q, K, V, 0.0, O, lse, hp.workspace(m.maskkv_attend_workspace_bytes(desc, True)))
    torch.cuda.synchronize()
    for h in range(H):
        ref, rl = orc.attend_full(*[x[0, h].float().numpy() for x in t], return_lse=True)
        assert np.abs(O[0, h].float().cpu().numpy() - ref).max() <= hp.ATTEND_ATOL_BF16
        assert np.abs(lse.cpu().numpy().reshape(H, n)[h] - rl).max() <= 1e-3


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [100, 256, 300])
def test_tiles_empty_parts(n, d):
    """The un-evicted call over a batch whose shortest sequences leave parts of the key axis without a key: such a part has nothing to
    wait for, and may not leave a transfer into LDS behind for whoever gets that LDS next."""
    m = hp.mk()
    gen = torch.Generator(device="cuda").manual_seed(n + d)
    B, H, Ps = 3, 4, [9000, 1, 200]
    N = max(Ps) + n
    desc = m.Desc(B=B, H=H, d=d, dtype=m.MASKKV_BF16, n_resp=n, P_max=max(Ps), prompt_len=Ps)
    Q, K, V = (torch.randn((B, H, x, d), generator=gen, device="cuda").to(torch.bfloat16) for x in (n, N, N))
    O = torch.full((B, H, n, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B * H, n), float("nan"), dtype=torch.float32, device="cuda")
    m.maskkv_attend_full(desc, Q, K, V, 0.0, O, lse, hp.workspace(m.maskkv_attend_workspace_bytes(desc, True)))
    for b, P in enumerate(Ps):
        for h in range(H):
            s = Q[b, h].double() @ K[b, h, :P + n].double().T / d ** 0.5
            p, v = torch.softmax(s, dim=1), V[b, h, :P + n].double()
            # a probability and the result are rounded to bf16, by up to 2^-8 of themselves each
            assert ((O[b, h].double() - p @ v).abs() <= 2.0 ** -7 * (p @ v.abs())).all()
            assert ((lse[b * H + h].double() - torch.logsumexp(s, dim=1)).abs() <= 2.0 ** -14).all()
