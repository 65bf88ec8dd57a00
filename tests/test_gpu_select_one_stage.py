"""The one-stage selection at the edges of its prompt lengths, windows and ranks, against the fp32 oracle on given
scores, and the head budgets on either side of one wave of heads (needs an MI355X)."""
import numpy as np
import pytest
import torch

from oracle import maskkv_oracle as orc
from tests import helpers as hp

pytestmark = pytest.mark.gpu


def _scores(kind, rng, P):
    if kind == "tailed":
        return np.exp(3 * rng.standard_normal(P)).astype(np.float32)
    if kind == "ties":         # a few values, so that hundreds of entries tie at the cut
        return rng.choice(np.array([0.0, -0.0, 0.25, 0.5], dtype=np.float32), size=P)
    if kind == "ends":         # the largest at both ends: windows cut by the prompt's ends
        return (np.abs(np.linspace(-1, 1, P)) + 1e-3 * rng.random(P)).astype(np.float32)
    return (rng.standard_normal(P) * 10.0 ** rng.integers(-38, 30, P)).astype(np.float32)   # "wide": signs, denormals


@pytest.mark.parametrize("P", [1, 3, 5, 64, 1023, 1024, 1025, 4096, 4097, 8192, 8193, 16384, 16385])
@pytest.mark.parametrize("window,mode", [(1, 0), (7, 0), (7, 1), (9, 0), (13, 0), (17, 1), (19, 0)])
def test_one_stage(P, window, mode):
    m = hp.mk()
    kinds = ["tailed", "ties", "ends", "wide"]
    rng = np.random.default_rng(P * 31 + window)
    sc = np.stack([_scores(kind, rng, P) for kind in kinds for _ in range(4)])
    H = len(sc)
    budgets = np.array([1, min(P, 65), P // 2, P - 1] * 4, dtype=np.int32)
    cap = int(budgets.sum())
    desc = m.Desc(B=1, H=H, d=64, dtype=m.MASKKV_BF16, n_resp=8, P_max=P)
    idx = torch.full((cap + 1,), -7, dtype=torch.int32, device="cuda")
    cu = torch.zeros(H + 1, dtype=torch.int32, device="cuda")
    m.maskkv_select(desc, torch.from_numpy(sc).to("cuda"), P, window, mode, torch.from_numpy(budgets).to("cuda"), idx, cu,
                    cap, hp.workspace(m.maskkv_select_workspace_bytes(desc)))
    torch.cuda.synchronize()
    keeps, _ = hp.split_idx(idx, cu)
    assert int(idx[cap]) == -7
    for h in range(H):
        ref = orc.select(orc.pool(sc[h], window, ["mean", "max"][mode], dtype=np.float32), int(budgets[h]))
        assert np.array_equal(keeps[h], ref), f"P {P} window {window} mode {mode} head {h} ({kinds[h // 4]})"


@pytest.mark.parametrize("P", [9, 3000, 9001, 20000])
@pytest.mark.parametrize("window", [5, 7, 11, 17])
@pytest.mark.parametrize("scale", [1.0, 2.0 ** -59, 2.0 ** -62, 2.0 ** 56, 2.0 ** 59, 2.0 ** 120])
def test_means_a_last_place_apart(P, window, scale):
    """Means whose order hangs on the rounding of the quotient, on either side of what the product with the reciprocal is taken for."""
    m = hp.mk()
    rng = np.random.default_rng(P + window)
    H = 6
    sc = ((1 + rng.integers(0, 64, (H, P)) * 2.0 ** -23) * scale).astype(np.float32)
    budgets = np.array([1, 2, P // 3, P // 2, min(P - 1, 900), P], dtype=np.int32)
    cap = int(budgets.sum())
    desc = m.Desc(B=1, H=H, d=64, dtype=m.MASKKV_BF16, n_resp=8, P_max=P)
    idx, cu = torch.zeros(cap, dtype=torch.int32, device="cuda"), torch.zeros(H + 1, dtype=torch.int32, device="cuda")
    m.maskkv_select(desc, torch.from_numpy(sc).to("cuda"), P, window, 0, torch.from_numpy(budgets).to("cuda"), idx, cu, cap,
                    hp.workspace(max(1, m.maskkv_select_workspace_bytes(desc))))
    keeps, _ = hp.split_idx(idx, cu)
    for h in range(H):
        assert np.array_equal(keeps[h], orc.select(orc.pool(sc[h], window, "mean", dtype=np.float32), int(budgets[h]))), h


@pytest.mark.parametrize("H", [1, 32, 64, 65, 256, 300])
def test_head_budgets_around_one_wave_of_heads(H):
    m = hp.mk()
    rng = np.random.default_rng(H)
    mass = rng.random((2, H)).astype(np.float32) * 16
    desc = m.Desc(B=2, H=H, d=64, dtype=m.MASKKV_BF16, n_resp=16, P_max=64)
    out = torch.zeros(2 * H, dtype=torch.int32, device="cuda")
    m.maskkv_head_budgets(desc, torch.from_numpy(mass).to("cuda"), 128, 0.1, out)
    share = mass.astype(np.float64) / mass.astype(np.float64).sum(1, keepdims=True)
    ref = 0.1 * 128 + 0.9 * H * 128 * share
    assert np.abs(out.cpu().numpy().reshape(2, H) - np.floor(ref)).max() <= 1      # (fp32 arithmetic before the floor)
