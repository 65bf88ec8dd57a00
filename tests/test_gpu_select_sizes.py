"""select around the edges of its launch shapes: prompts just below and above every step of threads and of groups a thread, windows
on both sides of the loaded pieces, and the ends of the prompt at every place of a lane's four positions."""
import numpy as np
import pytest

import helpers as hp
from oracle import maskkv_oracle as orc

pytestmark = pytest.mark.gpu

EDGES = [3, 4, 5, 6, 7, 255, 258, 1024, 1025, 2048, 2050, 3072, 3075, 4096, 4097, 6144, 6147, 8192, 8194, 9216, 9217, 12288, 12291,
         16383, 16384, 16385]


def run(sc, Ps, budgets, window, mode):
    """`sc` [B * H, P_max], one list of kept positions per head."""
    import torch
    m = hp.mk()
    BH, P_max = sc.shape
    desc = m.Desc(B=len(Ps), H=BH // len(Ps), d=128, dtype=m.MASKKV_BF16, n_resp=8, P_max=P_max, prompt_len=Ps)
    cap = int(budgets.sum())
    idx = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
    cu = torch.zeros(BH + 1, dtype=torch.int32, device="cuda")
    m.maskkv_select(desc, torch.from_numpy(sc).to("cuda"), P_max, window, mode, torch.from_numpy(budgets).to("cuda"), idx, cu, cap,
                    hp.workspace(m.maskkv_select_workspace_bytes(desc)))
    torch.cuda.synchronize()
    return hp.split_idx(idx, cu)[0]


@pytest.mark.parametrize("window,mode", [(1, "mean"), (5, "mean"), (7, "mean"), (9, "mean"), (11, "mean"), (17, "mean"), (7, "max"),
                                         (9, "max"), (17, "max")])
def test_every_launch_shape_is_bit_exact(window, mode):
    """Two sequences, the second one position to four short of the first; one head of each keeps a few, one almost all, one has ties
    at its cut.  Every decision is made in fp32 on both sides, so the lists are identical."""
    rng = np.random.default_rng(17 * window + len(mode))
    for P in EDGES:
        Ps = [P, P - 1 - P % 4 if P > 4 else P]
        sc = rng.random((6, P)).astype(np.float32)
        sc[2::3] = np.round(sc[2::3] * 8) / 8
        sc[1] -= np.float32(0.5)
        budgets = np.array([k for p in Ps for k in (min(p, 37), max(p - 2, 1), (p + 1) // 2)], dtype=np.int32)
        keeps = run(sc, Ps, budgets, window, 0 if mode == "mean" else 1)
        for bh in range(6):
            ref = orc.select(orc.pool(sc[bh, :Ps[bh // 3]], window, mode, dtype=np.float32), int(budgets[bh]))
            assert np.array_equal(keeps[bh], ref), f"P {Ps[bh // 3]} window {window} {mode} head {bh}"


@pytest.mark.parametrize("P", [1021, 4093, 16381, 20001])
def test_scores_of_the_lowest_key_are_ties_within_the_prompt(P):
    """A negative NaN of all ones is the lowest key there is, that of positions past the prompt: whatever is kept lies inside it."""
    sc = np.full((2, P), -1, dtype=np.int32).view(np.float32)
    budgets = np.array([P, P - 5], dtype=np.int32)
    keeps = run(sc, [P], budgets, 1, 0)
    for bh in range(2):
        assert np.array_equal(keeps[bh], np.arange(budgets[bh]))


@pytest.mark.parametrize("P", [8193, 9217, 12289, 16384])
def test_budgets_around_the_bounds_of_the_histogram(P):
    """As many kept positions as there are threads, quads and rows of lanes with a key, and one more or less; scores in ascending order and
    ones of which all but a few lie in one thread's four positions put the k-th largest at the bound."""
    rng = np.random.default_rng(P)
    threads = min((1024 if P > 9216 or P <= 8192 else 768), (P + 3) // 4)
    ks = [k + e for k in ((threads + 15) // 16, (threads + 3) // 4, threads) for e in (-1, 0, 1)]
    for kind in range(3):
        sc = rng.random((len(ks), P)).astype(np.float32)
        if kind == 1:
            sc = np.sort(sc, axis=1)
        if kind == 2:
            sc[:, 256:] *= np.float32(2.0 ** -20)
        budgets = np.array(ks, dtype=np.int32)
        for window in (1, 7):
            keeps = run(sc, [P], budgets, window, 0)
            for h in range(len(ks)):
                assert np.array_equal(keeps[h], orc.select(orc.pool(sc[h], window, "mean", dtype=np.float32), ks[h])), (kind, window, ks[h])
