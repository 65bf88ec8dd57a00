"""The narrow attention in fp32, where four waves share a head's keys, against the oracle (needs an MI355X): fewer 32-key blocks
than waves, blocks that end inside, empty heads, query tiles with one row, and the border to the tiled kernel."""
import numpy as np
import pytest
import torch

from oracle import maskkv_oracle as orc
from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,n,lo,hi", [(1, 1, 0, 0), (3, 33, 0, 5), (5, 64, 30, 140), (9, 100, 0, 300), (130, 256, 0, 40)])
def test_narrow_f32(H, n, lo, hi, d):
    m = hp.mk()
    rng = np.random.default_rng(H * 100 + n + d)
    budgets = [lo + (i * 37) % (hi - lo + 1) for i in range(H)]
    cu = np.concatenate([[0], np.cumsum(budgets)]).astype(np.int32)
    cap = int(cu[-1])
    desc = m.Desc(B=1, H=H, d=d, dtype=m.MASKKV_F32, n_resp=n, P_max=max(hi, 1))
    host = [rng.standard_normal(s, dtype=np.float32) for s in ((1, H, n, d), (max(cap, 1), d), (max(cap, 1), d), (1, H, n, d), (1, H, n, d))]
    Q, Kc, Vc, Kr, Vr = [torch.from_numpy(x).cuda() for x in host]
    O = torch.full((1, H, n, d), float("nan"), dtype=torch.float32, device="cuda")
    lse = torch.full((H * n,), float("nan"), dtype=torch.float32, device="cuda")
    m.maskkv_attend(desc, Q, Kc, Vc, torch.from_numpy(cu).cuda(), cap, Kr, Vr, 0.0, O, lse,
                    hp.workspace(m.maskkv_attend_workspace_bytes(desc, False)))
    torch.cuda.synchronize()
    for h in sorted({0, 1, H // 2, H - 1} & set(range(H))):
        rows = slice(cu[h], cu[h + 1])
        ref, rl = orc.attend(host[0][0, h], host[1][rows], host[2][rows], host[3][0, h], host[4][0, h], return_lse=True)
        # fp32 sums of up to 556 terms of order one
        assert np.abs(O[0, h].cpu().numpy() - ref).max() <= hp.ATTEND_ATOL_F32
        assert np.abs(lse.cpu().numpy().reshape(H, n)[h] - rl).max() <= 1e-5
