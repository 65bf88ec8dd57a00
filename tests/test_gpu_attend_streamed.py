"""The un-evicted call whose V is read past the memory-side cache, next to its largest neighbour that is not: keys and values together just
above and just below that cache's 256 MiB (needs an MI355X)."""
import pytest
import torch

from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,H,n,P", [(128, 32, 200, 16185), (128, 32, 200, 16184), (64, 32, 100, 32700), (128, 40, 257, 13000),
                                       (128, 32, 100, 16300), (64, 32, 200, 32700)])
def test_either_side_of_the_cache(d, H, n, P):  # (100 queries: 128 a workgroup, otherwise 256; 257: two tiles of queries, which is not streamed)
    m = hp.mk()
    gen = torch.Generator(device="cuda").manual_seed(P)
    Q, K, V = (torch.randn((1, H, x, d), generator=gen, device="cuda").to(torch.bfloat16) for x in (n, P + n, P + n))
    O, lse = torch.full((1, H, n, d), float("nan"), device="cuda").to(torch.bfloat16), torch.zeros(H, n, device="cuda")
    desc = m.Desc(B=1, H=H, d=d, dtype=m.MASKKV_BF16, n_resp=n, P_max=P)
    m.maskkv_attend_full(desc, Q, K, V, 0.0, O, lse, hp.workspace(m.maskkv_attend_workspace_bytes(desc, True)))
    for h in (0, H // 2, H - 1):
        s = Q[0, h].double() @ K[0, h].double().T / d ** 0.5
        p, v = torch.softmax(s, dim=1), V[0, h].double()
        # a probability and the result are rounded to bf16, by up to 2^-8 of themselves each
        assert ((O[0, h].double() - p @ v).abs() <= 2.0 ** -7 * (p @ v.abs())).all()
        assert torch.allclose(lse[h].double(), torch.logsumexp(s, dim=1), rtol=0, atol=32 * 2.0 ** -24)
