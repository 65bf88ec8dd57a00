"""The scoring workspace of descriptions that maskkv_score_static serves (no GPU: the query is host arithmetic).

maskkv_score_static has MASKKV_STATIC_SCRATCH_BYTES for whatever it runs, and what does not fit takes the two passes instead of the single
sweep: slower, and with other bits than maskkv_score.
"""
import pytest

from paper_2510_09309_amd import bench_binding as bb
from paper_2510_09309_amd import binding as m

STATIC = 16 << 20


# (the last two: two groups of rows, whose column sums one workgroup adds up itself)
@pytest.mark.parametrize("d,n,H,g,Ps", [
    (128, 234, 28, 1, (17452, 12950, 9000, 17000, 11000, 15000)), (128, 234, 28, 1, (12950,) * 6), (128, 512, 32, 1, (8464, 6000)),
    (128, 344, 8, 1, (28000, 20000, 25000, 27000, 26000))])
def test_swept_descriptions_fit_the_static_scratch(d, n, H, g, Ps):
    desc = m.Desc(B=len(Ps), H=H, d=d, dtype=m.MASKKV_BF16, n_resp=n, P_max=max(Ps), prompt_len=list(Ps), q_per_kv=0 if g == 1 else g)
    assert bb.maskkv_bench_score_plan(desc).groups > 0
    assert m.maskkv_score_workspace_bytes(desc) <= STATIC
