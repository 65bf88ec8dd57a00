"""The single-sweep scoring kernel (bf16, prompts of at most one chunk of 128 keys per compute unit): edges of its chunks, row
groups and response span, its fallback for row sums out of range, and calls on two streams at once (needs an MI355X).

Reference: the oracle, or for long prompts maskkv_score_given_lse with the normalisers of maskkv_attend_full, which is another
kernel (the second of two passes) on the same inputs.
"""
import numpy as np
import pytest
import torch

from oracle import maskkv_oracle as orc
from paper_2510_09309_amd import synth
from tests import helpers as hp

pytestmark = pytest.mark.gpu


def given_lse(batch):
    m = hp.mk()
    lse = torch.empty(batch.B * batch.H * batch.n_m, dtype=torch.float32, device="cuda")
    O = torch.empty_like(batch.Q)
    m.maskkv_attend_full(batch.desc, batch.Q, batch.K, batch.V, 0.0, O, lse,
                         hp.workspace(m.maskkv_attend_workspace_bytes(batch.desc, True)))
    return hp.gpu_score_given_lse(batch, lse)


@pytest.mark.parametrize("d,n_m,Ps", [
    (128, 1, (1,)), (128, 31, (127, 128, 129)), (64, 33, (96, 0, 2049)), (128, 257, (640, 1000)), (64, 300, (5, 4000, 1))])
def test_edges_of_chunks_and_row_groups(d, n_m, Ps):
    batch = hp.Batch([synth.make_layer(70 + i, H=3, d=d, P=P, n_m=n_m, dtype="bf16", n_planted=P // 50, amplitude=2.5)
                      for i, P in enumerate(Ps)])
    scores, mass = hp.gpu_score(batch)
    assert hp.check_scores(batch, scores, mass) <= 1e-4


@pytest.mark.parametrize("H,P", [(2, 32768), (2, 32769), (5, 17000), (3, 16384)])
def test_longest_prompts_agree_with_the_second_pass_alone(H, P):
    """One chunk per compute unit at most; 32769 tokens are one too many and take the two passes."""
    batch = hp.Batch([synth.make_layer(80, H=H, d=128, P=P, n_m=96, dtype="bf16", n_planted=P // 50, amplitude=2.5)])
    scores, mass = hp.gpu_score(batch)
    want, want_mass = given_lse(batch)
    assert torch.allclose(scores[:, :P], want[:, :P], rtol=2e-5, atol=0)
    assert torch.allclose(mass, want_mass, rtol=2e-5, atol=0)
    again, _ = hp.gpu_score(batch)
    assert torch.equal(again[:, :P], scores[:, :P])


@pytest.mark.parametrize("d,boost,keys", [(128, 12.0, 1), (128, 24.0, 1), (128, 40.0, 1), (64, 400.0, 1), (128, 60.0, 700)])
def test_prompt_far_above_the_response_span(d, boost, keys):
    """Row sums are exchanged in units of the response span's own: one prompt key that is e^12 or e^24 above it stays in range
    (of the wide unit), e^40 and e^400 do not and are left to the fallback, as is a prompt that lies above it as a whole."""
    L = synth.make_layer(90, H=2, d=d, P=700, n_m=40, dtype="bf16", n_planted=0, amplitude=0.0, query_shift=4.0)
    for h in range(L.H):
        where = slice(333, 334) if keys == 1 else slice(0, keys)
        L.K[h, where] += synth.round_to_bf16(np.float32(boost * np.sqrt(d) / 4.0) * L.u[h])
    L.K[:] = synth.round_to_bf16(L.K)
    batch = hp.Batch([L])
    scores, mass = hp.gpu_score(batch)
    for h in range(L.H):
        I, m = orc.score(L.Q[h], L.K[h], L.P)
        got = scores[h, :L.P].double().cpu().numpy()
        assert np.isfinite(got).all()
        assert np.abs(got - I).max() <= 1e-4 * I.max()
        big = I > 1e-30
        assert (np.abs(got - I)[big] <= 1e-3 * I[big]).all()
        assert abs(float(mass[h]) - m) <= 1e-4 * m


def test_calls_on_two_streams_at_once():
    """Only one sweep at a time has a device to itself; a call that finds another one running takes the fallback."""
    m = hp.mk()
    batches = [hp.Batch([synth.make_layer(95 + i, H=16, d=128, P=4000 + 77 * i, n_m=128, dtype="bf16", n_planted=50, amplitude=2.5)])
               for i in range(2)]
    want = [hp.gpu_score(b) for b in batches]
    streams = [torch.cuda.Stream() for _ in range(2)]
    ws = [hp.workspace(m.maskkv_score_workspace_bytes(b.desc)) for b in batches]
    got = [(torch.zeros_like(w[0]), torch.zeros_like(w[1])) for w in want]
    torch.cuda.synchronize()
    for rep in range(20):
        for b, st, w, g in zip(batches, streams, ws, got):
            m.maskkv_score(b.desc, b.Q, b.K, 0.0, g[0], g[0].stride(0), g[1], w, st)
    torch.cuda.synchronize()
    for b, w, g in zip(batches, want, got):
        P = b.P[0]
        assert torch.allclose(g[0][:, :P], w[0][:, :P], rtol=5e-6, atol=0)
        assert torch.allclose(g[1], w[1], rtol=5e-6, atol=0)
    after = hp.gpu_score(batches[0])     # the device is free again
    assert torch.equal(after[0][:, :batches[0].P[0]], want[0][0][:, :batches[0].P[0]])


@pytest.mark.parametrize("d,P,n_m,row_bytes", [(128, 40, 300, 1 << 24), (64, 200, 260, 1 << 24), (128, 60, 8230, 1 << 19)])
def test_response_rows_more_than_4_gib_apart(d, P, n_m, row_bytes):
    """Token strides up to 16 MiB: the response span of one head may reach over more than 32 bits of offset."""
    m = hp.mk()
    n_q = 40
    L = synth.make_layer(93, H=1, d=d, P=P, n_m=n_m, dtype="bf16", n_planted=0, amplitude=0.0, query_shift=4.0)
    for h in range(L.H):     # rows differ along the response span, so that rows read twice or not at all show
        L.K[h, P:] += (np.linspace(0.0, 4.0, n_m, dtype=np.float32) * np.float32(np.sqrt(d) / 4.0))[:, None] * L.u[h]
    L.K[:] = synth.round_to_bf16(L.K)
    wide = torch.empty((P + n_m, row_bytes // 2), dtype=torch.bfloat16, device="cuda")
    K = wide[:, :d]
    K.copy_(torch.from_numpy(L.K[0]).to("cuda"))
    Q = hp.upload(L.Q[None, :, :n_q], "bf16")
    desc = m.Desc(B=1, H=1, d=d, dtype=m.MASKKV_BF16, n_resp=n_m, P_max=P, n_query=n_q)
    scores = torch.full((1, 256), float("nan"), device="cuda")
    mass = torch.zeros(1, device="cuda")
    m.maskkv_score(desc, Q, K[None, None], 0.0, scores, 256, mass, hp.workspace(m.maskkv_score_workspace_bytes(desc)))
    I, want = orc.score(L.Q[0, :n_q], L.K[0], P)
    got = scores[0, :P].double().cpu().numpy()
    # raw logits below 100 in fp32 are 2^-17 coarse at most: some 1e-5 of an exponential, and rows read wrongly are off by 0.1
    assert np.abs(got / I - 1).max() <= 1e-4
    assert abs(float(mass[0]) / want - 1) <= 1e-4
