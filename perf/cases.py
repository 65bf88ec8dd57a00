"""What a program that serves a masked diffusion language model asks of this library, as measurable cases.

A program compresses the prompt's cache once per layer and request (score, select, compact), then attends over the
evicted cache at every denoising step.  The cases are whole layer steps from the smallest to the 32k-token prompt
(``call: layer``), the four parts of the batched, ragged workload on their own (``score``, ``evict``, ``denoise``),
the first step of a program that takes the row normalisers from its own un-evicted attention (``first``), and the two
streaming reductions over hidden states and values (``importance``, ``shift``).  Shapes are those of synth.CONFIGS and
of bench.py, next to odd lengths, grouped-query heads and head_dim 64.

A case: ``call``, ``dtype``, ``B`` sequences of ``H`` key/value heads with ``g`` query heads each, head_dim ``d``, ``n``
response (mask) tokens, prompts of ``P_lo`` .. ``P_hi`` tokens (spread evenly over the logarithm), per-head budgets of
``keep_lo`` .. ``keep_hi`` rows (likewise), pooling ``window`` and ``pool``, and where the budgets come from:
``host`` (a schedule that the program knows) or ``votes`` (maskkv_head_budgets on the device, ``keep_hi`` a head on average).
``importance`` and ``shift`` have ``rows`` of ``width`` elements.
"""
import math

import torch

from paper_2510_09309_amd import binding as mk


def _attn(name, call, B, H, d, n, P_lo, P_hi, keep_lo, keep_hi, g=1, dtype="bf16", window=7, pool="mean", budgets="host"):
    return {"name": name, "call": call, "dtype": dtype, "B": B, "H": H, "g": g, "d": d, "n": n, "P_lo": P_lo, "P_hi": P_hi,
            "keep_lo": keep_lo, "keep_hi": keep_hi, "window": window, "pool": pool, "budgets": budgets}


def _rows(name, call, rows, width, dtype="bf16"):
    return {"name": name, "call": call, "dtype": dtype, "rows": rows, "width": width}


def listed():
    return [
        # the smallest call: a short fp32 prompt, four heads; nothing but latency and launches
        _attn("layer, 512 tokens, fp32", "layer", 1, 4, 64, 64, 512, 512, 32, 32, dtype="f32"),
        # an ordinary prompt through one 32-head layer
        _attn("layer, 4k prompt", "layer", 1, 32, 128, 256, 4096, 4096, 171, 341),
        # one layer of the 8k-prompt stack with on-device head budgets
        _attn("layer, 8k prompt, voted", "layer", 1, 32, 128, 256, 8192, 8192, 128, 128, budgets="votes"),
        # the configuration the benchmark quotes
        _attn("layer, 32k prompt", "layer", 1, 32, 128, 256, 32768, 32768, 171, 341),
        # two sequences of odd lengths, head_dim 64, a response span that fills no tile
        _attn("layer, odd, head_dim 64", "layer", 2, 16, 64, 201, 2999, 5003, 97, 311),
        # grouped-query heads (7 query heads per KV head), a long odd prompt
        _attn("layer, grouped queries", "layer", 1, 4, 128, 256, 30011, 30011, 171, 341, g=7),
        # the batched ragged workload: compression once (scoring, then eviction) ...
        _attn("score, ragged batch", "score", 8, 32, 128, 512, 4096, 16384, 64, 1024),
        _attn("evict, ragged batch", "evict", 8, 32, 128, 512, 4096, 16384, 64, 1024),
        # ... and one denoising step over the evicted cache, with fresh response Q, K and V
        _attn("denoise, ragged batch", "denoise", 8, 32, 128, 512, 4096, 16384, 64, 1024),
        # the un-evicted attention of the first step, whose row normalisers then serve the scoring
        _attn("first step, 32k prompt", "first", 1, 32, 128, 256, 32768, 32768, 171, 341),
        # layer importance over a 32k prompt's hidden states; the refresh criterion over a batch's response tokens
        _rows("importance, 32k rows", "importance", 33024, 4096),
        _rows("value shift, 512 rows", "shift", 512, 4096),
    ]


# The most that a drawn case may ask for: scoring work (queries x keys x heads x head_dim) of the ragged batch, the key/value
# bytes of it, and the work of the un-evicted attention.
_MOST_SCORE = 8 * 32 * 512 * 128 * 8800
_MOST_FULL = 32 * 256 * 128 * 33024


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["layer"] * 6 + ["score", "evict", "denoise", "first", "importance", "shift"])
    if call == "importance":
        return _strip(_rows("", call, _spread(rng, 400, 33024), 8 * _spread(rng, 64, 512), rng.choice(["bf16", "bf16", "f32"])))
    if call == "shift":
        return _strip(_rows("", call, _spread(rng, 64, 4096), 8 * _spread(rng, 64, 512), rng.choice(["bf16", "bf16", "f32"])))
    while True:
        small = rng.random() < 0.2           # fp32 is for short prompts and few heads
        dtype = "f32" if small and rng.random() < 0.5 else "bf16"
        B = 1 if small or rng.random() < 0.5 else rng.randint(2, 8)
        H = rng.choice([4, 8, 12] if small else [4, 8, 16, 28, 32])
        g = 1 if H > 8 else rng.choice([1, 4, 7])
        d = rng.choice([64, 128, 128])
        n = _spread(rng, 32, 128) if small else _spread(rng, 64, 512)
        P_hi = _spread(rng, 300, 2500) if small else _spread(rng, 2000, 32768)
        P_lo = P_hi if B == 1 else max(200, int(P_hi * rng.uniform(0.25, 1.0)))
        keep_hi = _spread(rng, 32, 1024)
        keep_lo = max(16, int(keep_hi * rng.uniform(0.1, 1.0)))
        c = _attn("", call, B, H, d, n, P_lo, P_hi, keep_lo, keep_hi, g, dtype, rng.choice([1, 7, 7, 7, 13]),
                  rng.choice(["mean", "mean", "mean", "max"]), rng.choice(["host", "votes"]))
        work = sum(p + n for p in _prompts(c)) * H * g * n * d * (16 if dtype == "f32" else 1)
        kv = B * H * d * (P_hi + n)
        if work <= (_MOST_FULL if call == "first" else _MOST_SCORE) and kv <= 8 * 32 * 128 * 16896:
            return _strip(c)


def _strip(c):
    return {k: v for k, v in c.items() if k != "name"}


def _log_spaced(lo, hi, count, stride):
    """`count` whole numbers spread over log(lo) .. log(hi), dealt out in an order without a trend."""
    v = [int(round(math.exp(math.log(lo) + (math.log(hi) - math.log(lo)) * (i / (count - 1) if count > 1 else 1.0)))) for i in range(count)]
    while math.gcd(stride, count) != 1:
        stride += 1
    return [v[i * stride % count] for i in range(count)]


def _prompts(c):
    return _log_spaced(c["P_lo"], c["P_hi"], c["B"], 3)


def _budgets(c):
    return _log_spaced(c["keep_lo"], c["keep_hi"], c["B"] * c["H"], 37)


def _kept(c):
    if c["budgets"] == "votes":
        return c["B"] * c["H"] * c["keep_hi"]
    P = _prompts(c)
    return sum(min(k, P[i // c["H"]]) for i, k in enumerate(_budgets(c)))


_DT = {"bf16": torch.bfloat16, "f32": torch.float32}


class _State:
    """Inputs, and the buffers and workspaces that a program keeps for a shape."""


def prepare(case, seed):
    s = _State()
    s.call = case["call"]
    dt = _DT[case["dtype"]]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def gauss(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)

    if s.call in ("importance", "shift"):
        # hidden states before and after a sub-layer / value rows of two denoising steps: each row drifts by its own amount
        n, w = case["rows"], case["width"]
        a = gauss(n, w)
        drift = 0.1 + 0.9 * torch.rand((n, 1), generator=gen, device="cuda")
        s.a, s.b = a.to(dt), (a + drift * gauss(n, w)).to(dt)
        if s.call == "importance":
            s.out = torch.zeros(1, dtype=torch.float32, device="cuda")
            s.ws = torch.empty(mk.maskkv_layer_importance_workspace_bytes(), dtype=torch.uint8, device="cuda")
        else:
            s.cos = torch.zeros(n, dtype=torch.float32, device="cuda")
            s.refresh = torch.zeros(n, dtype=torch.int32, device="cuda")
            s.count = torch.zeros(1, dtype=torch.int32, device="cuda")
        return s

    B, H, g, d, n = case["B"], case["H"], case["g"], case["d"], case["n"]
    P = _prompts(case)
    P_max = max(P)
    N = P_max + n
    code = mk.MASKKV_BF16 if case["dtype"] == "bf16" else mk.MASKKV_F32
    s.desc = mk.Desc(B=B, H=H, d=d, dtype=code, n_resp=n, P_max=P_max, prompt_len=None if B == 1 else P, q_per_kv=0 if g == 1 else g)
    s.window, s.pool = case["window"], mk.POOL_MEAN if case["pool"] == "mean" else mk.POOL_MAX
    s.votes = case["budgets"] == "votes"
    s.k_l = case["keep_hi"]
    s.cap = _kept(case)
    s.host_budgets = None if s.votes else _budgets(case)
    s.budgets = (torch.zeros(B * H, dtype=torch.int32, device="cuda") if s.votes else
                 torch.tensor(s.host_budgets, dtype=torch.int32, device="cuda"))
    s.stride = (P_max + 63) // 64 * 64

    def buf(*shape, dtype=torch.float32):
        return torch.zeros(shape, dtype=dtype, device="cuda")

    def room(nbytes):
        return torch.empty(max(nbytes, 256), dtype=torch.uint8, device="cuda")

    # Attention logits with a row's own part (standard deviation about 1) and a part that all mask queries share, along one
    # direction per head: a key's share of the votes is then heavy-tailed, and 2 % of the prompt stands out further.
    u = gauss(B, H, 1, d)
    u = u / u.norm(dim=3, keepdim=True)
    own = math.sqrt(11.3)
    if s.call != "evict":
        q = gauss(B, H, g * n, d) * (own / d ** 0.25) + d ** 0.5 * u
        s.Q = q.view(B, H * g, n, d).to(dt)
    if s.call == "denoise":
        s.cu = torch.tensor([0] + [min(k, P[i // H]) for i, k in enumerate(_budgets(case))], device="cuda").cumsum(0).to(torch.int32)
        s.cap = int(s.cu[-1].item())
        s.Kc = (gauss(s.cap, d) * (own / d ** 0.25)).to(dt)
        s.Vc = gauss(s.cap, d).to(dt)
        s.Kr, s.Vr = (gauss(B, H, n, d) * (own / d ** 0.25)).to(dt), gauss(B, H, n, d).to(dt)
    else:
        k = gauss(B, H, N, d).mul_(own / d ** 0.25)
        stand_out = (torch.rand((B, H, N, 1), generator=gen, device="cuda") < 0.02).float() * 2.5
        k.addcmul_(gauss(B, H, N, 1).add_(stand_out), u)
        s.K = k.to(dt)
        del k
        if s.call != "score":
            s.V = gauss(B, H, N, d).to(dt)

    if s.call in ("layer", "score", "first"):
        s.scores, s.mass = buf(B * H, s.stride), buf(B * H)
        s.ws_score = room(mk.maskkv_score_workspace_bytes(s.desc))
    if s.call == "evict":     # votes as scoring leaves them: heavy-tailed, 2 % of the positions standing out
        hot = (torch.rand((B * H, s.stride), generator=gen, device="cuda") < 0.02).float() * 2.5
        s.scores = torch.exp(gauss(B * H, s.stride) + hot) * (n / N)
        s.mass = (s.scores.sum(1) / s.scores.sum(1).max()) * (0.9 * g * n)
    if s.call in ("layer", "evict"):
        s.idx, s.cu = buf(s.cap, dtype=torch.int32), buf(B * H + 1, dtype=torch.int32)
        s.Kc, s.Vc = buf(s.cap, d, dtype=dt), buf(s.cap, d, dtype=dt)
        s.ws_select = room(mk.maskkv_select_workspace_bytes(s.desc))
    if s.call in ("layer", "denoise"):
        s.ws_attend = room(mk.maskkv_attend_workspace_bytes(s.desc, False))
    if s.call == "layer":     # the response rows of the same K and V, behind each sequence's prompt
        s.Kr, s.Vr = mk.tensor_view(s.K, seq_start=P), mk.tensor_view(s.V, seq_start=P)
    if s.call == "first":
        s.ws_full = room(mk.maskkv_attend_workspace_bytes(s.desc, True))
        s.lse = buf(B * H * g * n)
    if s.call in ("layer", "denoise", "first"):
        s.O = buf(B, H * g, n, d, dtype=dt)
    return s


def _evict(s):
    if s.votes:
        mk.maskkv_head_budgets(s.desc, s.mass, s.k_l, 0.1, s.budgets)
    mk.maskkv_select(s.desc, s.scores, s.stride, s.window, s.pool, s.budgets, s.idx, s.cu, s.cap, s.ws_select,
                     budgets_host=s.host_budgets)
    mk.maskkv_compact(s.desc, s.K, s.V, s.idx, s.cu, s.cap, s.Kc, s.Vc)


def run(s):
    if s.call == "importance":
        mk.maskkv_layer_importance(s.a, s.b, s.out, s.ws)
        return {"importance": s.out}
    if s.call == "shift":
        mk.maskkv_value_shift(s.a, s.b, 0.8, s.cos, s.refresh, s.count)
        return {"cos": s.cos, "refresh": s.refresh, "count": s.count}
    if s.call == "score":
        mk.maskkv_score(s.desc, s.Q, s.K, 0.0, s.scores, s.stride, s.mass, s.ws_score)
        return {"scores": s.scores, "mass": s.mass}
    if s.call == "first":
        mk.maskkv_attend_full(s.desc, s.Q, s.K, s.V, 0.0, s.O, s.lse, s.ws_full)
        mk.maskkv_score_given_lse(s.desc, s.Q, s.K, 0.0, s.lse, s.scores, s.stride, s.mass, s.ws_score)
        return {"O": s.O, "lse": s.lse, "scores": s.scores, "mass": s.mass}
    if s.call == "evict":
        _evict(s)
        return {"idx": s.idx, "cu": s.cu, "Kc": s.Kc, "Vc": s.Vc}
    if s.call == "layer":
        mk.maskkv_score(s.desc, s.Q, s.K, 0.0, s.scores, s.stride, s.mass, s.ws_score)
        _evict(s)
    mk.maskkv_attend(s.desc, s.Q, s.Kc, s.Vc, s.cu, s.cap, s.Kr, s.Vr, 0.0, s.O, None, s.ws_attend)
    if s.call == "denoise":
        return {"O": s.O}
    # (the packed rows are what O is formed from, and come back as they are from the `evict` cases)
    return {"scores": s.scores, "mass": s.mass, "idx": s.idx, "cu": s.cu, "O": s.O}


def work(case):
    eb = 2 if case["dtype"] == "bf16" else 4
    if case["call"] in ("importance", "shift"):
        n, w = case["rows"], case["width"]
        return {"bytes": 2 * n * w * eb + (4 if case["call"] == "importance" else 8 * n), "flops": 6 * n * w}
    B, H, g, d, n = case["B"], case["H"], case["g"], case["d"], case["n"]
    P = _prompts(case)
    keys = H * sum(p + n for p in P)         # rows of K
    prompt = H * sum(P)                      # scores
    kept = _kept(case)
    rows = B * H * g * n                     # query rows
    logits = g * n * keys
    evict = 4 * prompt + 4 * kept + 4 * kept * d * eb      # scores in, positions out, K and V rows in and out
    call = case["call"]
    if call == "score":
        return {"bytes": (rows + keys) * d * eb + 4 * prompt, "flops": 2 * logits * d}
    if call == "evict":
        return {"bytes": evict, "flops": 0}
    if call == "first":
        return {"bytes": (2 * rows + 2 * keys) * d * eb + 4 * rows + 4 * prompt, "flops": 6 * logits * d}
    attend = {"bytes": (2 * rows + 2 * (kept + B * H * n)) * d * eb, "flops": 4 * g * n * (kept + B * H * n) * d}
    if call == "denoise":
        return attend
    # a layer step: K once, Q once, the scores, the kept rows of K and V in and out, the response rows of V, the output
    return {"bytes": (rows + keys) * d * eb + 4 * prompt + 4 * kept + 4 * kept * d * eb + (rows + B * H * n) * d * eb,
            "flops": 2 * logits * d + attend["flops"]}


def tolerance(case):
    call = case["call"]
    if call == "evict":
        return "exact"
    if call == "score":                      # fp32 sums of products of the rounded inputs
        return {"rel": 1e-5}
    if call == "importance":                 # one minus a mean of cosines near one
        return {"rel": 2e-5}
    if call == "shift":                      # a cosine within an ulp of the threshold may fall on either side
        return {"rel": 1e-5, "differ": 0.01}
    if case["dtype"] == "f32":
        return {"rel": 2e-5, "differ": 0.01}
    # attention outputs in bf16; two pooled scores within the rounding of fp32 may swap places
    return {"rel": 1e-2, "differ": 0.01}
