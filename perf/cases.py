"""Workloads by which this framework's speed is judged.

A pipeline stage's user does two kinds of things with it, and each is a family of cases here:

  window   one or two accumulation windows of the stage's AMDP schedule through the stage object: every
           forward, backward, accumulation and update in the order `amdp_schedule_generate` gives, each
           with its weight version. What leaves the GPU's stage in such a window comes back: the
           activations Y for the next stage, the gradients dX for the previous one, the gradient sum
           before each update (what a replica sends to the owner of the parameters) and the published
           weights after the last one (what the owner sends back).
  rows     the row operators that are entry points of their own: LayerNorm forward, LayerNorm backward
           with a residual, and the parameter gradients of both (column sums in the LayerNorm and the
           bias form).

Sizes are the repository's stage workloads or, for the odd ones, generic.
"""
import math

import torch

import paper_2605_29664_amd as amdp

DEV = "cuda:0"


#: What every window case has, the fields that a case does not name: the ordinary middle stage of a 24-layer GPT
#: at pipeline depth 6, eight minibatches of 4 x 1024 tokens to an update.
_WINDOW = dict(family="window", block=amdp.BLOCK_GPT, layers=4, d_model=1024, heads=16, d_ffn=4096, seq=1024, microbatch=4, dtype=amdp.BF16,
               lm_head=False, embedding=False, vocab=0, depth=6, pipelines=3, stage=3, stash=1, threshold=8, windows=1, fused_accumulate=False)


def _window(name, **other):
    return dict(_WINDOW, name=name, **other)


def listed():
    return [
        # Bring-up and precision runs: the small fp32 stage, two windows so that minibatches are in flight
        # across the first update. Nothing fills the GPU; launches and latency count.
        _window("gpt_d128_fp32", layers=1, d_model=128, heads=4, d_ffn=512, seq=64, microbatch=2, dtype=amdp.FP32,
                depth=4, pipelines=2, stage=1, threshold=4, windows=2),
        # A small bf16 stage whose width, sequence and FFN are no multiples of any tile.
        _window("gpt_d192_odd", layers=2, d_model=192, heads=3, d_ffn=448, seq=200, microbatch=2, stage=2, threshold=6, windows=2),
        # The ordinary middle stage.
        _window("gpt_d1024"),
        # The bidirectional stage with per-sequence padding.
        _window("bert_d1024_padded", block=amdp.BLOCK_BERT, layers=6, seq=512, microbatch=8, depth=4, pipelines=2, stage=1),
        # The last stage: tied vocabulary projection with an odd vocabulary, and cross-entropy.
        _window("gpt_d2048_lm_head", d_model=2048, heads=32, d_ffn=8192, seq=2048, microbatch=2, lm_head=True, vocab=50257, depth=8, stage=7),
        # The large stage, 0.8 G parameters: the benchmark's headline workload.
        _window("gpt_d4096", d_model=4096, heads=32, d_ffn=16384, seq=2048, microbatch=1, depth=16, pipelines=4, stage=8, stash=3,
                threshold=16),
        # The paper's own widths: hidden 1600, 25 heads of 64 (GPT) with the accumulation fused into backward,
        # and 32 heads of 50 (BERT).
        _window("gpt_h1600_fused", layers=6, d_model=1600, heads=25, d_ffn=6400, depth=8, pipelines=4, stage=4, fused_accumulate=True),
        _window("bert_h1600", block=amdp.BLOCK_BERT, layers=6, d_model=1600, heads=32, d_ffn=6400, depth=8, pipelines=4, stage=4),
        # The first stage of the ordinary GPT: token and position embedding.
        _window("gpt_d1024_embedding", embedding=True, vocab=50257, stage=0),
        # Sequences cut to a round decimal length: 3 x 1000 tokens, no multiple of 64.
        _window("gpt_d768_s1000", layers=2, d_model=768, heads=12, d_ffn=3072, seq=1000, microbatch=3, threshold=4),
        # The row operators at the large stage's activations, and on a small odd fp32 matrix.
        dict(name="rows_bf16_2048x4096", family="rows", rows=2048, cols=4096, dtype=amdp.BF16),
        dict(name="rows_fp32_333x1000", family="rows", rows=333, cols=1000, dtype=amdp.FP32),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    if rng.random() < 0.25:
        dtype = amdp.BF16 if rng.random() < 0.7 else amdp.FP32
        vec = 8 if dtype == amdp.BF16 else 4
        return dict(family="rows", rows=_log_int(rng, 1, 20000), cols=max(1, _log_int(rng, 64, 12000) // vec) * vec, dtype=dtype)
    while True:
        dtype = amdp.BF16 if rng.random() < 0.85 else amdp.FP32
        head = rng.choice([64, 64, 64, 128, 128, 32, 50, 80, 96]) if dtype == amdp.BF16 else rng.choice([16, 32, 64])
        heads = max(1, _log_int(rng, 128, 4096 if dtype == amdp.BF16 else 512) // head)
        d = head * heads
        if d % 8:
            heads *= 4
            d = head * heads
        odd = rng.random() < 0.35
        seq = _log_int(rng, 64, 2048)
        seq = max(8, seq // 8 * 8) if odd else max(128, seq // 128 * 128)
        kind = rng.choice(["gpt", "gpt", "gpt", "bert", "bert", "lm", "first"])
        depth = rng.choice([4, 6, 8])
        case = dict(family="window", block=amdp.BLOCK_BERT if kind == "bert" else amdp.BLOCK_GPT,
                    layers=rng.randint(1, 4), d_model=d, heads=heads, d_ffn=4 * d if not odd else max(8, int(rng.uniform(2, 4.5) * d) // 8 * 8),
                    seq=seq, microbatch=rng.randint(1, 6), dtype=dtype, lm_head=kind == "lm", embedding=kind == "first",
                    vocab=_log_int(rng, 500, 50257) if kind in ("lm", "first") else 0, depth=depth, pipelines=rng.randint(1, depth // 2),
                    stage={"lm": depth - 1, "first": 0}.get(kind, depth // 2), stash=1, threshold=rng.choice([2, 4, 8]), windows=1,
                    fused_accumulate=rng.random() < 0.3)
        # at most the work of the largest listed case; less where nothing can be tiled evenly or in fp32
        if work(case)["flops"] <= (3e13 if dtype == amdp.BF16 and not odd else 1e12 if dtype == amdp.BF16 else 2e11):
            return case


def _randn(g, shape, dtype, std=1.0):
    return (torch.randn(shape, generator=g, device=DEV, dtype=torch.float32) * std).to(dtype)


def _torch_dtype(case):
    return torch.bfloat16 if case["dtype"] == amdp.BF16 else torch.float32


def _prepare_rows(case, g):
    dt, n, c = _torch_dtype(case), case["rows"], case["cols"]
    ws = [torch.empty(amdp.amdp_column_sums_workspace_bytes(n, c, case["dtype"], ln), dtype=torch.uint8, device=DEV) for ln in (True, False)]
    return dict(x=_randn(g, (n, c), dt), dy=_randn(g, (n, c), dt, 1e-3), res=_randn(g, (n, c), dt, 1e-3),
                gamma=(1 + _randn(g, (c,), torch.float32, 0.02)).to(dt), beta=_randn(g, (c,), dt, 0.02),
                y=torch.empty((n, c), dtype=dt, device=DEV), dx=torch.empty((n, c), dtype=dt, device=DEV),
                stats=torch.empty((n, 2), dtype=torch.float32, device=DEV), ws=ws,
                ln_grad=torch.empty(2 * c, dtype=torch.float32, device=DEV), bias_grad=torch.empty(c, dtype=torch.float32, device=DEV))


def _run_rows(s):
    amdp.amdp_layernorm_forward(s["x"], s["gamma"], s["beta"], s["y"], s["stats"], 1e-5)
    amdp.amdp_layernorm_backward(s["dy"], s["x"], s["stats"], s["gamma"], s["res"], s["dx"])
    amdp.amdp_column_sums(s["dy"], s["x"], s["stats"], s["ln_grad"], s["ws"][0])
    amdp.amdp_column_sums(s["dy"], None, None, s["bias_grad"], s["ws"][1])
    return [s["y"], s["stats"], s["dx"], s["ln_grad"], s["bias_grad"]]


def _prepare_window(case, g):
    dt, n, d, T = _torch_dtype(case), case["seq"] * case["microbatch"], case["d_model"], case["threshold"]
    M = T * case["windows"]
    slots = min(2, case["depth"] - case["stage"]) * case["pipelines"]
    cfg = amdp.make_config(case["block"], case["layers"], d, case["heads"], case["d_ffn"], case["seq"], case["microbatch"], case["dtype"],
                           has_lm_head=case["lm_head"], vocab=case["vocab"], act_slots=slots, stash_slots=case["stash"],
                           has_embedding=case["embedding"])
    stage = amdp.Stage(cfg, device=DEV)
    theta = _randn(g, (stage.n_params,), torch.float32, 0.02)
    for name, off, r, c in amdp.amdp_stage_param_layout(cfg):
        if name.endswith("gamma"):
            theta[off:off + r * c] += 1.0
    stage.amdp_stage_set_state(theta)
    del theta
    if case["fused_accumulate"]:
        stage.amdp_stage_set_fused_accumulate(True)
    events = [(e.kind, e.mb, e.version) for e in
              amdp.amdp_schedule_generate(case["depth"], case["pipelines"], case["stage"], T, M)]

    def ints(lo, hi, k):
        return torch.randint(lo, hi, (k,), generator=g, device=DEV, dtype=torch.int32)

    aux = []
    for _ in range(M):
        a = [ints(0, case["vocab"], n)] if case["lm_head"] or case["embedding"] else []
        if case["block"] == amdp.BLOCK_BERT:
            a.append(ints(max(1, case["seq"] // 4), case["seq"] + 1, case["microbatch"]))
        aux.append(torch.cat(a) if a else None)
    new = lambda shape, t=dt: torch.empty(shape, dtype=t, device=DEV)  # noqa: E731
    return dict(stage=stage, events=events, version=0, scale=1.0 / T, aux=aux,
                x=[None if case["embedding"] else _randn(g, (n, d), dt) for _ in range(M)],
                dy=[None if case["lm_head"] else _randn(g, (n, d), dt, 1e-3) for _ in range(M)],
                y=[new((1,), torch.float32) if case["lm_head"] else new((n, d)) for _ in range(M)],
                dx=[None if case["embedding"] else new((n, d)) for _ in range(M)],
                grad_sum=[new((stage.n_params,), torch.float32) for _ in range(case["windows"])],
                # room for a whole number of 32-bit words
                weights=torch.zeros(stage.n_params + stage.n_params % 2, dtype=dt, device=DEV))


def _run_window(s):
    stage, base, updates = s["stage"], s["version"], 0
    for kind, mb, version in s["events"]:
        if kind == amdp.EV_F:
            stage.amdp_stage_forward(mb, base + version, s["x"][mb], s["aux"][mb], s["y"][mb])
        elif kind == amdp.EV_B:
            stage.amdp_stage_backward(mb, base + version, s["dy"][mb], s["dx"][mb])
        elif kind == amdp.EV_A:
            stage.amdp_grad_accumulate(mb)
        else:
            stage.amdp_stage_get_state(G=s["grad_sum"][updates])
            s["version"] = stage.amdp_apply_update(1e-4, grad_scale=s["scale"])
            updates += 1
    stage.amdp_stage_read_version(s["version"], s["weights"])
    return dict(y=s["y"], dx=s["dx"], grad_sum=s["grad_sum"], weights=s["weights"])


def prepare(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    state = _prepare_rows(case, g) if case["family"] == "rows" else _prepare_window(case, g)
    state["family"] = case["family"]
    return state


def run(state):
    return _run_rows(state) if state["family"] == "rows" else _run_window(state)


def _n_params(case):
    d, f = case["d_model"], case["d_ffn"]
    return (case["layers"] * (4 * d * d + 2 * d * f + 9 * d + f) + (case["vocab"] * d if case["vocab"] else 0)
            + (2 * d if case["lm_head"] else 0) + (case["seq"] * d if case["embedding"] else 0))


def work(case):
    e = 2 if case["dtype"] == amdp.BF16 else 4
    if case["family"] == "rows":
        n, c = case["rows"], case["cols"]
        # x, dy, res read once, y and dx written once; both gains' sums, the statistics and the parameters
        return dict(bytes=5 * n * c * e + 8 * n + 12 * c + 2 * c * e, flops=0)
    n, d, f, s = case["seq"] * case["microbatch"], case["d_model"], case["d_ffn"], case["seq"]
    M, p = case["threshold"] * case["windows"], _n_params(case)
    pairs = case["microbatch"] * s * ((s + 1) / 2 if case["block"] == amdp.BLOCK_GPT else s)
    # linear maps: one product forward, two backward; attention: two forward, four backward; the vocabulary projection like a linear map
    flops = M * (case["layers"] * (6 * n * (4 * d * d + 2 * d * f) + 12 * pairs * d) + (6 * n * d * case["vocab"] if case["lm_head"] else 0))
    # per minibatch: X, dY in, Y, dX out and one weight version; per window: G out, theta, m, v in and out, the version out
    act = (0 if case["embedding"] else 2 * n * d * e) + (4 * n if case["lm_head"] else 2 * n * d * e)
    return dict(bytes=M * (act + p * e) + case["windows"] * p * (4 + 24 + e), flops=flops)


def tolerance(case):
    # Measured between the default kernels and the same path with other tiles, the contractions summed the other
    # way round and the attention with its scores in memory: bf16 stages, whose activations and saved tensors are
    # rounded to 8 bits at every layer, up to 1.2e-2 in norm and 0.3 for one value; fp32 stages up to 1.1e-6. The
    # gradient of the key bias is zero up to rounding, so Adam moves that bias by up to lr = 1e-4 either way at an
    # update: 1e-2 of the weights' root mean square for one value.
    if case["family"] == "rows":
        return {"rel": 5e-3} if case["dtype"] == amdp.BF16 else {"rel": 1e-5}
    return {"rel": 3e-2, "max": 1.0} if case["dtype"] == amdp.BF16 else {"rel": 1e-5, "max": 2e-2}
