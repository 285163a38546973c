"""GPU parity tests: the HIP library, called through its C ABI, against the CPU
oracle on identical seeded inputs. Tolerances per compared tensor: norm-wise
relative error 2e-2 for bf16 stages, 1e-5 for fp32 stages, and an element-wise
bound on the largest deviation (tests/parity.py)."""
import numpy as np
import pytest

import workloads as W
from oracle import schedule as OSched
from tests.parity import run_parity, worst_entries, GpuStage, rel_err, TOL
from paper_2605_29664_amd.binding import (OPT_GEMM_TILE, OPT_GEMM_TRANSPOSING_READS, OPT_GEMM_DIRECT_TO_LDS,
                                          OPT_LAZY_JOIN, OPT_SPLIT_K_MIN_TOKENS, OPT_SPLIT_MAIN_MIN_K, OPT_LEAF_FORKS, ATTN_UNFUSED)

pytestmark = pytest.mark.gpu


def _report(name, rep):
    print(f"\n[{name}] ok={rep['ok']} worst={rep['worst']:.3e} tol={rep['tol']:.0e} elem={rep['worst_elem']:.3e} "
          f"elem_tol={rep['elem_tol']:.0e} events={rep['events']} "
          f"sched={rep['schedule_equal']} resid={rep['residency_equal']} {rep['seconds']:.1f}s", flush=True)
    we = worst_entries(rep, 4)
    for d in we["norm"] + we["elem"]:
        print("    ", d, flush=True)


# ---- small fp32 stages: every op, ragged shapes ------------------------------
@pytest.mark.parametrize("key", ["gpt", "bert", "lmhead"])
@pytest.mark.parametrize("policy", [OSched.STASHED, OSched.CURRENT])
def test_tiny_fp32(key, policy):
    rep = run_parity(W.TINY[key], n_windows=2, policy=policy, verbose=False)
    _report(f"tiny_{key}_p{policy}", rep)
    assert rep["ok"], worst_entries(rep)


def test_config1_fp32_full_schedule():
    rep = run_parity(W.CONFIGS[1], n_windows=3, verbose=False)
    _report("cfg1", rep)
    assert rep["ok"], worst_entries(rep)


def test_config1_eager_and_current():
    rep = run_parity(W.CONFIGS[1], n_windows=2, policy=OSched.CURRENT, placement=OSched.EAGER, verbose=False)
    _report("cfg1_eager_current", rep)
    assert rep["ok"], worst_entries(rep)


# ---- bf16, shapes that are not tile multiples: ragged last tiles -------------
@pytest.mark.parametrize("key", ["gpt_mid", "bert_mid", "lmhead_mid"])
def test_mid_bf16_ragged(key):
    rep = run_parity(W.TINY[key], n_windows=1, verbose=False)
    _report(key, rep)
    assert rep["ok"], worst_entries(rep)


# ---- bf16, tile-aligned shapes: the MFMA kernels ----------------------------
@pytest.mark.parametrize("key", ["gpt_tile", "bert_tile", "lmhead_tile"])
@pytest.mark.parametrize("tr", [1, 0])
def test_tile_bf16_mfma(key, tr):
    """tr 1: the library's choice; 0: every product on the register-staged kernel (attention with its scores in
    memory, so that its batched and banded products run there too) reading LDS element by element."""
    rep = run_parity(W.TINY[key], n_windows=1, verbose=False,
                     **({} if tr else dict(options={OPT_GEMM_TRANSPOSING_READS: 0, OPT_GEMM_DIRECT_TO_LDS: 0},
                                           cfg_kw=dict(attention=ATTN_UNFUSED))))
    _report(f"{key}_tr{tr}", rep)
    assert rep["ok"], worst_entries(rep)


@pytest.mark.parametrize("key", ["gpt_tile", "bert_tile", "lmhead_tile", "gpt_tile128"])
def test_tile_bf16_current_weights_in_backward(key):
    """The mismatched backward of Section 3.1 on the matrix-core kernels: two
    windows, so that the minibatches in flight across an update run their
    backward with the version published after their forward."""
    w = W.TINY[key].with_(lr=1e-3)
    rep = run_parity(w, n_windows=2, policy=OSched.CURRENT, verbose=False)
    _report(f"{key}_current", rep)
    assert rep["ok"], worst_entries(rep)
    mism = [d for d in rep["details"] if d[1] == "dX"]
    assert len(mism) >= 2 * w.threshold


@pytest.mark.parametrize("key", ["gpt_tile128", "bert_tile128"])
def test_tile_bf16_head_dim_128(key):
    rep = run_parity(W.TINY[key], n_windows=1, verbose=False)
    _report(key, rep)
    assert rep["ok"], worst_entries(rep)


@pytest.mark.parametrize("direct,tr", [(1, 1), (0, 1), (0, 0)])
@pytest.mark.parametrize("tile", [256, 128, 128064, 64128, 64])
def test_tile_bf16_forced_tile(tile, direct, tr):
    """Every matrix-core tile shape on the same workload: the plain products loading their tiles straight into LDS
    (1; the rectangular tiles are the register-staged kernel's either way) and through the register-staged kernel
    (0; a tile that does not divide a product's shape leaves that product to the default choice), with and without
    the transposing LDS read."""
    rep = run_parity(W.TINY["gpt_tile"], n_windows=1, verbose=False,
                     options={OPT_GEMM_TILE: tile, OPT_GEMM_DIRECT_TO_LDS: direct, OPT_GEMM_TRANSPOSING_READS: tr})
    _report(f"gpt_tile_forced_{tile}", rep)
    assert rep["ok"], worst_entries(rep)


@pytest.mark.parametrize("key", ["gpt_tile_edge", "gpt_tile64"])
@pytest.mark.parametrize("tile", [256, 128])
def test_tile_bf16_ragged_last_tile(key, tile):
    """Widths and token counts that are multiples of 64 but not of the tile: the
    last tile of a row or column of tiles has 64, 128 or 192 of its 256 rows
    (64 of 128), its missing rows are neither loaded from outside the matrix
    nor stored."""
    rep = run_parity(W.TINY[key], n_windows=1, verbose=False, options={OPT_GEMM_TILE: tile})
    _report(f"{key}_ragged_{tile}", rep)
    assert rep["ok"], worst_entries(rep)


@pytest.mark.parametrize("key", ["gpt_tile", "bert_tile"])
def test_weight_gradients_split_over_tokens(key):
    """Weight-gradient products too small to fill the GPU are split over their
    tokens into parts that are added in fixed order. At the tile test shapes
    that needs the part size set to 64 tokens: the 256x256
    product then runs in four parts, the wider ones in two. Checked against the
    oracle, run to run, and with the accumulation fused into the second stage."""
    import torch
    w = W.TINY[key]
    rep = run_parity(w, n_windows=1, verbose=False, options={OPT_SPLIT_K_MIN_TOKENS: 64})
    _report(f"{key}_split_k", rep)
    assert rep["ok"], worst_entries(rep)
    from oracle.stage import Stage as OStage
    theta0 = W.make_theta(w, OStage.from_workload(w).layout)
    aux = W.make_aux(w, 0)
    sums = []
    for fused, split in ((False, 64), (False, 64), (True, 64), (False, 1 << 20)):
        gpu = GpuStage(w, act_slots=2, stash_slots=1, options={OPT_SPLIT_K_MIN_TOKENS: split})
        gpu.set_state(theta0)
        gpu.stage.amdp_stage_set_fused_accumulate(fused)
        x, dy = gpu.to_dev(W.make_x(w, 0), gpu.dt), gpu.to_dev(W.make_dy(w, 0), gpu.dt)
        a = None if aux is None else gpu.to_dev(np.asarray(aux, dtype=np.int32))
        y = torch.empty_like(x)
        for mb in (0, 1):
            gpu.stage.amdp_stage_forward(mb, 0, x, a, y)
            gpu.stage.amdp_stage_backward(mb, 0, dy, None)
            gpu.stage.amdp_grad_accumulate(mb)
        sums.append(gpu.state(("G",))["G"])
        gpu.stage.close()
    assert np.array_equal(sums[0], sums[1]) and np.array_equal(sums[0], sums[2])
    assert not np.array_equal(sums[0], sums[3]), "the split path did not run"      # another summation order
    assert rel_err(sums[0], sums[3]) < 1e-5


@pytest.mark.parametrize("key", ["gpt_tile", "bert_tile", "lmhead_tile"])
def test_main_chain_products_with_split_contraction(key):
    """Products of the forward / dX chain with few 256x256 tiles and a long
    contraction run in two halves into fp32 scratch, added in order with bias and
    residual by a second kernel. At the tile test shapes that needs the minimum
    half set to 64; the profile shows that the path ran."""
    import torch
    w = W.TINY[key]
    rep = run_parity(w, n_windows=1, verbose=False, options={OPT_SPLIT_MAIN_MIN_K: 64})
    _report(f"{key}_split_main", rep)
    assert rep["ok"], worst_entries(rep)
    from oracle.stage import Stage as OStage
    gpu = GpuStage(w, act_slots=2, stash_slots=1, options={OPT_SPLIT_MAIN_MIN_K: 64})
    gpu.set_state(W.make_theta(w, OStage.from_workload(w).layout))
    gpu.stage.amdp_stage_profile_begin()
    gpu.forward(0, 0, W.make_x(w, 0), W.make_aux(w, 0))
    gpu.backward(0, 0, None if w.has_lm_head else W.make_dy(w, 0))
    prof = gpu.stage.amdp_stage_profile_end()
    split = {k: v["launches"] for k, v in prof.items() if k.endswith("_splitk")}
    assert split.get("gemm_mfma256x256_NN_splitk", 0) >= 2 * w.n_layers, prof.keys()   # QKV and out-projection at least
    assert split.get("gemm_mfma256x256_NT_splitk", 0) >= 2 * w.n_layers, prof.keys()   # dX of W_1, W_o (and W_qkv)
    assert prof["splitk_reduce"]["launches"] == sum(split.values())
    gpu.stage.close()


@pytest.mark.parametrize("key", ["gpt_tile64", "bert_dh50", "bert_tile_dh50", "gpt_tile_dh96"])
def test_bf16_multiples_of_64_and_odd_head_dims(key):
    rep = run_parity(W.TINY[key], n_windows=1, verbose=False)
    _report(key, rep)
    assert rep["ok"], worst_entries(rep)


@pytest.mark.parametrize("key", ["bert_tile", "bert_mid"])
def test_padding_mask_extremes(key):
    """Valid lengths at the ends of their range and on key-block boundaries:
    one visible key, a whole sequence, exactly one block of 64, one past it."""
    w = W.TINY[key]
    pool = [1, w.seq_len, 64, 65, 2, w.seq_len - 1, 128, 63]
    def aux(w_, mb):
        return np.array([min(pool[(mb * w_.microbatch + i) % len(pool)], w_.seq_len) for i in range(w_.microbatch)],
                        dtype=np.int32)
    rep = run_parity(w, n_windows=1, verbose=False, aux_fn=aux)
    _report(f"{key}_mask_extremes", rep)
    assert rep["ok"], worst_entries(rep)


@pytest.mark.parametrize("d,P,i,T,M", [(1, 1, 0, 1, 3), (2, 1, 1, 1, 1), (4, 2, 3, 3, 7), (6, 3, 0, 4, 10)])
def test_degenerate_schedules(d, P, i, T, M):
    """One stage / one pipeline, an update after every minibatch, a single
    minibatch, a last partial window."""
    w = W.TINY["gpt_tile"].with_(depth=d, pipelines=P, stage=i, threshold=T, n_layers=1)
    rep = run_parity(w, n_minibatches=M, verbose=False)
    _report(f"degenerate_d{d}P{P}i{i}T{T}M{M}", rep)
    assert rep["ok"] and rep["events"] == 3 * M + -(-M // T), worst_entries(rep)


def test_tile_bf16_generic_kernels_agree():
    rep = run_parity(W.TINY["gpt_tile"], n_windows=1, verbose=False, options={OPT_GEMM_TILE: -1})
    _report("gpt_tile_generic", rep)
    assert rep["ok"], worst_entries(rep)


def test_three_stashed_versions():
    """Stress list for the stash: injection limit 3 and short windows keep three
    older versions resident next to the current one; each backward must read
    the version its forward used."""
    w = W.TINY["gpt_tile"].with_(depth=16, pipelines=4, stage=8, threshold=4, stash_slots=3, lr=1e-3)
    rep = run_parity(w, inject_limit=3, n_minibatches=40, verbose=False)
    _report("stash3", rep)
    assert rep["ok"], worst_entries(rep)


def test_zero_lr_versions_bit_identical():
    """With lr = 0 every version holds the same numbers, so stashed and current
    backward must produce bit-identical results."""
    w = W.TINY["gpt_tile"].with_(lr=0.0)
    outs = []
    for policy in (OSched.STASHED, OSched.CURRENT):
        gpu = GpuStage(w, act_slots=w.act_slots, stash_slots=2)
        from oracle.stage import Stage as OStage
        theta0 = W.make_theta(w, OStage.from_workload(w).layout)
        gpu.set_state(theta0)
        import paper_2605_29664_amd as amdp
        ev = amdp.amdp_schedule_generate(w.depth, w.pipelines, w.stage, w.threshold, 2 * w.threshold, 2, 0, policy)
        log = []
        for e in ev:
            if e.kind == amdp.EV_F:
                log.append(gpu.forward(e.mb, e.version, W.make_x(w, e.mb), None))
            elif e.kind == amdp.EV_B:
                dx, g = gpu.backward(e.mb, e.version, W.make_dy(w, e.mb))
                log += [dx, g]
            elif e.kind == amdp.EV_A:
                gpu.accumulate(e.mb)
            else:
                gpu.update(w, 1.0 / w.threshold)
        outs.append(log)
        gpu.stage.close()
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


# heads whose width no fused kernel takes: odd (rows at odd multiples of 2 bytes), wider than 128
@pytest.mark.parametrize("key", ["gpt_mid", "bert_mid"])
@pytest.mark.parametrize("heads,width", [(8, 25), (8, 3), (2, 136)])
def test_bf16_attention_with_scores_in_memory(key, heads, width):
    import paper_2605_29664_amd as amdp
    w = W.TINY[key].with_(n_layers=1, d_model=heads * width, n_heads=heads, d_ffn=2 * heads * width)
    auto, unfused = (amdp.amdp_stage_workspace_bytes(amdp.make_config(**W.stage_config_args(w, attention=a)))
                     for a in (0, ATTN_UNFUSED))
    assert auto == unfused                           # the probabilities are kept, as in the form that asks for it
    rep = run_parity(w, n_windows=1, verbose=False)
    _report(f"{key}_{heads}x{width}", rep)
    assert rep["ok"], worst_entries(rep)


@pytest.mark.parametrize("key", ["gpt_tile", "bert_tile", "gpt_mid", "bert_mid", "bert_dh50"])
def test_unfused_attention_fallback(key):
    """The configuration can ask for the three-kernel attention (scores, softmax
    and probabilities in HBM); it must meet the same tolerance as the fused one.
    Tile-aligned stages run its products on the matrix cores, the others on the
    generic kernel."""
    rep = run_parity(W.TINY[key], n_windows=1, verbose=False, cfg_kw=dict(attention=ATTN_UNFUSED))
    _report(f"{key}_unfused_attention", rep)
    assert rep["ok"], worst_entries(rep)


def test_side_stream_on_off_bit_identical():
    """A whole schedule enqueued back to back with no read in between (so the
    gradient leaves and the accumulations really run beside the main chain)
    must end in exactly the state the single-stream order produces. The 12
    activation slots are the schedule's in-flight bound (inject limit 3, four
    pipelines), so every forward reuses the slot that was freed last, whose
    backward's gradient leaves may still be running."""
    import paper_2605_29664_amd as amdp
    from oracle.stage import Stage as OStage
    w = W.TINY["gpt_tile"].with_(depth=16, pipelines=4, stage=8, threshold=4, stash_slots=3, lr=1e-3)
    theta0 = W.make_theta(w, OStage.from_workload(w).layout)
    ev = amdp.amdp_schedule_generate(w.depth, w.pipelines, w.stage, w.threshold, 24, 3, amdp.U_NEXT_BUBBLE,
                                     amdp.BWD_STASHED)
    import torch
    xs = {m: torch.from_numpy(W.make_x(w, m)).to("cuda:0").to(torch.bfloat16) for m in range(24)}
    dys = {m: torch.from_numpy(W.make_dy(w, m)).to("cuda:0").to(torch.bfloat16) for m in range(24)}
    finals = []
    # lazy 0: every backward ends by joining its leaves; forks: hand-overs to the side stream per layer
    # (0 = one per product)
    for overlap, lazy, forks in ((True, 1, 0), (True, 0, 0), (False, 1, 0), (True, 1, 1), (True, 1, 2)):
        gpu = GpuStage(w, act_slots=12, stash_slots=3, options={OPT_LAZY_JOIN: lazy, OPT_LEAF_FORKS: forks})
        gpu.set_state(theta0)
        gpu.stage.amdp_stage_set_overlap(overlap)           # small stage: off by default
        assert gpu.stage.amdp_stage_get_overlap() == overlap
        y = torch.empty((w.tokens, w.d_model), dtype=torch.bfloat16, device="cuda:0")
        dx = torch.empty_like(y)
        for e in ev:
            if e.kind == amdp.EV_F:
                gpu.stage.amdp_stage_forward(e.mb, e.version, xs[e.mb], None, y)
            elif e.kind == amdp.EV_B:
                gpu.stage.amdp_stage_backward(e.mb, e.version, dys[e.mb], dx)
            elif e.kind == amdp.EV_A:
                gpu.stage.amdp_grad_accumulate(e.mb)
            else:
                gpu.stage.amdp_apply_update(w.lr, w.beta1, w.beta2, w.eps, w.weight_decay, 1.0 / w.threshold, True)
        s = gpu.state()
        torch.cuda.synchronize()
        finals.append((s["theta"], s["m"], s["v"], s["G"], dx.float().cpu().numpy(), y.float().cpu().numpy()))
        gpu.stage.close()
    assert np.any(finals[0][0] != theta0)
    for other in finals[1:]:
        for a, b in zip(finals[0], other):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("vocab", [5000, 17000])
def test_lm_head_wide_vocabulary(vocab):
    """Rows of logits many vectors long per lane (the cross-entropy kernel's
    running maximum and rescaled sum), a last vector round that is not full,
    padding columns behind the vocabulary."""
    w = W.TINY["lmhead_tile"].with_(vocab=vocab, n_layers=1)
    rep = run_parity(w, n_windows=1, verbose=False)
    _report(f"lmhead_tile_vocab{vocab}", rep)
    assert rep["ok"], worst_entries(rep)


def test_caller_may_overwrite_dy_right_after_backward():
    """Gradient leaves keep running on the side stream after backward returns,
    and the first ones read the caller's dY: overwriting dY on the caller's
    stream right behind the call must not change the gradient."""
    import torch
    from oracle.stage import Stage as OStage
    w = W.TINY["gpt_tile"]
    theta0 = W.make_theta(w, OStage.from_workload(w).layout)
    x = torch.from_numpy(W.make_x(w, 0)).to("cuda:0").to(torch.bfloat16)
    dy0 = torch.from_numpy(W.make_dy(w, 0)).to("cuda:0").to(torch.bfloat16)
    grads = []
    for clobber in (False, True):
        gpu = GpuStage(w)
        gpu.set_state(theta0)
        gpu.stage.amdp_stage_set_overlap(True)              # small stage: off by default
        assert gpu.stage.amdp_stage_get_overlap()
        y, dx, dy = torch.empty_like(x), torch.empty_like(x), dy0.clone()
        gpu.stage.amdp_stage_forward(0, 0, x, None, y)
        gpu.stage.amdp_stage_backward(0, 0, dy, dx)
        if clobber:
            dy.fill_(float("nan"))
        g = torch.empty(gpu.n, dtype=torch.float32, device="cuda:0")
        gpu.stage.amdp_stage_get_staged_grad(g)
        torch.cuda.synchronize()
        grads.append(g.cpu().numpy())
        gpu.stage.close()
    assert np.all(np.isfinite(grads[1])) and np.array_equal(grads[0], grads[1])


@pytest.mark.parametrize("key", ["gpt_tile", "lmhead_tile", "bert_mid", "gpt"])
def test_fused_accumulate_bit_identical(key):
    """amdp_stage_set_fused_accumulate(1): backward adds into G directly. A
    whole schedule must end in exactly the state of the two-step form; the
    per-minibatch gradient is then not available."""
    import torch
    import paper_2605_29664_amd as amdp
    from oracle.stage import Stage as OStage
    w = W.TINY[key]
    theta0 = W.make_theta(w, OStage.from_workload(w).layout)
    M = 2 * w.threshold + w.act_slots
    ev = amdp.amdp_schedule_generate(w.depth, w.pipelines, w.stage, w.threshold, M, w.inject_limit,
                                     amdp.U_NEXT_BUBBLE, amdp.BWD_STASHED)
    finals = []
    for fused in (False, True):
        gpu = GpuStage(w, act_slots=w.act_slots, stash_slots=2)
        gpu.stage.amdp_stage_set_overlap(True)      # small stage: off by default
        gpu.set_state(theta0)
        gpu.stage.amdp_stage_set_fused_accumulate(fused)
        dt = gpu.dt
        y = torch.empty(1, dtype=torch.float32, device="cuda:0") if w.has_lm_head else \
            torch.empty((w.tokens, w.d_model), dtype=dt, device="cuda:0")
        dx = torch.empty((w.tokens, w.d_model), dtype=dt, device="cuda:0")
        keep, sums = [], []
        n_partial = 0
        for e in ev:
            if e.kind == amdp.EV_F:
                x = gpu.to_dev(W.make_x(w, e.mb), dt)
                a = W.make_aux(w, e.mb)
                a = None if a is None else gpu.to_dev(np.asarray(a, dtype=np.int32))
                keep += [x, a]
                gpu.stage.amdp_stage_forward(e.mb, e.version, x, a, y)
            elif e.kind == amdp.EV_B:
                dy = None if w.has_lm_head else gpu.to_dev(W.make_dy(w, e.mb), dt)
                keep.append(dy)
                gpu.stage.amdp_stage_backward(e.mb, e.version, dy, dx)
                if fused and n_partial == 0:
                    n_partial = 1
                    with pytest.raises(amdp.AmdpError):
                        gpu.stage.amdp_stage_get_staged_grad(torch.empty(gpu.n, dtype=torch.float32, device="cuda:0"))
                    with pytest.raises(amdp.AmdpError):      # not between a backward and its accumulate
                        gpu.stage.amdp_stage_set_fused_accumulate(False)
            elif e.kind == amdp.EV_A:
                gpu.stage.amdp_grad_accumulate(e.mb)
            else:
                sums.append(gpu.state()["G"])           # the window's gradient sum, just before it is applied
                gpu.stage.amdp_apply_update(w.lr, w.beta1, w.beta2, w.eps, w.weight_decay, 1.0 / w.threshold, True)
        s = gpu.state()
        torch.cuda.synchronize()
        finals.append([s["theta"], s["m"], s["v"], dx.float().cpu().numpy()] + sums)
        gpu.stage.close()
    assert np.any(finals[0][0] != theta0) and all(np.any(G != 0.0) for G in finals[0][4:])
    assert len(finals[0]) == len(finals[1]) >= 6
    for k, (a, b) in enumerate(zip(*finals)):
        assert np.array_equal(a, b), k


@pytest.mark.parametrize("key", ["embed", "embed_tile", "embed_bert_mid"])
def test_first_stage_with_input_embedding(key):
    """Token ids in, token + position embedding in front of the blocks; the
    vocabularies are small so that tokens repeat inside a minibatch and the
    deterministic row sums of the token gradient are exercised."""
    rep = run_parity(W.TINY[key], n_windows=1, verbose=False)
    _report(key, rep)
    assert rep["ok"], worst_entries(rep)


def test_input_embedding_gradient_is_deterministic_and_fuses():
    import torch
    w = W.TINY["embed_tile"]
    from oracle.stage import Stage as OStage
    theta0 = W.make_theta(w, OStage.from_workload(w).layout)
    res = []
    for fused in (False, False, True):
        gpu = GpuStage(w, act_slots=2, stash_slots=1)
        gpu.stage.amdp_stage_set_overlap(True)      # small stage: off by default
        gpu.set_state(theta0)
        gpu.stage.amdp_stage_set_fused_accumulate(fused)
        tok = gpu.to_dev(W.make_tokens(w, 0))
        dy = gpu.to_dev(W.make_dy(w, 0), gpu.dt)
        y = torch.empty((w.tokens, w.d_model), dtype=gpu.dt, device="cuda:0")
        for mb in (0, 1):                        # two minibatches into the sum
            gpu.stage.amdp_stage_forward(mb, 0, None, tok, y)
            gpu.stage.amdp_stage_backward(mb, 0, dy, None)
            gpu.stage.amdp_grad_accumulate(mb)
        res.append(gpu.state()["G"])
        gpu.stage.close()
    assert np.any(res[0] != 0.0)
    assert np.array_equal(res[0], res[1]) and np.array_equal(res[0], res[2])


def test_tied_embedding_gradients_are_summed_into_both_stages():
    import torch
    import paper_2605_29664_amd as amdp
    wf = W.TINY["embed_tile"].with_(vocab=1931)
    wl = W.TINY["lmhead_tile"]
    assert wf.vocab == wl.vocab and wf.d_model == wl.d_model
    first, last = GpuStage(wf, act_slots=2, stash_slots=1), GpuStage(wl, act_slots=2, stash_slots=1)
    first.stage.amdp_stage_set_overlap(True)        # small stages: off by default
    last.stage.amdp_stage_set_overlap(True)
    from oracle.stage import Stage as OStage
    first.set_state(W.make_theta(wf, OStage.from_workload(wf).layout))
    last.set_state(W.make_theta(wl, OStage.from_workload(wl).layout))
    y = torch.empty((wf.tokens, wf.d_model), dtype=first.dt, device="cuda:0")
    first.stage.amdp_stage_forward(0, 0, None, first.to_dev(W.make_tokens(wf, 0)), y)
    first.stage.amdp_stage_backward(0, 0, first.to_dev(W.make_dy(wf, 0), first.dt), None)
    first.stage.amdp_grad_accumulate(0)
    loss = torch.empty(1, dtype=torch.float32, device="cuda:0")
    last.stage.amdp_stage_forward(0, 0, last.to_dev(W.make_x(wl, 0), last.dt), last.to_dev(W.make_targets(wl, 0)), loss)
    last.stage.amdp_stage_backward(0, 0, None, None)
    last.stage.amdp_grad_accumulate(0)
    Gf, Gl = first.state()["G"], last.state()["G"]
    VD = wf.vocab * wf.d_model
    off_l = [off for name, off, r, c in amdp.amdp_stage_param_layout(last.cfg) if name == "embed"][0]
    want = Gf[:VD] + Gl[off_l:off_l + VD]                      # fp32 addition, as the kernel does it
    assert np.any(Gf[:VD] != 0.0) and np.any(Gl[off_l:off_l + VD] != 0.0)
    amdp.amdp_tie_embedding_grads(first.stage, last.stage)
    Gf2, Gl2 = first.state()["G"], last.state()["G"]
    assert np.array_equal(Gf2[:VD], want) and np.array_equal(Gl2[off_l:off_l + VD], want)
    assert np.array_equal(Gf2[VD:], Gf[VD:]) and np.array_equal(Gl2[:off_l], Gl[:off_l])
    with pytest.raises(amdp.AmdpError):
        amdp.amdp_tie_embedding_grads(last.stage, first.stage)
    first.stage.close()
    last.stage.close()


@pytest.mark.parametrize("name,kw", [
    ("pipedream", dict(inject_limit=4, threshold=1, placement=OSched.EAGER, policy=OSched.STASHED)),
    ("pipedream_2bw", dict(inject_limit=4, threshold=4, placement=OSched.EAGER, policy=OSched.STASHED)),
    ("sync_1f1b", dict(inject_limit=4, threshold=6, placement=OSched.FLUSH, policy=OSched.STASHED)),
])
def test_comparison_schedules_through_the_stage_library(name, kw):
    """The schedules Table 1 compares AMDP with, run through the same stage
    library: PipeDream's stage 1 of 4 stashes three versions, 2BW two, the
    flushed schedule none."""
    w = W.TINY["gpt_tile"].with_(depth=4, pipelines=1, stage=1, n_layers=1, lr=1e-3)
    rep = run_parity(w, n_minibatches=14, verbose=False, **kw)
    _report(name, rep)
    assert rep["ok"], worst_entries(rep)


@pytest.mark.parametrize("overlap", [True, False])
def test_hip_graph_replay_matches_eager(overlap):
    """Forward + backward + accumulate captured once in a HIP graph (the library
    clears and copies with its own kernels and, with the side stream on, forks and
    joins it with events, all of which a capture records) and replayed three times with
    eager work and synchronisation in between must reproduce, bit for bit, the
    eager results: Y, dX, and G after one, two and three accumulations."""
    import torch
    import paper_2605_29664_amd as amdp
    from tests.parity import make_cfg
    w = W.TINY["gpt_tile"]
    dev = torch.device("cuda:0")
    cfg = make_cfg(w, act_slots=2, stash_slots=1)
    theta0 = torch.from_numpy(W.make_theta(w, amdp.amdp_stage_param_layout(cfg))).to(dev)
    s = torch.cuda.Stream(device=dev)
    dt = torch.bfloat16
    xs = [torch.from_numpy(W.make_x(w, k)).to(dev).to(dt) for k in (0, 1, 0)]
    dy = torch.from_numpy(W.make_dy(w, 0)).to(dev).to(dt)

    def fresh():
        st = amdp.Stage(cfg, device="cuda:0", stream=s)
        st.amdp_stage_set_overlap(overlap)
        with torch.cuda.stream(s):
            st.amdp_stage_set_state(theta0)
        s.synchronize()
        return st

    def fba(st, X, Y, dX):
        st.amdp_stage_forward(0, 0, X, None, Y)
        st.amdp_stage_backward(0, 0, dy, dX)
        st.amdp_grad_accumulate(0)
        st.amdp_stage_join()            # the accumulation runs on the stage's side stream

    def read_G(st):
        G = torch.empty(st.n_params, dtype=torch.float32, device=dev)
        with torch.cuda.stream(s):
            st.amdp_stage_get_state(None, None, None, G)
        s.synchronize()
        return G

    st = fresh()
    Y, dX, ref = torch.empty_like(xs[0]), torch.empty_like(xs[0]), []
    for X in xs:
        with torch.cuda.stream(s):
            fba(st, X, Y, dX)
        s.synchronize()
        ref.append((Y.clone(), dX.clone(), read_G(st)))
    st.close()

    st = fresh()                        # same process: kernel attributes and occupancy queries are cached
    Xs = xs[0].clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        fba(st, Xs, Y, dX)
    for k, X in enumerate(xs):
        Xs.copy_(X)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        got = (Y, dX, read_G(st))
        for name, a, b in zip(("Y", "dX", "G"), got, ref[k]):
            assert torch.equal(a, b), f"replay {k}: {name} differs from the eager run"
    st.close()


def test_run_to_run_determinism():
    w = W.TINY["bert_tile"]
    res = []
    for _ in range(2):
        gpu = GpuStage(w)
        from oracle.stage import Stage as OStage
        gpu.set_state(W.make_theta(w, OStage.from_workload(w).layout))
        y = gpu.forward(0, 0, W.make_x(w, 0), W.make_valid_len(w, 0))
        dx, g = gpu.backward(0, 0, W.make_dy(w, 0))
        res.append((y, dx, g))
        gpu.stage.close()
    for a, b in zip(*res):
        assert np.array_equal(a, b)


def test_adam_kernel_in_isolation():
    """Same fp32 G, m, v, theta into kernel and oracle: one update must agree
    to fp32 rounding (norm-wise <= 1e-6)."""
    import torch
    from oracle import optim
    from oracle.stage import Stage as OStage
    w = W.TINY["gpt_tile"]
    ost = OStage.from_workload(w)
    rng = np.random.default_rng(7)
    n = ost.n_params
    theta = W.make_theta(w, ost.layout)
    m = (1e-4 * rng.standard_normal(n)).astype(np.float32)
    v = (1e-8 * rng.random(n)).astype(np.float32)
    gpu = GpuStage(w)
    gpu.set_state(theta, m, v, step=6, version=3)
    # build a known G by one forward/backward/accumulate
    gpu.forward(0, 3, W.make_x(w, 0), None)
    gpu.backward(0, 3, W.make_dy(w, 0))
    gpu.accumulate(0)
    G = gpu.state()["G"]
    nv = gpu.update(w, 0.25)
    s = gpu.state()
    th_ref, m_ref, v_ref = optim.adam_step(theta.astype(np.float64), m.astype(np.float64), v.astype(np.float64),
                                           G.astype(np.float64), 7, w.lr, w.beta1, w.beta2, w.eps,
                                           grad_scale=0.25)
    assert nv == 4 and s["step"] == 7
    assert rel_err(s["theta"], th_ref) <= 1e-6
    assert rel_err(s["m"], m_ref) <= 1e-6 and rel_err(s["v"], v_ref) <= 1e-6
    assert rel_err(s["theta"] - theta, th_ref - theta) <= 1e-4
    assert np.all(s["G"] == 0.0)
    gpu.stage.close()


def test_state_machine_errors():
    import paper_2605_29664_amd as amdp
    from oracle.stage import Stage as OStage
    w = W.TINY["gpt_tile"]
    gpu = GpuStage(w, act_slots=2, stash_slots=1)
    gpu.set_state(W.make_theta(w, OStage.from_workload(w).layout))
    x, dy = W.make_x(w, 0), W.make_dy(w, 0)

    def code(fn):
        with pytest.raises(amdp.AmdpError) as ei:
            fn()
        return ei.value.code

    assert code(lambda: gpu.backward(0, 0, dy)) == amdp.E_MB_STATE         # backward without forward
    assert code(lambda: gpu.accumulate(0)) == amdp.E_MB_STATE
    assert code(lambda: gpu.forward(0, 5, x, None)) == amdp.E_VERSION      # version never published
    gpu.forward(0, 0, x, None)
    assert code(lambda: gpu.forward(0, 0, x, None)) == amdp.E_MB_STATE     # already in flight
    gpu.forward(1, 0, x, None)
    assert code(lambda: gpu.forward(2, 0, x, None)) == amdp.E_NO_SLOT      # act_slots = 2
    gpu.update(w, 1.0)                                                      # v1; v0 pinned by mb 0, 1
    assert gpu.stage.amdp_stage_resident_versions() == [0, 1]
    assert code(lambda: gpu.update(w, 1.0)) == amdp.E_STASH_FULL           # both slots still needed
    gpu.backward(0, 0, dy)
    assert code(lambda: gpu.backward(1, 0, dy)) == amdp.E_MB_STATE         # staging buffer occupied
    assert code(lambda: gpu.update(w, 1.0)) == amdp.E_MB_STATE             # gradient not yet accumulated
    gpu.accumulate(0)
    gpu.backward(1, 0, dy)
    gpu.accumulate(1)
    assert gpu.stage.amdp_stage_resident_versions() == [1]                  # v0 dropped with its last reader
    assert code(lambda: gpu.forward(3, 0, x, None)) == amdp.E_VERSION
    gpu.update(w, 1.0)
    assert gpu.stage.amdp_stage_resident_versions() == [2]
    gpu.stage.close()
