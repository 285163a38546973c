"""Products whose sides are multiples of 8 but of no tile, on every tile of the
direct-to-LDS matrix kernel in each of its forms, and products whose contraction the
library splits by itself: whole small stages against the CPU oracle (tests/parity.py)."""
import numpy as np
import pytest

import workloads as W
from tests.parity import run_parity, worst_entries, GpuStage, rel_err
from paper_2605_29664_amd.binding import OPT_GEMM_TILE, OPT_SPLIT_K_MIN_TOKENS, OPT_SPLIT_MAIN_MIN_K

pytestmark = pytest.mark.gpu

# tokens x width x FFN: one 8-wide step past a tile edge, one short of it, less than a k-tile, and
# contractions with a tail of 8 and of 56
SHAPES = {
    "264x136x520": dict(seq_len=88, microbatch=3, d_model=136, n_heads=4, d_ffn=520),
    "504x248x760": dict(seq_len=168, microbatch=3, d_model=248, n_heads=4, d_ffn=760),
    "24x40x72": dict(seq_len=24, microbatch=1, d_model=40, n_heads=1, d_ffn=72),
    "1000x320x328": dict(seq_len=200, microbatch=5, d_model=320, n_heads=5, d_ffn=328),
}


@pytest.mark.parametrize("tile", [0, 256, 256128, 128, 64])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_sides_of_no_tile(shape, tile):
    w = W.TINY["gpt_mid"].with_(n_layers=1, depth=2, pipelines=1, stage=1, threshold=2, **SHAPES[shape])
    rep = run_parity(w, n_windows=1, verbose=False, options={OPT_GEMM_TILE: tile})
    assert rep["ok"], worst_entries(rep)


def _product_names(w, options):
    """Profile names of one minibatch's products."""
    import torch
    from oracle.stage import Stage as OStage
    gpu = GpuStage(w, act_slots=1, stash_slots=1, options=options)
    gpu.set_state(W.make_theta(w, OStage.from_workload(w).layout))
    x, dy = gpu.to_dev(W.make_x(w, 0), gpu.dt), gpu.to_dev(W.make_dy(w, 0), gpu.dt)
    y, dx = torch.empty_like(x), torch.empty_like(x)
    gpu.stage.amdp_stage_profile_begin()
    gpu.stage.amdp_stage_forward(0, 0, x, None, y)
    gpu.stage.amdp_stage_backward(0, 0, dy, dx)
    names = {k for k in gpu.stage.amdp_stage_profile_end() if k.startswith("gemm_")}
    gpu.stage.close()
    return names


# More than 256 tiles of 128x128 and more than 512 of 64x64 in products of every layout (2064 x 4104, 2064 x 3096 and
# 1032 x 4104 outputs, no side a multiple of any tile, contractions with tails of 8 and 16): there 128 and 64 take
# their forms with two and five workgroups to a compute unit, and the smaller shapes above those with one and two
@pytest.mark.parametrize("tile", [256, 256128, 128, 64])
def test_many_tiles_with_odd_sides(tile):
    w = W.TINY["gpt_mid"].with_(n_layers=1, depth=2, pipelines=1, stage=1, seq_len=1032, microbatch=2, d_model=1032, n_heads=12,
                                d_ffn=4104)
    rep = run_parity(w, threshold=1, n_minibatches=1, verbose=False, options={OPT_GEMM_TILE: tile})
    assert rep["ok"], worst_entries(rep)
    size = "256x128" if tile == 256128 else f"{tile}x{tile}"
    assert _product_names(w, {OPT_GEMM_TILE: tile}) == {f"gemm_mfma{size}_{layout}" for layout in ("NN", "NT", "TN")}


def test_library_choice_with_odd_sides():
    """3 x 1000 tokens, 768 wide: the choice goes to 256x128 and 128x128 tiles, whose last rows are cut."""
    w = W.TINY["gpt_mid"].with_(n_layers=1, depth=2, pipelines=1, stage=1, seq_len=1000, microbatch=3, d_model=768, n_heads=12,
                                d_ffn=3072)
    rep = run_parity(w, threshold=1, n_minibatches=1, verbose=False)
    assert rep["ok"], worst_entries(rep)
    names = _product_names(w, None)
    assert any("256x128" in n for n in names) and any("128x128" in n for n in names), names


def test_lm_head_with_odd_sides():
    w = W.TINY["lmhead_mid"].with_(seq_len=104, microbatch=3, d_model=200, n_heads=4, d_ffn=520, vocab=777, threshold=2)
    rep = run_parity(w, n_windows=1, verbose=False)
    assert rep["ok"], worst_entries(rep)


@pytest.mark.parametrize("fused", [False, True])
def test_contractions_split_by_the_plan(fused):
    """Many tokens on a narrow stage (weight gradients in parts, the last one shorter) and a long FFN on few
    tokens (forward and dX products in parts). The profile shows that parts ran; the sums agree with the
    unsplit products to fp32 summation error and are the same bits run to run."""
    import torch
    for w in (W.TINY["gpt_tile64"].with_(n_layers=1, seq_len=1288, microbatch=5),
              W.TINY["gpt_tile64"].with_(n_layers=1, seq_len=200, microbatch=2, d_ffn=16392)):
        from oracle.stage import Stage as OStage
        theta0 = W.make_theta(w, OStage.from_workload(w).layout)
        sums, dxs, names = [], [], []
        for options in ({}, {}, {OPT_SPLIT_K_MIN_TOKENS: 1 << 20, OPT_SPLIT_MAIN_MIN_K: 1 << 20}):
            gpu = GpuStage(w, act_slots=2, stash_slots=1, options=options)
            gpu.set_state(theta0)
            gpu.stage.amdp_stage_set_fused_accumulate(fused)
            x, dy = gpu.to_dev(W.make_x(w, 0), gpu.dt), gpu.to_dev(W.make_dy(w, 0), gpu.dt)
            y, dx = torch.empty_like(x), torch.empty_like(x)
            gpu.stage.amdp_stage_profile_begin()
            gpu.stage.amdp_stage_forward(0, 0, x, None, y)
            gpu.stage.amdp_stage_backward(0, 0, dy, dx)
            gpu.stage.amdp_grad_accumulate(0)
            names.append([k for k in gpu.stage.amdp_stage_profile_end() if k.endswith("_splitk")])
            sums.append(gpu.state(("G",))["G"])
            dxs.append(dx.float().cpu().numpy())
            gpu.stage.close()
        assert names[0] and names[0] == names[1] and not names[2]
        assert np.array_equal(sums[0], sums[1]) and np.array_equal(dxs[0], dxs[1])
        # one bf16 rounding of an activation may flip between the two orders of summation: 2^-9 of some entries
        assert rel_err(sums[0], sums[2]) < 2e-3 and rel_err(dxs[0], dxs[2]) < 4e-3


def test_split_options_give_the_choice_back():
    """0 takes both split options back to the library's own choice, as before either was set."""
    import torch
    w = W.TINY["gpt_tile64"].with_(n_layers=1, seq_len=200, microbatch=2, d_ffn=16392)
    from oracle.stage import Stage as OStage
    gpu = GpuStage(w, act_slots=1, stash_slots=1)
    gpu.set_state(W.make_theta(w, OStage.from_workload(w).layout))
    x, dy = gpu.to_dev(W.make_x(w, 0), gpu.dt), gpu.to_dev(W.make_dy(w, 0), gpu.dt)
    y, dx = torch.empty_like(x), torch.empty_like(x)
    splits = []
    for value in (None, 1 << 20, 0):
        for opt in (OPT_SPLIT_K_MIN_TOKENS, OPT_SPLIT_MAIN_MIN_K):
            if value is not None:
                gpu.stage.amdp_stage_set_option(opt, value)
        gpu.stage.amdp_stage_profile_begin()
        gpu.stage.amdp_stage_forward(0, 0, x, None, y)
        gpu.stage.amdp_stage_backward(0, 0, dy, dx)
        gpu.stage.amdp_grad_accumulate(0)
        splits.append({k: v["launches"] for k, v in gpu.stage.amdp_stage_profile_end().items() if k.endswith("_splitk")})
    gpu.stage.close()
    assert splits[0] and not splits[1] and splits[2] == splits[0]
