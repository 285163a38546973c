"""Products whose operands are longer than the 2 GiB that a buffer offset reaches."""
import numpy as np
import pytest
import torch

import paper_2605_29664_amd as amdp
from tests.parity import rel_err

pytestmark = pytest.mark.gpu


def _need(gib):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < gib * 2**30:
        pytest.skip(f"needs {gib} GiB of GPU memory")


@pytest.mark.parametrize("tile", [256, 128, 64])
def test_weight_gradients_over_2_gib_operands(tile):
    """66560 tokens x d_ffn 16384 are 2.03 GiB: the gradients of W_1 (the second operand that long) and W_2 (the first)
    contract over all of them on the matrix cores (72 columns divide into no tile, so no other matrix kernel takes them)
    and agree with the generic kernel's. The last 1024 tokens, which lie past 2 GiB, are an eighth of the gradient's norm."""
    _need(40)
    seq, batch, d, f = 64, 1040, 72, 16384
    n = seq * batch
    cfg = amdp.make_config(amdp.BLOCK_GPT, 1, d, 1, f, seq, batch, amdp.BF16, act_slots=1, stash_slots=1)
    layout = {name: (off, off + r * c) for name, off, r, c in amdp.amdp_stage_param_layout(cfg)}
    g = torch.Generator(device="cuda:0").manual_seed(5)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda:0")  # noqa: E731
    stage = amdp.Stage(cfg, device="cuda:0")
    theta = 0.02 * randn(stage.n_params)
    for name, (a, b) in layout.items():
        if name.endswith("gamma"):
            theta[a:b] += 1.0
    stage.amdp_stage_set_state(theta)
    x, dy = randn(n, d).bfloat16(), (1e-3 * randn(n, d)).bfloat16()
    y, dx = torch.empty_like(x), torch.empty_like(x)
    got = {}
    for opt in (-1, tile):
        stage.amdp_stage_set_option(amdp.OPT_GEMM_TILE, 0)
        stage.amdp_stage_forward(0, 0, x, None, y)
        stage.amdp_stage_set_option(amdp.OPT_GEMM_TILE, opt)
        stage.amdp_stage_profile_begin()
        stage.amdp_stage_backward(0, 0, dy, dx)
        names = stage.amdp_stage_profile_end()
        grad = torch.empty(stage.n_params, dtype=torch.float32, device="cuda:0")
        stage.amdp_stage_get_staged_grad(grad)
        stage.amdp_grad_accumulate(0)
        got[opt] = {k: grad[a:b].cpu().numpy() for k, (a, b) in layout.items()}
        assert any(k.startswith("gemm_generic") for k in names) == (opt == -1), list(names)
    # W_2: the same bf16 operands, 66560 fp32 additions in another order: sqrt(66560 / 2) roundings of 2^-25 of the
    # partial sums' size, 5e-6 of the result. The others contract activations' gradients, of which some round to the
    # neighbouring bf16 value: 2^-9 of some entries
    assert rel_err(got[tile]["l0.w_2"], got[-1]["l0.w_2"]) < 2e-5
    for name in ("l0.w_1", "l0.w_o", "l0.w_qkv"):
        assert rel_err(got[tile][name], got[-1][name]) < 4e-3, name
    assert all(np.isfinite(v).all() for v in got[tile].values())
    stage.close()


def test_vocabulary_gradient_with_rows_over_8_mib():
    """The logits of 4.2 M words: rows of 8.4 MB, of which the gradient of the vocabulary projection contracts 64 at a
    time. 72 columns divide into no tile, so no other matrix kernel takes it; agrees with the generic kernel's."""
    _need(30)
    seq, batch, d, f, vocab = 64, 2, 72, 72, 4_200_001
    cfg = amdp.make_config(amdp.BLOCK_GPT, 1, d, 1, f, seq, batch, amdp.BF16, has_lm_head=True, vocab=vocab, act_slots=1, stash_slots=1)
    a, b = next((off, off + r * c) for name, off, r, c in amdp.amdp_stage_param_layout(cfg) if name == "embed")
    g = torch.Generator(device="cuda:0").manual_seed(6)
    stage = amdp.Stage(cfg, device="cuda:0")
    theta = 0.02 * torch.randn(stage.n_params, generator=g, device="cuda:0")
    stage.amdp_stage_set_state(theta)
    x = torch.randn((seq * batch, d), generator=g, device="cuda:0").bfloat16()
    targets = torch.randint(0, vocab, (seq * batch,), generator=g, device="cuda:0", dtype=torch.int32)
    loss = torch.empty(1, dtype=torch.float32, device="cuda:0")
    got, names = [], []
    for opt in (-1, 0):
        stage.amdp_stage_set_option(amdp.OPT_GEMM_TILE, 0)
        stage.amdp_stage_forward(0, 0, x, targets, loss)
        stage.amdp_stage_set_option(amdp.OPT_GEMM_TILE, opt)
        stage.amdp_stage_profile_begin()
        stage.amdp_stage_backward(0, 0, None, None)
        names.append([k for k in stage.amdp_stage_profile_end() if k.endswith("_TN")])
        grad = torch.empty(stage.n_params, dtype=torch.float32, device="cuda:0")
        stage.amdp_stage_get_staged_grad(grad)
        stage.amdp_grad_accumulate(0)
        got.append(grad[a:b].cpu().numpy())
    assert names[0] == ["gemm_generic_TN"] and "gemm_generic_TN" not in names[1], names
    assert np.isfinite(got[1]).all()
    assert rel_err(got[1], got[0]) < 1e-6      # 128 fp32 additions of the same products in another order
    stage.close()
