"""Launches of more lanes than one dimension of a grid holds (2^32; a larger one wraps without an error)."""
import pytest
import torch

import paper_2605_29664_amd as amdp

pytestmark = pytest.mark.gpu


def _need(gib):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < gib * 2**30:
        pytest.skip(f"needs {gib} GiB of GPU memory")


def _sample(rows, cols):
    """The first two and last four rows random, all others zero."""
    at = torch.tensor([0, 1, rows - 4, rows - 3, rows - 2, rows - 1], device="cuda:0")
    t = torch.zeros((rows, cols), dtype=torch.bfloat16, device="cuda:0")
    t[at] = torch.randn((6, cols), generator=torch.Generator(device="cuda:0").manual_seed(9), device="cuda:0").bfloat16()
    return at, t


# rows that a workgroup takes over from a wave (forward from 257 vectors on with many rows, backward from 129)
@pytest.mark.parametrize("vectors,forward", [(257, True), (129, False)])
def test_layernorm_of_more_rows_than_2_to_24(vectors, forward):
    """A workgroup of 256 lanes to each row."""
    rows, cols = 2**24 + 3, vectors * 8
    _need(150 if forward else 80)
    at, x = _sample(rows, cols)
    gamma = (1 + 0.1 * torch.randn(cols, device="cuda:0")).bfloat16()
    beta = (0.1 * torch.randn(cols, device="cuda:0")).bfloat16()
    out = torch.full((rows, cols), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    xs = x[at].double()
    mean, rstd = xs.mean(1, keepdim=True), (xs.var(1, unbiased=False, keepdim=True) + 1e-5).rsqrt()
    xh = (xs - mean) * rstd
    stats = torch.zeros((rows, 2), dtype=torch.float32, device="cuda:0")
    if forward:
        amdp.amdp_layernorm_forward(x, gamma, beta, out, stats, 1e-5)
        want, rest = xh * gamma.double() + beta.double(), beta
    else:
        stats[at] = torch.cat([mean, rstd], 1).float()
        amdp.amdp_layernorm_backward(x, x, stats, gamma, None, out)      # dy = x
        d = xs * gamma.double()
        want, rest = rstd * (d - d.mean(1, keepdim=True) - xh * (d * xh).mean(1, keepdim=True)), torch.zeros_like(beta)
    # one bf16 rounding (2^-9) of values of at most the largest one's size, beside fp32 sums
    assert (out[at].double() - want).abs().max() <= 2.0**-8 * want.abs().max()
    for first in range(2, rows - 4, 2**20):
        assert bool((out[first:min(first + 2**20, rows - 4)] == rest).all()), first
    del x, out, stats
    torch.cuda.empty_cache()


def test_copy_of_more_than_64_gib():
    """One 16-byte vector to a lane: 2^32 lanes move 64 GiB."""
    _need(135)
    n = 2**33 + 2**20                     # 64-bit words: 64 GiB and 8 MiB
    src = torch.empty(n, dtype=torch.int64, device="cuda:0")
    dst = torch.zeros(n, dtype=torch.int64, device="cuda:0")
    parts = [slice(first, min(first + 2**28, n)) for first in range(0, n, 2**28)]
    for p in parts:
        src[p] = torch.arange(p.start + 1, p.stop + 1, device="cuda:0")
    amdp.amdp_device_copy(dst, src)
    for p in parts:
        assert torch.equal(dst[p], torch.arange(p.start + 1, p.stop + 1, device="cuda:0")), p
    del src, dst
    torch.cuda.empty_cache()
