"""LayerNorm forward and backward around the row lengths at which a workgroup takes over a row from a wave, and around
the number of rows that decides it for the forward; column sums around the number of rows up to which one launch does
them. Against float64 on the CPU."""
import pytest
import torch

import paper_2605_29664_amd as amdp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("rows,vectors", [(r, v) for r in (1, 7) for v in (1, 128, 129, 255, 256, 257, 512, 513, 1024, 1025)] +
                         [(4096, v) for v in (129, 256, 257)])
def test_rows(rows, vectors, dtype, residual):
    dt, n = (torch.bfloat16, 8) if dtype == "bf16" else (torch.float32, 4)
    cols = vectors * n
    g = torch.Generator().manual_seed(rows * 4099 + cols)
    x, dy, res = (torch.randn((rows, cols), generator=g).to(dt) for _ in range(3))
    gamma, beta = (1 + 0.1 * torch.randn(cols, generator=g)).to(dt), (0.1 * torch.randn(cols, generator=g)).to(dt)
    dev = [t.cuda() for t in (x, dy, res, gamma, beta)]
    y, dx = torch.empty_like(dev[0]), torch.empty_like(dev[0])
    stats = torch.empty((rows, 2), dtype=torch.float32, device="cuda:0")
    amdp.amdp_layernorm_forward(dev[0], dev[3], dev[4], y, stats, 1e-5)
    amdp.amdp_layernorm_backward(dev[1], dev[0], stats, dev[3], dev[2] if residual else None, dx)
    x, dy, res, gamma, beta = (t.double() for t in (x, dy, res, gamma, beta))
    mean, rstd = x.mean(1, keepdim=True), (x.var(1, unbiased=False, keepdim=True) + 1e-5).rsqrt()
    xh, d = (x - mean) * rstd, dy * gamma
    ref = rstd * (d - d.mean(1, keepdim=True) - xh * (d * xh).mean(1, keepdim=True)) + (res if residual else 0.0)
    # one rounding of the result (2^-9 of it in bf16) and fp32 sums of at most 8200 terms; a value of a one-vector row
    # can be the small difference of its terms, so the unit is the largest value of the tensor
    tol = 2.0 ** -8 if dtype == "bf16" else 2e-6
    for got, want in ((y, xh * gamma + beta), (dx, ref), (stats[:, :1], mean), (stats[:, 1:], rstd)):
        scale = tol if got.dtype == dt else 2e-6
        err = (got.cpu().double() - want).abs().max().item()
        assert err <= scale * max(1.0, want.abs().max().item()), (err, want.abs().max().item())


@pytest.mark.parametrize("layernorm", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("rows,vectors", [(1, 1), (31, 7), (32, 8), (33, 9), (127, 250), (129, 64), (384, 17), (385, 17)])
def test_column_sums(rows, vectors, dtype, layernorm):
    dt, n = (torch.bfloat16, 8) if dtype == "bf16" else (torch.float32, 4)
    cols = vectors * n
    g = torch.Generator().manual_seed(rows * 4099 + cols)
    dy, x = (torch.randn((rows, cols), generator=g).to(dt) for _ in range(2))
    stats = torch.stack([0.1 * torch.randn(rows, generator=g), 1 + 0.1 * torch.rand(rows, generator=g)], 1).contiguous()
    out = torch.full(((2 if layernorm else 1) * cols,), 7.0, dtype=torch.float32, device="cuda:0")
    ws = torch.empty(amdp.amdp_column_sums_workspace_bytes(rows, cols, amdp.BF16 if dtype == "bf16" else amdp.FP32, layernorm),
                     dtype=torch.uint8, device="cuda:0")
    amdp.amdp_column_sums(dy.cuda(), x.cuda() if layernorm else None, stats.cuda() if layernorm else None, out, ws)
    dy, x, stats = dy.double(), x.double(), stats.double()
    parts = ([dy * (x - stats[:, :1]) * stats[:, 1:]] if layernorm else []) + [dy]
    want, size = (torch.cat([f(p).sum(0) for p in parts]) for f in (lambda p: p, torch.abs))
    # an fp32 sum of `rows` terms: fewer than 32 roundings in a row in any order used, each 2^-24 of the sum of magnitudes
    assert torch.all((out.cpu().double() - want).abs() <= 32 * 2.0 ** -24 * size + 1e-30)


def test_column_sums_of_no_rows():
    out = torch.full((24,), 7.0, dtype=torch.float32, device="cuda:0")
    ws = torch.empty(amdp.amdp_column_sums_workspace_bytes(0, 24, amdp.BF16, False), dtype=torch.uint8, device="cuda:0")
    amdp.amdp_column_sums(torch.empty((0, 24), dtype=torch.bfloat16, device="cuda:0"), None, None, out, ws)
    assert torch.all(out == 0)
