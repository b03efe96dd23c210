"""LayerNorm backward with its gamma / beta sums in the same launch: row counts around a block and a chunk, widths around a vector per lane,
one chunk and several, results equal to the wide form's reference and repeatable."""
import pytest
import torch

from paper_2111_04007_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,width", [(1, 8), (3, 72), (5, 520), (255, 64), (256, 1016), (257, 1928), (513, 2048), (1030, 4096), (600, 4104)])
def test_joint_backward(dtype, rows, width):
    """dx: one rounding of the storage type on fp32 arithmetic; the sums: fp32 over `rows` terms."""
    g = torch.Generator(device="cuda").manual_seed(rows)
    x, dy, res = (torch.empty(rows, width, device="cuda").normal_(0, 1, generator=g).to(dtype) for _ in range(3))
    gamma, beta = (torch.empty(width, device="cuda").normal_(m, 0.1, generator=g).to(dtype) for m in (1.0, 0.0))
    stats, y = torch.empty(2 * rows, device="cuda"), torch.empty_like(x)
    B.op_layernorm_fwd(x, gamma, beta, y, stats)
    partial = torch.empty(B.colreduce_scratch_bytes(rows, 2 * width) // 4, device="cuda")
    got = []
    for _ in range(2):
        dx, dg, db = torch.full_like(x, 7.0), torch.full((width,), 0.5, device="cuda"), torch.full((width,), -0.25, device="cuda")
        B.op_layernorm_bwd(dy, x, stats, gamma, res, dx, dg, db, partial)
        got.append((dx, dg, db))
    assert all(torch.equal(a, b) for a, b in zip(*got))
    xd, gd = x.double().requires_grad_(True), gamma.double().requires_grad_(True)
    mu = xd.mean(-1, keepdim=True)
    xh = (xd - mu) / ((xd - mu).square().mean(-1, keepdim=True) + 1e-5).sqrt()
    wx, wg = torch.autograd.grad(xh * gd, (xd, gd), dy.double())
    tol = 2.5e-3 if dtype == torch.bfloat16 else 1e-6
    assert float((got[0][0].double() - wx - res.double()).norm() / (wx + res.double()).norm()) <= tol
    assert float((got[0][1].double() - wg - 0.5).norm() / (wg + 0.5).norm()) <= 1e-5
    assert float((got[0][2].double() - dy.double().sum(0) + 0.25).norm() / (dy.double().sum(0) - 0.25).norm()) <= 1e-5
