"""Forms of the row-in-registers LayerNorm forward: one to sixteen 16-byte pieces per lane, gamma and beta fetched early or late
(by the number of rows)."""
import pytest
import torch

from paper_2111_04007_amd import binding as B
from tests.test_ops_parity import rnd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,rows,h", [
    ("bf16", 9, 512), ("bf16", 9, 520), ("bf16", 11, 2056), ("bf16", 3072, 4096), ("bf16", 3073, 2056), ("bf16", 5121, 2064), ("bf16", 6, 8192),
    ("f32", 9, 256), ("f32", 9, 260), ("f32", 11, 1028), ("f32", 3073, 2048), ("f32", 7168, 1028), ("f32", 7169, 1028), ("f32", 6, 4096),
])
def test_layernorm_forward_forms(dtype, rows, h):
    """fp32 arithmetic: 1e-6 (two sums over a row, 2^-24 sqrt(h) each at most), bf16 the rounding of the result (2^-9 / sqrt(3))."""
    x, gamma, beta = rnd((rows, h), dtype, 3, 2.0) + 0.5, (rnd((h,), dtype, 4, 0.2) + 1.0), rnd((h,), dtype, 5, 0.2)
    y, stats = torch.empty_like(x), torch.empty(2 * rows, device="cuda")
    B.op_layernorm_fwd(x, gamma, beta, y, stats)
    xd = x.double()
    mu, rs = xd.mean(1), 1 / (xd.var(1, unbiased=False) + 1e-5).sqrt()
    want = gamma.double() * (xd - mu[:, None]) * rs[:, None] + beta.double()
    assert float((y.double() - want).norm() / want.norm()) <= (1e-6 if dtype == "f32" else 2e-3)
    assert float((stats.double() - torch.cat([mu, rs])).norm() / torch.cat([mu, rs]).norm()) <= 1e-6
