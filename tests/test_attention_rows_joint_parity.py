"""Row kernels' backward in one launch (up to 1024 rows) and in two: the same gradients against 64 bits on either side of the limit."""
import pytest
import torch

from paper_2111_04007_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("b,heads,s,d", [(1, 1, 1, 4), (2, 2, 64, 64), (1, 3, 37, 40), (4, 8, 32, 99), (33, 1, 31, 7), (33, 1, 32, 7), (1, 2, 130, 256)])
def test_joint_and_separate(dtype, causal, b, heads, s, d):
    """fp32: sums of up to 256 terms, 2e-6 with the cancellation in dP - delta (2e-5 for one token, where dQ and dK vanish); bf16: its rounding."""
    g = torch.Generator(device="cuda").manual_seed(s)
    h = heads * d
    qkv, dctx = (torch.empty(b * s, n, device="cuda").normal_(0, 1, generator=g).to(dtype) for n in (3 * h, h))
    ctx, dqkv = torch.empty_like(dctx), torch.full_like(qkv, 7.0)
    lse, delta = torch.empty(b * heads * s, device="cuda"), torch.full((b * heads * s,), 7.0, device="cuda")
    B.op_attention_fwd(qkv, ctx, lse, b, s, heads, d, causal, variant=-1)
    B.op_attention_bwd(qkv, ctx, lse, dctx, dqkv, delta, b, s, heads, d, causal, variant=-1)
    x = qkv.double().requires_grad_(True)
    q, k, v = (t.reshape(b, s, heads, d).transpose(1, 2).contiguous() for t in x.split(h, 1))
    sc = torch.matmul(q, k.transpose(2, 3).contiguous()) / d ** 0.5
    if causal:
        sc = sc.masked_fill(torch.ones(s, s, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
    out = torch.matmul(sc.softmax(-1), v).transpose(1, 2).reshape(b * s, h)
    want, = torch.autograd.grad(out, x, dctx.double())
    tol = 2e-6 if dtype == torch.float32 else 4e-3
    assert float((dqkv.double() - want).norm() / want.norm()) <= (2e-5 if s == 1 and dtype == torch.float32 else tol)
    rows = (dctx.double() * ctx.double()).reshape(b, s, heads, d).sum(-1).transpose(1, 2).reshape(-1)
    assert float((delta.double() - rows).abs().max()) <= 1e-6 * d ** 0.5 * float(dctx.double().abs().max() * ctx.double().abs().max() + 1)
