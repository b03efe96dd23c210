"""Calls whose number of blocks times threads passes 2^32 in one grid dimension of the usual kernels."""
import pytest
import torch

from paper_2111_04007_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 8), (torch.bfloat16, 3), (torch.float32, 4)])
def test_attention_with_more_than_2_24_heads(dtype, d):
    """16.8 million sequences of one token: the context is V, dV is the upstream gradient, dQ and dK vanish."""
    b, heads = 65535, 257
    h = heads * d
    g = torch.Generator(device="cuda").manual_seed(1)
    qkv = torch.empty((b, 3 * h), dtype=dtype, device="cuda").normal_(generator=g)
    dctx = torch.empty((b, h), dtype=dtype, device="cuda").normal_(generator=g)
    ctx, dqkv = torch.full_like(dctx, 7.0), torch.full_like(qkv, 7.0)
    lse = torch.empty(b * heads, device="cuda")
    delta = torch.empty_like(lse)
    B.op_attention_fwd(qkv, ctx, lse, b, 1, heads, d, 1)
    assert torch.equal(ctx, qkv[:, 2 * h:])
    B.op_attention_bwd(qkv, ctx, lse, dctx, dqkv, delta, b, 1, heads, d, 1)
    assert torch.equal(dqkv[:, 2 * h:], dctx)
    # dP - delta is the difference of two orders of one sum of d products: 2^-24 of it each, times values of a few units
    assert float(dqkv[:, :2 * h].abs().max()) <= 1e-4


@pytest.mark.parametrize("dtype,M,N", [(torch.float32, (1 << 28) + 40, 1), (torch.bfloat16, (1 << 28) + 40, 1), (torch.float32, 3, (1 << 28) + 33)])
def test_gemm_of_more_than_2_23_tiles(dtype, M, N):
    """One-term products, so every output has one rounding: the tall and the wide side of 32x32 tiles."""
    g = torch.Generator(device="cuda").manual_seed(2)
    x, w, bias = (torch.empty(n, dtype=dtype, device="cuda").normal_(generator=g) for n in ((M, 1), (N, 1), (N,)))
    out = torch.full((M, N), 7.0, dtype=dtype, device="cuda")
    B.op_gemm(B.OP_FWD, 0, x, w, out, bias=bias, M=M, N=N, K=1)
    for lo in range(0, max(M, N), 1 << 26):   # (the reference in pieces)
        rows, cols = (slice(lo, lo + (1 << 26)), slice(None)) if M > N else (slice(None), slice(lo, lo + (1 << 26)))
        want = torch.addcmul(bias[cols].float()[None], x[rows].float(), w[cols].float().t())
        assert float((out[rows, cols].float() - want).abs().max()) <= (2.0 ** -18 if dtype == torch.float32 else 2.0 ** -4)
        assert float((out[rows, cols].float() - want).norm() / want.norm()) <= (2.0 ** -22 if dtype == torch.float32 else 2.0 ** -8)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_colsum_of_more_than_2_29_columns(dtype):
    n = (1 << 30) + 256 if dtype == torch.bfloat16 else (1 << 29) + 128
    a = torch.empty((1, n), dtype=dtype, device="cuda").normal_(generator=torch.Generator(device="cuda").manual_seed(3))
    out = torch.ones(n, device="cuda")
    B.op_colsum(a, out, torch.empty(B.colreduce_scratch_bytes(1, n) // 4, device="cuda"))
    for lo in range(0, n, 1 << 27):   # one addition
        assert torch.equal(out[lo:lo + (1 << 27)], a[0, lo:lo + (1 << 27)].float() + 1.0)
