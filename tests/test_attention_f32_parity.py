"""Attention with fp32 products on the matrix cores: tile and vector-load remainders, idle waves, both operand types."""
import pytest

from paper_2111_04007_amd import synth
from tests import parity_util as U
from tests.test_ops_parity import run_attention_case

pytestmark = pytest.mark.gpu

# 32-row tiles shared by 4 waves: fewer tiles than waves, one to three tiles per wave; head dims on both sides of every padding
SHAPES = [(1, 1, 1, 4, 1), (2, 31, 2, 32, 0), (1, 33, 1, 36, 1), (1, 64, 3, 64, 1), (2, 127, 1, 68, 0), (1, 129, 2, 96, 1),
          (1, 160, 1, 100, 1), (1, 257, 1, 128, 0), (3, 300, 1, 24, 1), (1, 70, 2, 7, 0), (1, 97, 1, 35, 1), (1, 40, 1, 127, 0)]


@pytest.mark.parametrize("b,s,heads,d,causal", SHAPES)
def test_attention_fp32_products_f32(b, s, heads, d, causal):
    """rel-L2 1e-5 (measured 2e-7 .. 5e-7), log-sum-exp 1e-4."""
    run_attention_case("f32", b, s, heads, d, causal, variant=3, seed=80 + d)


@pytest.mark.parametrize("b,s,heads,d,causal", SHAPES)
def test_attention_fp32_products_bf16(b, s, heads, d, causal):
    run_attention_case("bf16", b, s, heads, d, causal, variant=3, seed=90 + d)


def test_attention_fp32_rising_row_maxima():
    """Each wave's running maximum keeps rising and the waves' maxima differ: the combination must rescale all four."""
    run_attention_case("f32", 1, 400, 2, 64, 0, variant=0, seed=5, key_ramp=(0.5, 4.0))


@pytest.mark.parametrize("heads,d,s,causal", [(3, 20, 45, True), (2, 64, 132, False)])
def test_dropout_fp32(heads, d, s, causal):
    cfg = synth.StageConfig("f32-dropout", 1, heads * d, heads, s, 2, 1, 2 * heads * d, causal, "f32", 0.05, seed=77, dropout_p=0.3)
    params = synth.make_params(cfg, perturb=0.05)
    xs, dys = synth.make_activations(cfg, 1)
    st, ys, dxs = U.gpu_stage_step(cfg, params, xs, dys, seed=3)
    U.compare_step(cfg, st, ys, dxs, U.oracle_stage_step(cfg, params, xs, dys, seed=3), label=f"s={s} d={d}")
    st.close()


@pytest.mark.parametrize("dtype,b,s,heads,d,fwd,bwd", [
    ("f32", 1, 64, 8, 128, -1, -1), ("f32", 4, 64, 16, 128, 3, 3), ("f32", 1, 193, 1, 128, 3, 3), ("f32", 1, 64, 2, 64, 3, -1), ("f32", 1, 65, 2, 64, 3, 3),
    ("f32", 1, 256, 2, 63, -1, -1), ("f32", 2, 257, 16, 63, 3, 3), ("f32", 1, 33, 1, 32, 3, -1), ("f32", 1, 32, 2, 16, -1, -1),
    ("bf16", 1, 48, 4, 20, 3, -1), ("bf16", 1, 64, 16, 92, -1, -1), ("bf16", 1, 70, 2, 92, 3, 3), ("bf16", 1, 192, 1, 127, -1, -1), ("bf16", 1, 200, 1, 127, 3, 3),
    ("bf16", 1, 100, 2, 7, 3, 3),
])
def test_short_rows_go_to_the_row_kernels(dtype, b, s, heads, d, fwd, bwd):
    """Both sides of the lines between the two forms: the library's choice is, bit for bit, the form named here."""
    import torch
    from paper_2111_04007_amd import binding as B
    from tests.test_ops_parity import rnd
    h = heads * d
    qkv, dctx = rnd((b * s, 3 * h), dtype, 7), rnd((b * s, h), dtype, 8)
    got = []
    for vf, vb in ((0, 0), (fwd, bwd)):
        ctx, dqkv, lse = torch.empty_like(dctx), torch.empty_like(qkv), torch.empty(b * heads * s, device="cuda")
        B.op_attention_fwd(qkv, ctx, lse, b, s, heads, d, 1, variant=vf)
        B.op_attention_bwd(qkv, ctx, lse, dctx, dqkv, torch.empty_like(lse), b, s, heads, d, 1, variant=vb)
        got.append((ctx, lse, dqkv))
    assert all(torch.equal(x, y) for x, y in zip(*got))


@pytest.mark.parametrize("dtype,variant,b,s,heads,d,causal,peak", [
    ("f32", 3, 2, 130, 4, 112, 0, 4), ("f32", 3, 2, 130, 4, 112, 0, 16), ("f32", 3, 1, 90, 2, 80, 1, 16), ("f32", 3, 2, 333, 3, 40, 1, 4),
    ("f32", 3, 1, 1500, 1, 64, 1, 16), ("f32", 0, 2, 130, 4, 112, 0, 16), ("f32", 0, 2, 64, 2, 64, 1, 16), ("bf16", 2, 2, 333, 3, 40, 1, 4), ("bf16", 2, 1, 1000, 2, 72, 1, 1),
])
def test_no_further_from_64_bits_than_the_row_kernels(dtype, variant, b, s, heads, d, causal, peak):
    """Softmax rows flat and peaked (queries `peak` times as long).  Both forms round scores, exponents and sums in fp32; their errors
    are samples of the same size, 15 % apart at most on these many values.  The log-sum-exp may differ
    by the rounding of the scale (2^-24 of the score, a constant of d and the form) and of the result (2^-24 / sqrt(3)).  Variant 0
    mixes the forms: forward and backward of one call choose by themselves."""
    import torch
    from paper_2111_04007_amd import binding as B
    from tests.test_ops_parity import DT, rnd
    h = heads * d
    qkv, dctx = rnd((b * s, 3 * h), "f32", 11), rnd((b * s, h), dtype, 12)
    qkv[:, :h] *= peak
    qkv = qkv.to(DT[dtype])
    x = qkv.double().requires_grad_(True)
    q, k, v = (t.reshape(b, s, heads, d).transpose(1, 2).contiguous() for t in x.split(h, 1))
    sc = torch.matmul(q, k.transpose(2, 3).contiguous()) / d ** 0.5
    if causal:
        sc = sc.masked_fill(torch.ones(s, s, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
    want = torch.matmul(sc.softmax(-1), v).transpose(1, 2).reshape(-1, h)
    dwant, = torch.autograd.grad(want, x, dctx.double())
    errs = []
    for vn in (variant, -1):
        ctx, dqkv, lse = torch.empty_like(dctx), torch.empty_like(qkv), torch.empty(b * heads * s, device="cuda")
        B.op_attention_fwd(qkv, ctx, lse, b, s, heads, d, causal, variant=vn)
        B.op_attention_bwd(qkv, ctx, lse, dctx, dqkv, torch.empty_like(lse), b, s, heads, d, causal, variant=vn)
        pairs = [(ctx, want.detach()), (lse, sc.detach().logsumexp(-1).reshape(-1))] + [(dqkv[:, i * h:(i + 1) * h], dwant[:, i * h:(i + 1) * h]) for i in range(3)]
        errs.append([float((g.double() - w).norm() / w.norm()) for g, w in pairs])
    for i, (new, row) in enumerate(zip(*errs)):
        assert new <= max(1.15 * row, 2.0 ** -24 * 1.6 if i == 1 else 0.0), (("ctx", "lse", "dq", "dk", "dv")[i], new, row)
