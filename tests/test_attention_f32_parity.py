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
