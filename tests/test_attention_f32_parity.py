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
