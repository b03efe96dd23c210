"""fp32 attention in tiles of 16: edges of tiles, waves without one, several tiles per wave, every padded head dim; the sizes that stay in tiles of 32."""
import pytest
import torch

from paper_2111_04007_amd import binding as B, synth
from tests import parity_util as U
from tests.test_ops_parity import rnd, run_attention_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,s,heads,d,causal", [
    (256, 1, 1, 64, 1), (16, 15, 2, 32, 0), (8, 16, 2, 60, 1), (8, 17, 3, 28, 1), (2, 64, 2, 64, 1), (2, 65, 3, 100, 0), (3, 130, 2, 96, 1), (1, 300, 4, 68, 0),
    (1, 257, 2, 128, 1), (2, 500, 2, 8, 1), (1, 1000, 1, 4, 0), (9, 64, 1, 128, 1), (1, 300, 16, 64, 0), (1, 300, 16, 120, 0), (2, 200, 20, 128, 0),
])
def test_attention(b, s, heads, d, causal):
    """Same bounds as the other fp32 forms (rel-L2 1e-5, measured 2e-7 .. 8e-7)."""
    run_attention_case("f32", b, s, heads, d, causal, variant=0, seed=30 + d)


def test_rising_row_maxima():
    run_attention_case("f32", 2, 200, 2, 64, 0, variant=0, seed=5, key_ramp=(0.5, 4.0))


@pytest.mark.parametrize("heads,d,s,causal", [(8, 20, 45, True), (4, 64, 130, False), (3, 100, 131, True)])
def test_dropout(heads, d, s, causal):
    cfg = synth.StageConfig("f32-16-dropout", 1, heads * d, heads, s, 2, 1, heads * d, causal, "f32", 0.05, seed=77, dropout_p=0.3)
    params = synth.make_params(cfg, perturb=0.05)
    xs, dys = synth.make_activations(cfg, 1)
    st, ys, dxs = U.gpu_stage_step(cfg, params, xs, dys, seed=3)
    U.compare_step(cfg, st, ys, dxs, U.oracle_stage_step(cfg, params, xs, dys, seed=3), label=f"s={s} d={d}")
    st.close()


@pytest.mark.parametrize("d", [16, 64])
def test_scores_are_those_of_the_row_kernels(d):
    """One visible key and a scale that is a power of two: the log-sum-exp is the scaled score, and the same to the bit in either form."""
    b, heads, s = 600, 1, 1
    qkv = rnd((b, 3 * d), "f32", 3)
    got = []
    for variant in (0, -1):
        ctx, lse = torch.empty(b, d, device="cuda"), torch.empty(b, device="cuda")
        B.op_attention_fwd(qkv, ctx, lse, b, s, heads, d, 1, variant=variant)
        got.append((ctx, lse))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("side", ["key", "value", "gradient"])
def test_what_masked_tokens_hold_stays_out(side, value):
    """An infinity or NaN of a later token reaches no row before it, forward or backward: those equal the clean call's (2e-5: a block with such a row is worked out
    again on one wave a row, whose sums have another order)."""
    b, s, heads, d = 4, 70, 2, 64
    h, bad = heads * d, 40
    qkv, dctx = rnd((b * s, 3 * h), "f32", 5), rnd((b * s, h), "f32", 6)
    dctx.view(b, s, h)[:, bad:] = 0   # so that the clean and the other gradients of earlier keys are the same sums
    got = []
    for spoil in (False, True):
        q, g = qkv.clone(), dctx.clone()
        if spoil and side != "gradient":
            q.view(b, s, 3, heads, d)[:, bad, 1 if side == "key" else 2, :, 3] = value
        if spoil and side == "gradient":
            g.view(b, s, heads, d)[:, bad, :, 3] = value
        ctx, dqkv, lse = torch.empty_like(g), torch.empty_like(q), torch.empty(b * heads * s, device="cuda")
        B.op_attention_fwd(q, ctx, lse, b, s, heads, d, 1)
        B.op_attention_bwd(q, ctx, lse, g, dqkv, torch.empty_like(lse), b, s, heads, d, 1)
        got.append((ctx.view(b, s, h)[:, :bad], lse.view(b, heads, s)[:, :, :bad], dqkv.view(b, s, 3 * h)[:, :bad, :h]))
    for x, y in zip(*got):
        assert float((x - y).abs().max()) <= 2e-5 and bool(torch.isfinite(y).all())
