"""The bf16 MFMA attention kernels on sequence lengths and head dims that fit no tile (EDGE form)."""
import pytest
import torch

from paper_2111_04007_amd import binding as B, synth
from tests import parity_util as U
from tests.test_ops_parity import rnd, run_attention_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,s,heads,d,causal", [
    (1, 1, 1, 8, 1), (2, 33, 3, 24, 0), (1, 64, 2, 32, 1), (2, 63, 1, 40, 1), (1, 65, 2, 64, 0), (1, 127, 1, 72, 1),
    (1, 129, 2, 96, 1), (2, 191, 1, 104, 0), (1, 200, 1, 128, 1), (1, 257, 2, 120, 0), (3, 130, 2, 64, 1), (1, 256, 1, 48, 0),
])
def test_attention_edge(b, s, heads, d, causal):
    """Same bound as the whole-tile kernels' tests; one to three blocks of queries and keys, every padded head dim."""
    run_attention_case("bf16", b, s, heads, d, causal, variant=2, seed=50 + d)


def test_attention_edge_agrees_with_whole_tiles():
    """On shapes both forms take they differ by the rounding of the probabilities and score gradients to bf16 (2^-9 each,
    averaged over a row's keys) and by the rounding of the outputs (2^-9 / sqrt(3) rms): 2^-8 covers both."""
    for b, s, heads, d, causal in ((1, 256, 2, 64, 1), (2, 128, 1, 96, 0), (1, 256, 1, 128, 1)):
        h = heads * d
        qkv, dctx = rnd((b * s, 3 * h), "bf16", 7), rnd((b * s, h), "bf16", 8)
        got = []
        for v in (1, 2):
            ctx, dqkv = torch.empty_like(dctx), torch.empty_like(qkv)
            lse = torch.empty(b * heads * s, device="cuda")
            delta = torch.empty_like(lse)
            B.op_attention_fwd(qkv, ctx, lse, b, s, heads, d, causal, variant=v)
            B.op_attention_bwd(qkv, ctx, lse, dctx, dqkv, delta, b, s, heads, d, causal, variant=v)
            got.append((ctx, lse, dqkv))
        for x, y in zip(*got):
            assert float((x.double() - y.double()).norm() / x.double().norm()) <= 2.0 ** -8


def test_attention_edge_stays_inside_its_tensors():
    """Tensors end where a guard begins: NaNs behind the inputs must not spread, values behind the outputs must stay."""
    b, s, heads, d = 2, 77, 3, 40
    h, T = heads * d, b * s

    def guarded(n, fill, src=None):
        buf = torch.full((n + 65536,), fill, dtype=torch.bfloat16, device="cuda")
        if src is not None:
            buf[:n] = src.reshape(-1)
        return buf

    qkv, dctx = guarded(T * 3 * h, float("nan"), rnd((T, 3 * h), "bf16", 1)), guarded(T * h, float("nan"), rnd((T, h), "bf16", 2))
    ctx, dqkv = guarded(T * h, 3.0), guarded(T * 3 * h, 3.0)
    lse, delta = (torch.full((b * heads * s + 4096,), 5.0, device="cuda") for _ in range(2))
    for causal in (0, 1):
        B.op_attention_fwd(qkv, ctx, lse, b, s, heads, d, causal, variant=2)
        B.op_attention_bwd(qkv, ctx, lse, dctx, dqkv, delta, b, s, heads, d, causal, variant=2)
        for t, n, fill in ((ctx, T * h, 3.0), (dqkv, T * 3 * h, 3.0), (lse, b * heads * s, 5.0), (delta, b * heads * s, 5.0)):
            assert bool(torch.isfinite(t[:n]).all()) and bool((t[n:] == fill).all())


@pytest.mark.parametrize("s,d,causal", [(132, 40, True), (70, 64, False), (131, 96, True), (45, 128, True)])
def test_dropout_edge(s, d, causal):
    """Dropout masks at lengths that are and are not multiples of the 4x4 mask patches, against the oracle's generator."""
    cfg = synth.StageConfig("edge-dropout", 1, 3 * d, 3, s, 2, 1, 6 * d, causal, "bf16", 0.02, seed=60 + s, dropout_p=0.3)
    params = synth.make_params(cfg, perturb=0.05)
    xs, dys = synth.make_activations(cfg, 1)
    st, ys, dxs = U.gpu_stage_step(cfg, params, xs, dys, seed=9)
    U.compare_step(cfg, st, ys, dxs, U.oracle_stage_step(cfg, params, xs, dys, seed=9), label=f"s={s} d={d}")
    st.close()


@pytest.mark.parametrize("s,causal", [(220, False), (220, True), (333, False)])
def test_dropout_edge_many_heads_of_32(s, causal):
    """Enough waves for products to follow their operands' conversions without a gap: what dK multiplied before the last
    conversion had landed was an fp32 number's lower half, up to 1e38."""
    cfg = synth.StageConfig("edge-dropout-32", 1, 704, 22, s, 6, 1, 704, causal, "bf16", 0.02, seed=90 + s, dropout_p=0.1)
    params = synth.make_params(cfg, perturb=0.05)
    xs, dys = synth.make_activations(cfg, 1)
    want = U.oracle_stage_step(cfg, params, xs, dys, seed=9)
    for _ in range(3):
        st, ys, dxs = U.gpu_stage_step(cfg, params, xs, dys, seed=9)
        U.compare_step(cfg, st, ys, dxs, want, label=f"s={s}")
        st.close()


@pytest.mark.parametrize("variant,d", [(2, 20), (2, 136), (3, 136), (7, 64)])
def test_other_forms_leave_shapes_they_do_not_take_to_the_row_kernels(variant, d):
    b, s, heads = 1, 37, 2
    qkv, dctx = rnd((b * s, 3 * heads * d), "bf16", 7), rnd((b * s, heads * d), "bf16", 8)
    got = []
    for v in (variant, -1):
        ctx, dqkv, lse = torch.empty_like(dctx), torch.empty_like(qkv), torch.empty(b * heads * s, device="cuda")
        B.op_attention_fwd(qkv, ctx, lse, b, s, heads, d, 1, variant=v)
        B.op_attention_bwd(qkv, ctx, lse, dctx, dqkv, torch.empty_like(lse), b, s, heads, d, 1, variant=v)
        got.append((ctx, lse, dqkv))
    assert all(torch.equal(x, y) for x, y in zip(*got))


@pytest.mark.parametrize("b,s,heads,d,causal", [(1, 500, 2, 64, 0), (1, 333, 1, 128, 1), (1, 390, 1, 40, 0), (1, 450, 2, 72, 1)])
def test_attention_edge_rising_row_maxima(b, s, heads, d, causal):
    """Both branches of the thresholded rescale after the first block, as for the whole tiles."""
    run_attention_case("bf16", b, s, heads, d, causal, variant=2, seed=70 + d, key_ramp=(0.5, 4.0))


@pytest.mark.parametrize("variant,b,s,heads,d,causal", [
    (2, 2, 31, 1, 64, 1), (2, 1, 32, 2, 128, 0), (2, 2, 97, 1, 96, 1), (2, 1, 161, 2, 128, 1), (2, 2, 225, 1, 32, 0), (2, 1, 289, 2, 88, 0),
    (1, 2, 128, 3, 64, 0), (1, 1, 384, 1, 96, 1), (1, 2, 256, 2, 128, 1), (1, 1, 512, 1, 128, 0),
])
def test_attention_steps_of_32_queries(variant, b, s, heads, d, causal):
    """The key side walks 32 queries at a time, last to first: one step, a last step of one row, first and last waves that start or
    end elsewhere than their workgroup.  Same bound as the other shapes."""
    run_attention_case("bf16", b, s, heads, d, causal, variant=variant, seed=110 + d)


@pytest.mark.parametrize("d", [64, 96, 128])
def test_attention_on_whole_tiles_takes_any_alignment(d):
    """Tensors that start at an odd element: bit for bit the results of aligned ones."""
    b, s, heads = 1, 128, 2
    T, h = b * s, heads * d

    def shifted(t):
        buf = torch.empty(t.numel() + 9, dtype=t.dtype, device="cuda")
        buf[1:1 + t.numel()] = t.reshape(-1)
        return buf[1:1 + t.numel()].view(t.shape)

    qkv, dctx = rnd((T, 3 * h), "bf16", 3), rnd((T, h), "bf16", 4)
    got = []
    for q, g in ((qkv, dctx), (shifted(qkv), shifted(dctx))):
        ctx, dqkv, lse = torch.empty_like(dctx), torch.empty_like(qkv), torch.empty(heads * s, device="cuda")
        B.op_attention_fwd(q, ctx, lse, b, s, heads, d, 1, variant=1)
        B.op_attention_bwd(q, ctx, lse, g, dqkv, torch.empty_like(lse), b, s, heads, d, 1, variant=1)
        got.append((ctx, lse, dqkv))
    assert all(torch.equal(x, y) for x, y in zip(*got))


@pytest.mark.parametrize("b,s,heads,d,causal", [(1, 33, 1, 64, 1), (1, 70, 2, 96, 0), (2, 129, 2, 128, 1), (1, 1000, 1, 40, 1)])
def test_statistics_past_the_last_query_are_not_read(b, s, heads, d, causal):
    """The last tile of 32 queries is partly filled.  What lies behind the log-sum-exps and the deltas (here NaN) has no part in it, and neither
    have those of the next head, which hold a NaN: the same bits as without either."""
    h, n = heads * d, b * heads * s
    qkv, dctx = rnd((b * s, 3 * h), "bf16", 3), rnd((b * s, h), "bf16", 4)
    got = []
    for behind in (0.0, float("nan")):
        ctx, dqkv = torch.empty_like(dctx), torch.empty_like(qkv)
        lse, delta = (torch.full((n + 64,), behind, device="cuda") for _ in range(2))
        B.op_attention_fwd(qkv, ctx, lse, b, s, heads, d, causal, variant=2)
        if heads > 1:
            lse.view(-1)[s:s + 31] += behind   # the second head of the first sequence, its first 31 queries
        B.op_attention_bwd(qkv, ctx, lse, dctx, dqkv, delta, b, s, heads, d, causal, variant=2)
        got.append((lse[:s], delta[:s], dqkv[:s].view(s, 3, heads, d)[:, :, 0].clone()))
    assert all(torch.equal(x, y) for x, y in zip(*got))
