"""Attention on inputs that hold infinities and NaNs: a row reads only the tokens its mask admits, on every kernel form the
library picks.  The reference is the kernel that works row by row (variant -1)."""
import pytest
import torch

from paper_2111_04007_amd import binding as B, synth
from tests import parity_util as U
from tests.test_ops_parity import TOL, rnd

pytestmark = pytest.mark.gpu
INF, NAN = float("inf"), float("nan")

# fp32 products (fp32, and bf16 with an odd head dim) and the EDGE form (bf16), every padded head dim, causal and not;
# lengths of one to five key tiles
FORMS = [("f32", 1, 70, 2, 64, 1), ("f32", 2, 129, 1, 20, 1), ("f32", 1, 100, 1, 96, 0), ("f32", 1, 131, 1, 128, 1), ("bf16", 1, 75, 2, 7, 1),
         ("bf16", 1, 70, 2, 64, 1), ("bf16", 2, 129, 1, 32, 1), ("bf16", 1, 100, 1, 96, 0), ("bf16", 1, 200, 1, 128, 1), ("bf16", 1, 300, 2, 40, 1)]


def same(got, want, tol, what):
    got, want = got.double(), want.double()
    for kind in (torch.isnan, torch.isposinf, torch.isneginf):
        assert torch.equal(kind(got), kind(want)), (what, kind.__name__)
    ok = torch.isfinite(want)
    assert bool(ok.any()), what
    assert float((got - want)[ok].norm()) <= tol * float(want[ok].norm()), what


def forward(qkv, dims, variant):
    b, s, heads, d, causal = dims
    ctx = torch.empty((b * s, heads * d), dtype=qkv.dtype, device="cuda")
    lse = torch.empty(b * heads * s, device="cuda")
    B.op_attention_fwd(qkv, ctx, lse, b, s, heads, d, causal, variant=variant)
    return ctx, lse


def backward(qkv, ctx, lse, dctx, dims, variant):
    b, s, heads, d, causal = dims
    dqkv, delta = torch.empty_like(qkv), torch.empty_like(lse)
    B.op_attention_bwd(qkv, ctx, lse, dctx, dqkv, delta, b, s, heads, d, causal, variant=variant)
    return dqkv


@pytest.mark.parametrize("dtype,b,s,heads,d,causal", FORMS)
@pytest.mark.parametrize("where", ["q", "k", "v", "dctx"])
def test_one_token_that_is_not_finite(where, dtype, b, s, heads, d, causal):
    """One token's row of Q, K, V or the upstream gradient, the forward results of the backward pass from finite inputs."""
    if where == "k" and not causal:
        return   # every row of the head sees the key: nothing finite is left to compare
    dims, h, tol = (b, s, heads, d, causal), heads * d, TOL[dtype]
    qkv, dctx = rnd((b * s, 3 * h), dtype, 11 + d), rnd((b * s, h), dtype, 12 + d)
    ctx, lse = forward(qkv, dims, -1)
    for token in (s // 2 + 1, s - 2):
        bad, g = qkv.clone(), dctx.clone()
        row = g[token] if where == "dctx" else bad[token, "qkv".index(where) * h:]
        row[0], row[1], row[2] = INF, NAN, -INF
        if where != "dctx":
            same_fwd = [forward(bad, dims, v) for v in (0, -1)]
            same(same_fwd[0][0], same_fwd[1][0], tol, "ctx")
            same(same_fwd[0][1], same_fwd[1][1], 1e-5, "log-sum-exp")
        got, want = (backward(bad, ctx, lse, g, dims, v) for v in (0, -1))
        if where == "dctx" and not causal:   # every key sees it: the finite part that is left is dQ of the other tokens
            got, want = got[:, :h], want[:, :h]
        same(got, want, tol, where)


@pytest.mark.parametrize("dtype,b,s,heads,d", [("f32", 1, 65, 1, 64), ("f32", 1, 97, 2, 24), ("bf16", 1, 65, 1, 64), ("bf16", 1, 129, 1, 104), ("bf16", 1, 65, 1, 9)])
def test_key_that_no_query_attends_to(dtype, b, s, heads, d):
    """A key whose every score is -inf, alone in its tile: its weight is 0 and its value row has no part in the result."""
    h = heads * d
    qkv = rnd((b * s, 3 * h), dtype, 5)
    qkv[:, :h] = qkv[:, :h].abs() + 0.125
    qkv[s - 1, h:2 * h] = -INF
    got, want = (forward(qkv, (b, s, heads, d, 0), v) for v in (0, -1))
    assert bool(torch.isfinite(want[0]).all())
    same(got[0], want[0], TOL[dtype], "ctx")
    same(got[1], want[1], 1e-5, "log-sum-exp")


@pytest.mark.parametrize("dtype,heads,d,s,drop", [("f32", 2, 40, 150, 0.0), ("f32", 2, 32, 90, 0.3), ("bf16", 3, 40, 150, 0.0), ("bf16", 2, 32, 91, 0.3)])
def test_stage_forward_is_causal(dtype, heads, d, s, drop):
    """A token that is not finite leaves the outputs of the tokens before it as they are without it."""
    cfg = synth.StageConfig("causal", 2, heads * d, heads, s, 1, 1, 4 * heads * d, True, dtype, 0.05, seed=s, dropout_p=drop)
    st = B.Stage(cfg)
    st.set_params(synth.make_params(cfg, perturb=0.05))
    st.set_dropout_seed(5)
    x = synth.make_activations(cfg, 1)[0][0].cuda()
    clean, y = torch.empty_like(x), torch.empty_like(x)
    st.forward(0, x, clean)
    token = s - s // 3
    x[token, 3] = NAN
    st.forward(0, x, y)
    assert bool(torch.isnan(y[token]).any())
    same(y[:token], clean[:token], U.TOL[dtype], "outputs before the token")
    st.close()


@pytest.mark.parametrize("d", [64, 96, 128])
@pytest.mark.parametrize("value", [INF, NAN])
def test_masked_query_on_whole_tiles(d, value):
    """Whole tiles: a query that is not finite, and with it its log-sum-exp, has no part in dV of the keys after it nor in dQ of other queries, in the
    diagonal tile it lies in either: the bits of a clean call."""
    s, heads = 256, 2
    h, dims = heads * d, (1, s, heads, d, 1)
    qkv, dctx = rnd((s, 3 * h), "bf16", 11 + d), rnd((s, h), "bf16", 12 + d)
    clean = backward(qkv, *forward(qkv, dims, 1), dctx, dims, 1)
    for token in (40, 200):
        bad = qkv.clone()
        bad[token, 3] = value
        got = backward(bad, *forward(bad, dims, 1), dctx, dims, 1)
        assert torch.equal(got[token + 1:, 2 * h:], clean[token + 1:, 2 * h:])
        assert torch.equal(got[:token, :h], clean[:token, :h]) and torch.equal(got[token + 1:, :h], clean[token + 1:, :h])
