"""fp32 attention by form: one wave per row (-1), tiles of 16 (4), tiles of 32 (5).  Which one the library's choice is, and on either tile size rows whose maxima
rise, values that are not finite and dropout."""
import pytest
import torch

from paper_2111_04007_amd import binding as B, synth
from tests import parity_util as U
from tests.test_attention_nonfinite_parity import INF, NAN, TOL, backward, forward, same
from tests.test_ops_parity import rnd, run_attention_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,s,heads,d,causal,fwd,bwd", [
    # the smallest calls: up to 128 rows, 512 above d = 64
    (1, 64, 2, 64, 1, 4, -1), (1, 65, 2, 64, 1, 4, 4), (1, 33, 1, 32, 1, 4, -1), (1, 32, 2, 16, 1, -1, -1), (1, 43, 3, 64, 1, 4, 4),
    (1, 64, 8, 128, 1, -1, -1), (1, 64, 9, 128, 1, 4, 4), (1, 171, 3, 96, 1, 4, 4), (1, 193, 1, 128, 1, 4, 4), (4, 64, 16, 128, 1, 4, 4),
    # rows of a few tokens, by the number of heads
    (33, 1, 4, 32, 1, 4, -1), (33, 2, 4, 32, 0, 4, 4), (33, 2, 4, 64, 0, 4, -1), (33, 3, 4, 64, 1, 4, 4), (75, 2, 4, 128, 1, -1, -1), (75, 3, 4, 128, 0, 4, -1),
    (64, 2, 17, 32, 0, -1, 4), (64, 3, 24, 32, 1, 4, -1), (64, 3, 17, 64, 0, -1, -1), (64, 4, 17, 64, 1, 4, -1), (64, 5, 17, 64, 1, 4, 4),
    (64, 3, 13, 96, 1, -1, -1), (64, 8, 13, 96, 0, 4, -1), (64, 9, 13, 96, 1, 4, 4), (8, 5, 16, 96, 1, 4, 4), (3, 4, 43, 128, 0, 4, -1), (64, 5, 13, 128, 1, 4, -1),
    # unmasked rows in equal and in fewer rounds; head dims in single elements
    (8, 330, 2, 64, 0, 5, 4), (5, 330, 5, 64, 0, 4, 4), (3, 330, 9, 64, 0, 5, 4), (3, 900, 7, 64, 0, 4, 4), (3, 912, 7, 64, 0, 5, 4), (8, 320, 2, 64, 0, 4, 4), (8, 330, 2, 64, 1, 4, 4),
    (32, 512, 4, 32, 0, 5, 4), (30, 512, 4, 32, 0, 4, 4), (1, 512, 16, 96, 0, 4, 4), (8, 330, 2, 100, 0, 4, 5), (4, 384, 5, 128, 0, 4, 5), (7, 384, 5, 128, 0, 4, 4),
    (14, 512, 8, 128, 0, 4, 5), (16, 512, 8, 128, 0, 4, 4), (1, 256, 2, 63, 1, -1, -1), (2, 257, 16, 63, 1, 5, 5),
    # many heads on an XCD
    (30, 512, 8, 32, 1, 4, 4), (32, 512, 8, 32, 1, 5, 4), (45, 416, 1, 32, 1, 4, 4), (47, 416, 1, 32, 1, 5, 4), (47, 400, 1, 32, 1, 4, 4),
    (5, 1600, 5, 64, 1, 4, 4), (5, 1616, 5, 64, 1, 5, 4), (5, 700, 7, 64, 1, 4, 4), (5, 704, 7, 64, 1, 5, 4), (47, 350, 1, 64, 1, 4, 4), (47, 352, 1, 64, 1, 5, 4), (45, 384, 8, 64, 1, 4, 4), (46, 384, 8, 64, 1, 5, 4),
    (9, 224, 7, 64, 0, 4, 4), (9, 232, 7, 64, 0, 5, 4), (9, 232, 5, 64, 0, 4, 4), (15, 232, 5, 32, 0, 4, 4), (11, 232, 7, 32, 0, 5, 4),
    (170, 256, 8, 64, 0, 5, 4), (171, 256, 8, 64, 0, 5, 5), (268, 256, 8, 32, 0, 5, 4), (269, 256, 8, 32, 0, 5, 5),
])
def test_which_form_the_choice_is(b, s, heads, d, causal, fwd, bwd):
    """The library's choice is, bit for bit, the form named here, and not the nearest other one (for tiles of 16 one wave per row up to 32 tokens and tiles of 32
    beyond, for these two tiles of 16): the forms sum in other orders."""
    qkv, dctx, dims = rnd((b * s, 3 * heads * d), "f32", 7), rnd((b * s, heads * d), "f32", 8), (b, s, heads, d, causal)
    rows = forward(qkv, dims, -1)   # one forward for every backward

    def call(vf, vb):
        return *forward(qkv, dims, vf), backward(qkv, *rows, dctx, dims, vb)

    got = call(0, 0)
    assert all(torch.equal(x, y) for x, y in zip(got, call(fwd, bwd)))
    if d % 4 == 0:
        other = call(*(-1 if v == 4 and s <= 32 else 5 if v == 4 else 4 for v in (fwd, bwd)))
        assert not torch.equal(got[2], other[2]) and (s == 1 or not torch.equal(got[0], other[0]))


@pytest.mark.parametrize("variant", [4, 5])
def test_rising_row_maxima(variant):
    """Each wave's running maximum keeps rising and the waves' maxima differ: the combination must rescale all four."""
    run_attention_case("f32", 1, 400, 2, 64, 0, variant=variant, seed=5, key_ramp=(0.5, 4.0))


@pytest.mark.parametrize("heads,d,s,causal", [
    (2, 64, 330, False),    # forward in tiles of 32, backward of 16
    (2, 100, 330, False),   # and the other way round
    (2, 64, 66, True),      # both of 16
    (2, 35, 132, False),    # both of 32
])
def test_dropout(heads, d, s, causal):
    cfg = synth.StageConfig("f32-forms-dropout", 1, heads * d, heads, s, 8, 1, 2 * heads * d, causal, "f32", 0.05, seed=77, dropout_p=0.3)
    params = synth.make_params(cfg, perturb=0.05)
    xs, dys = synth.make_activations(cfg, 1)
    st, ys, dxs = U.gpu_stage_step(cfg, params, xs, dys, seed=3)
    U.compare_step(cfg, st, ys, dxs, U.oracle_stage_step(cfg, params, xs, dys, seed=3), label=f"s={s} d={d}")
    st.close()


@pytest.mark.parametrize("variant", [4, 5])
@pytest.mark.parametrize("b,s,heads,d,causal", [(1, 70, 2, 64, 1), (2, 129, 1, 20, 1), (1, 100, 1, 96, 0), (1, 131, 1, 128, 1)])
@pytest.mark.parametrize("where", ["q", "v", "dctx"])
def test_one_token_that_is_not_finite(where, b, s, heads, d, causal, variant):
    """One token's row of Q, V or the upstream gradient, against one wave per row (rel-L2 1e-5 of what is finite)."""
    dims, h = (b, s, heads, d, causal), heads * d
    qkv, dctx = rnd((b * s, 3 * h), "f32", 11 + d), rnd((b * s, h), "f32", 12 + d)
    ctx, lse = forward(qkv, dims, -1)
    for token in (s // 2 + 1, s - 2):
        bad, g = qkv.clone(), dctx.clone()
        row = g[token] if where == "dctx" else bad[token, "qkv".index(where) * h:]
        row[0], row[1], row[2] = INF, NAN, -INF
        if where != "dctx":
            for got, want, what in zip(forward(bad, dims, variant), forward(bad, dims, -1), ("ctx", "log-sum-exp")):
                same(got, want, TOL["f32"], what)
        got, want = (backward(bad, ctx, lse, g, dims, v) for v in (variant, -1))
        if where == "dctx" and not causal:   # every key sees it: the finite part that is left is dQ of the other tokens
            got, want = got[:, :h], want[:, :h]
        same(got, want, TOL["f32"], where)


@pytest.mark.parametrize("variant", [4, 5])
@pytest.mark.parametrize("s,heads,d", [(65, 1, 64), (97, 2, 24)])
def test_key_that_no_query_attends_to(s, heads, d, variant):
    """A key whose every score is -inf, alone in its tile: its weight is 0 and its value row has no part in the result."""
    h = heads * d
    qkv = rnd((s, 3 * h), "f32", 5)
    qkv[:, :h] = qkv[:, :h].abs() + 0.125
    qkv[s - 1, h:2 * h] = -INF
    got, want = (forward(qkv, (1, s, heads, d, 0), v) for v in (variant, -1))
    assert bool(torch.isfinite(want[0]).all())
    same(got[0], want[0], TOL["f32"], "ctx")
    same(got[1], want[1], TOL["f32"], "log-sum-exp")


@pytest.mark.parametrize("d", [16, 64])
def test_scores_are_those_of_the_row_kernels(d):
    """One visible key and a scale that is a power of two: the log-sum-exp is the scaled score, and the same to the bit in every form."""
    qkv, dims = rnd((600, 3 * d), "f32", 3), (600, 1, 1, d, 1)
    rows = forward(qkv, dims, -1)
    for variant in (4, 5):
        assert all(torch.equal(x, y) for x, y in zip(forward(qkv, dims, variant), rows))
