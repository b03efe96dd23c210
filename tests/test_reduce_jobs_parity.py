"""Bias and LayerNorm parameter gradients of a layer in one launch: one chunk of 256 rows, several, a partial last one; widths
that are and are not whole 16-byte pieces; with and without the side stream."""
import pytest
import torch

from oracle import stage_oracle as O
from paper_2111_04007_amd import binding as B, synth
from paper_2111_04007_amd.synth import to_f64
from tests import parity_util as U
from tests.test_ops_parity import rnd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,heads,d,s,f", [
    ("f32", 2, 32, 64, 96), ("f32", 3, 20, 256, 132), ("f32", 1, 37, 257, 75), ("bf16", 2, 40, 300, 328), ("bf16", 3, 12, 520, 100),
])
def test_reduce_jobs(dtype, heads, d, s, f):
    cfg = synth.StageConfig("reduce-jobs", 2, heads * d, heads, s, 1, 2, f, True, dtype, 0.05, seed=s)
    params = synth.make_params(cfg, perturb=0.05)
    xs, dys = synth.make_activations(cfg, 2)
    ref = U.oracle_stage_step(cfg, params, xs, dys)
    grads = []
    for side in (True, False):
        st, ys, dxs = U.gpu_stage_step(cfg, params, xs, dys, side_stream=side)
        U.compare_step(cfg, st, ys, dxs, ref, label=f"{dtype} side={side}")
        grads.append(st.grads.clone())
        st.close()
    assert torch.equal(*grads)


@pytest.mark.parametrize("dtype,rows,n", [
    ("f32", 3, 66000), ("bf16", 70, 132000), ("f32", 1030, 16004), ("bf16", 1800, 20008), ("bf16", 1281, 264), ("f32", 257, 33000),
])
def test_colsum_wide_and_narrow_blocks(dtype, rows, n):
    """Both block shapes of the partial sums (2 blocks of 32 column groups per CU and fewer) and of the second stage (up to 4
    chunks of 256 rows and more); 1e-5 as for every column sum."""
    a = rnd((rows, n), dtype, 8)
    out = torch.full((n,), 1.0, dtype=torch.float32, device="cuda")
    B.op_colsum(a, out, torch.empty(B.colreduce_scratch_bytes(rows, n) // 4, dtype=torch.float32, device="cuda"))
    assert O.rel_l2(to_f64(out), 1.0 + to_f64(a).sum(axis=0)) <= 1e-5


@pytest.mark.parametrize("dtype,rows,h", [("f32", 16000, 1540), ("bf16", 16000, 3080), ("bf16", 1500, 3080)])
def test_layernorm_parameter_gradients_wide_and_narrow_blocks(dtype, rows, h):
    x, dy, res = rnd((rows, h), dtype, 3), rnd((rows, h), dtype, 6), rnd((rows, h), dtype, 7)
    gamma = (rnd((h,), dtype, 4, 0.2) + 1.0).to(x.dtype)
    y, dx, stats = torch.empty_like(x), torch.empty_like(x), torch.empty(2 * rows, device="cuda")
    dg, db = (torch.zeros(h, device="cuda") for _ in range(2))
    B.op_layernorm_fwd(x, gamma, gamma, y, stats)
    B.op_layernorm_bwd(dy, x, stats, gamma, res, dx, dg, db, torch.empty(B.colreduce_scratch_bytes(rows, 2 * h) // 4, device="cuda"))
    xd, dyd = x.double(), dy.double()
    xhat = (xd - xd.mean(1, keepdim=True)) / (xd.var(1, unbiased=False, keepdim=True) + 1e-5).sqrt()
    for got, want in ((dg, (dyd * xhat).sum(0)), (db, dyd.sum(0))):   # the bound of the LayerNorm tests' fp32 sums
        assert float((got.double() - want).norm() / want.norm()) <= 1e-5
