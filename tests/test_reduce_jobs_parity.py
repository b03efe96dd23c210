"""Bias and LayerNorm parameter gradients of a layer in one launch: one chunk of 256 rows, several, a partial last one; widths
that are and are not whole 16-byte pieces; with and without the side stream."""
import pytest
import torch

from paper_2111_04007_amd import synth
from tests import parity_util as U

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
