"""Weight gradients of several matrices in one launch: whole tiles, ragged tiles, more matrices than one launch holds."""
import pytest
import torch

from paper_2111_04007_amd import binding as B, synth
from tests import parity_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers,heads,d,s,group", [
    (1, 8, 128, 128, 1),    # 768 128x128 tiles
    (1, 13, 80, 100, 1),    # ragged in every direction, a partly filled k-tile
    (5, 8, 64, 128, 1),     # 20 matrices: a launch of 16, the fifth layer's four one by one
    (1, 15, 64, 192, 2),    # two stacked micro-batches and a flush of one
])
def test_grouped_weight_gradients(layers, heads, d, s, group):
    h = heads * d
    cfg = synth.StageConfig("grouped-wgrad", layers, h, heads, s, 1, 3 if group > 1 else 1, 4 * h, True, "bf16", 0.02, seed=51 + s, wgrad_group=group)
    params = synth.make_params(cfg, perturb=0.05)
    xs, dys = synth.make_activations(cfg, cfg.n_micro_batches)
    st, ys, dxs = U.gpu_stage_step(cfg, params, xs, dys)
    U.compare_step(cfg, st, ys, dxs, U.oracle_stage_step(cfg, params, xs, dys), label=cfg.name)
    first = st.grads.clone()
    st.close()
    st, _, _ = U.gpu_stage_step(cfg, params, xs, dys)
    assert torch.equal(first, st.grads)   # the order of every sum is fixed
    st.close()


@pytest.mark.parametrize("layers,heads,d,s,f,kernel", [
    (2, 12, 64, 333, 3072, 23),   # 256x256 tiles, ragged in K only
    (2, 21, 64, 200, 5000, 23),   # ... ragged in every direction
    (4, 16, 64, 128, 4096, 18),   # 256x256 whole tiles
    (8, 8, 64, 128, 2048, 19),    # 32 matrices: two launches of 16
    (8, 13, 40, 100, 2080, 22),   # ... of ragged tiles
])
def test_grouped_weight_gradients_on_every_kernel(layers, heads, d, s, f, kernel):
    h = heads * d
    assert B.debug_wgrad_group_choice(min(layers, 4), h, f, s) == kernel
    cfg = synth.StageConfig("grouped-kernels", layers, h, heads, s, 1, 1, f, True, "bf16", 0.02, seed=61 + s)
    params = synth.make_params(cfg, perturb=0.05)
    xs, dys = synth.make_activations(cfg, 1)
    st, ys, dxs = U.gpu_stage_step(cfg, params, xs, dys)
    U.compare_step(cfg, st, ys, dxs, U.oracle_stage_step(cfg, params, xs, dys), label=cfg.name)
    st.close()


@pytest.mark.parametrize("heads,d,s,f", [(12, 64, 70, 3072), (13, 59, 70, 3001)])
def test_grouped_weight_gradients_fp32_64x64_tiles(heads, d, s, f):
    """About 1700 64x64 tiles (7 rounds of the chip against 27 of 32x32), with and without whole 16-byte pieces; 1e-5 as for fp32."""
    cfg = synth.StageConfig("grouped-f32", 1, heads * d, heads, s, 1, 1, f, True, "f32", 0.02, seed=71)
    params = synth.make_params(cfg, perturb=0.05)
    xs, dys = synth.make_activations(cfg, 1)
    st, ys, dxs = U.gpu_stage_step(cfg, params, xs, dys)
    U.compare_step(cfg, st, ys, dxs, U.oracle_stage_step(cfg, params, xs, dys), label=cfg.name)
    st.close()
