"""Weight gradients of several matrices in one launch: whole tiles, ragged tiles, more matrices than one launch holds."""
import pytest
import torch

from paper_2111_04007_amd import synth
from tests import parity_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers,heads,d,s,group", [
    (1, 8, 128, 128, 1),    # 768 128x128 tiles
    (1, 13, 80, 100, 1),    # ragged in every direction, a partly filled k-tile
    (5, 8, 64, 128, 1),     # 20 matrices: two launches
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
