"""Weight gradients that 256x256 tiles take from 128x128 ones: single products of odd sides, and whole groups."""
import pytest
import torch

from paper_2111_04007_amd import binding as B, synth
from tests import parity_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(1920, 7680, 512), (7680, 1920, 576), (9984, 1152, 512), (384, 25600, 640)])
def test_single_products_of_odd_sides(M, N, K):
    """Twice +=: the same bits as the named kernel, and against fp64 within K roundings of the products' sum (2^-24 of the largest partial sum each)."""
    assert B.debug_gemm_choice(B.OP_WGRAD, M, N, K) == 19
    g = torch.Generator(device="cuda").manual_seed(K)
    a, b = (torch.empty(K, n, device="cuda").normal_(0, 1, generator=g).bfloat16() for n in (M, N))
    got, named = (torch.full((M, N), 3.0, device="cuda") for _ in range(2))
    for _ in range(2):
        B.op_gemm(B.OP_WGRAD, 0, a, b, got, M=M, N=N, K=K)
        B.op_gemm(B.OP_WGRAD, 0, a, b, named, variant=23, M=M, N=N, K=K)
    assert torch.equal(got, named)
    for m in range(0, M, 1920):
        x = a[:, m:m + 1920].double().t()
        bound = (K + 4) * 2.0 ** -24 * (2 * (x.abs() @ b.double().abs()) + 3.0)
        assert bool(((got[m:m + 1920].double() - (2 * (x @ b.double()) + 3.0)).abs() <= bound).all())


@pytest.mark.parametrize("h,f,heads,s,b,choice", [
    (1024, 4096, 8, 512, 4, 19),    # whole 256x256 tiles
    (1152, 3456, 12, 512, 4, 19),   # sides of 9 and 27 x 128
    (1000, 4000, 25, 410, 5, 22),   # ragged in every direction, a partly filled k-tile
])
def test_groups_of_long_reductions(h, f, heads, s, b, choice):
    assert B.debug_wgrad_group_choice(1, h, f, s * b) == choice
    cfg = synth.StageConfig("wide-groups", 1, h, heads, s, b, 1, f, True, "bf16", 0.02, seed=81)
    params = synth.make_params(cfg, perturb=0.05)
    xs, dys = synth.make_activations(cfg, 1)
    st, ys, dxs = U.gpu_stage_step(cfg, params, xs, dys)
    U.compare_step(cfg, st, ys, dxs, U.oracle_stage_step(cfg, params, xs, dys), label=cfg.name)
    st.close()
