"""The fp32-product GEMM kernels at the edges of their tiles, stages and vector loads, against fp64."""
import pytest
import torch

from oracle import stage_oracle as O
from paper_2111_04007_amd import binding as B
from paper_2111_04007_amd.synth import to_f64
from tests.test_ops_parity import rnd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K", [
    (32, 32, 128), (33, 31, 129), (64, 36, 4), (1, 4, 127), (40, 44, 256),   # 32x32 tiles: remainders of tile, stage and piece
    (1025, 1026, 67), (1024, 1028, 64), (1100, 1000, 63), (2048, 516, 132),  # 64x64 tiles
    (128, 128, 3), (5, 3, 2),
])
def test_gemm_fp32_products(dtype, M, N, K):
    """fp32 sums of K products in any order: rel-L2 of a row's result is below sqrt(K) * 2^-24 * a small constant; 4e-7 * K^0.5
    / 8 + 2e-7 covers K up to 256 with a factor of two.  A bf16 output adds the rounding of the output (2^-9 / sqrt(3))."""
    tol = (2e-7 + 5e-8 * K ** 0.5) if dtype == "f32" else 2.5e-3
    x, w, wd = rnd((M, K), dtype, 1), rnd((N, K), dtype, 2, 0.05), rnd((K, N), dtype, 3, 0.05)
    bias, aux = rnd((N,), dtype, 4, 0.5), rnd((M, N), dtype, 5)
    out = torch.empty((M, N), dtype=x.dtype, device="cuda")
    v = 0 if dtype == "f32" else -1
    B.op_gemm(B.OP_FWD, 2, x, w, out, bias=bias, aux_in=aux, variant=v, M=M, N=N, K=K)
    assert O.rel_l2(to_f64(out), to_f64(aux) + O.linear_forward(to_f64(x), to_f64(w), to_f64(bias))) <= tol
    B.op_gemm(B.OP_DGRAD, 0, x, wd, out, variant=v, M=M, N=N, K=K)
    assert O.rel_l2(to_f64(out), to_f64(x) @ to_f64(wd)) <= tol
    dy, xx = rnd((K, M), dtype, 6), rnd((K, N), dtype, 7)
    acc = torch.full((M, N), 0.25, dtype=torch.float32, device="cuda")
    B.op_gemm(B.OP_WGRAD, 0, dy, xx, acc, variant=v, M=M, N=N, K=K)
    assert O.rel_l2(to_f64(acc), 0.25 + to_f64(dy).T @ to_f64(xx)) <= 2e-7 + 5e-8 * K ** 0.5
