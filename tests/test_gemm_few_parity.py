"""fp32 products of few output elements (16x16 tiles, operands straight into registers): edges of tiles and units of the reduction, either side of the
limits that send a product there."""
import pytest
import torch

from paper_2111_04007_amd import binding as B, synth
from tests import parity_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [
    (1, 4, 4), (15, 20, 12), (16, 16, 16), (17, 36, 124), (33, 52, 128), (128, 128, 132), (31, 16, 256), (47, 68, 260), (100, 100, 512), (64, 64, 516),
    (5, 8, 1020), (128, 512, 900), (256, 512, 1000), (250, 516, 768), (512, 512, 128), (512, 512, 132), (2048, 256, 64), (2049, 256, 64), (3, 8192, 20),
])
def test_few_outputs(M, N, K):
    """fp32 sums of K terms: 2e-7 + 5e-8 sqrt(K), as the other fp32 products; GeLU and its derivative have slopes up to 1.13 and
    add roundings of their own (3e-7)."""
    g = torch.Generator(device="cuda").manual_seed(K)
    x, w, v, bias, aux = (torch.empty(s, device="cuda").normal_(0, d, generator=g) for s, d in
                          (((M, K), 1.0), ((N, K), 0.1), ((K, N), 0.1), ((N,), 1.0), ((M, N), 1.0)))
    tol = 2e-7 + 5e-8 * K ** 0.5

    def near(got, want, extra=0.0):
        assert float((got.double() - want).norm() / want.norm()) <= tol + extra

    out, u = torch.full((M + 1, N), 7.0, device="cuda"), torch.full((M, N), 7.0, device="cuda")
    fwd = x.double() @ w.double().t() + bias.double()
    B.op_gemm(0, 0, x, w, out, bias=bias, M=M, N=N, K=K)
    near(out[:M], fwd)
    B.op_gemm(0, 1, x, w, out, bias=bias, aux_out=u, M=M, N=N, K=K)
    near(u, fwd)
    near(out[:M], torch.nn.functional.gelu(fwd, approximate="tanh"), 3e-7)
    B.op_gemm(0, 2, x, w, out, bias=bias, aux_in=aux, M=M, N=N, K=K)
    near(out[:M], fwd + aux.double())
    back = x.double() @ v.double()
    B.op_gemm(1, 0, x, v, out, M=M, N=N, K=K)
    near(out[:M], back)
    B.op_gemm(1, 3, x, v, out, aux_in=aux, M=M, N=N, K=K)
    y = aux.double().requires_grad_(True)
    near(out[:M], back * torch.autograd.grad(torch.nn.functional.gelu(y, approximate="tanh").sum(), y)[0], 3e-7)
    assert bool((out[M] == 7.0).all())


@pytest.mark.parametrize("op", [0, 1])
def test_values_behind_the_operands_stay_out(op):
    """NaNs behind both operands and in rows of other products: k and rows past the end are not multiplied."""
    M, N, K = 37, 44, 100
    g = torch.Generator(device="cuda").manual_seed(1)
    shapes = ((M, K), (N, K) if op == 0 else (K, N))
    bufs = [torch.full((a * b + 4096,), float("nan"), device="cuda") for a, b in shapes]
    a, b = (buf[:p * q].view(p, q).normal_(generator=g) for buf, (p, q) in zip(bufs, shapes))
    out = torch.empty(M, N, device="cuda")
    bias = torch.zeros(N, device="cuda")
    B.op_gemm(op, 0, a, b, out, bias=bias if op == 0 else None, M=M, N=N, K=K)
    want = a.double() @ (b.double().t() if op == 0 else b.double())
    assert float((out.double() - want).norm() / want.norm()) <= 1e-6


@pytest.mark.parametrize("h,heads,s,b,f", [(100, 5, 33, 1, 0), (128, 2, 17, 2, 40), (256, 4, 50, 1, 0), (260, 2, 16, 1, 516), (512, 8, 31, 1, 0), (516, 6, 20, 1, 0), (42, 3, 20, 1, 0)])
def test_layer_norm_in_front_of_a_product(h, heads, s, b, f):
    """Forward, recompute and backward of stages whose norms join the product that follows (widths up to 512 in whole 16-byte pieces) and of two whose
    do not, at the fp32 path's tolerance; inputs that start at an odd element give the same bits."""
    cfg = synth.StageConfig("norm-product", 2, h, heads, s, b, 2, f or 4 * h, True, "f32", 0.05, seed=h)
    params = synth.make_params(cfg, perturb=0.05)
    xs, dys = synth.make_activations(cfg, 2)
    st, ys, dxs = U.gpu_stage_step(cfg, params, xs, dys)
    U.compare_step(cfg, st, ys, dxs, U.oracle_stage_step(cfg, params, xs, dys), label=f"h={h}")
    x = torch.as_tensor(xs[0]).reshape(b * s, h).float().cuda()
    odd = torch.empty(x.numel() + 1, device="cuda")[1:].view_as(x).copy_(x)
    y, z = torch.empty_like(x), torch.empty_like(x)
    st.forward(0, x, y)
    st.forward(1, odd, z)
    assert torch.equal(y, z)
    st.close()
