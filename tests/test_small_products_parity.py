"""bf16 products on either side of the limits that send them to the small shared-reduction tiles, and weight gradients of a whole stage in one launch."""
import pytest
import torch

from paper_2111_04007_amd import binding as B
from paper_2111_04007_amd.synth import StageConfig

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("op,epi", [(0, "plain"), (0, "fused"), (1, "plain"), (1, "fused"), (2, "plain")])
@pytest.mark.parametrize("M,N,K", [(128, 256, 64), (300, 768, 72), (768, 384, 1000), (384, 896, 256), (500, 1024, 2048), (1000, 1024, 1536), (1000, 1024, 1528), (1024, 1024, 4096), (1152, 1024, 4096)])
def test_either_side_of_the_limits(op, M, N, K, epi):
    """Exact products and fp32 sums: a bf16 output is off by its rounding (2^-9 / sqrt(3) and a margin), an fp32 one by 2e-7 + 5e-8 sqrt(K)."""
    g = torch.Generator(device="cuda").manual_seed(op)
    a, b = ((M, K), (N, K)) if op == 0 else ((M, K), (K, N)) if op == 1 else ((K, M), (K, N))
    a, b, aux = (torch.empty(s, device="cuda").normal_(0, d, generator=g).bfloat16() for s, d in ((a, 1.0), (b, 0.1), ((M, N), 1.0)))
    bias = torch.empty(N, device="cuda").normal_(0, 1, generator=g).bfloat16()
    want = (a.double() @ b.double().t()) if op == 0 else a.double() @ b.double() if op == 1 else a.double().t() @ b.double()
    if op == 2:
        out = torch.full((M, N), 0.5, device="cuda")
        B.op_gemm(2, 0, a, b, out, M=M, N=N, K=K)
        assert float((out.double() - want - 0.5).norm() / (want + 0.5).norm()) <= 2e-7 + 5e-8 * K ** 0.5
        return
    out, u = torch.full((M, N), 7.0, device="cuda").bfloat16(), torch.full((M, N), 7.0, device="cuda").bfloat16()
    if op == 0 and epi == "fused":
        B.op_gemm(0, 1, a, b, out, bias=bias, aux_out=u, M=M, N=N, K=K)
        pre = want + bias.double()
        assert float((u.double() - pre).norm() / pre.norm()) <= 2.5e-3
        want = torch.nn.functional.gelu(pre, approximate="tanh")
    elif op == 0:
        B.op_gemm(0, 2, a, b, out, bias=bias, aux_in=aux, M=M, N=N, K=K)
        want = want + bias.double() + aux.double()
    elif epi == "fused":
        B.op_gemm(1, 3, a, b, out, aux_in=aux, M=M, N=N, K=K)
        v = aux.double().requires_grad_(True)
        want = want * torch.autograd.grad(torch.nn.functional.gelu(v, approximate="tanh").sum(), v)[0]
    else:
        B.op_gemm(1, 0, a, b, out, M=M, N=N, K=K)
    assert float((out.double() - want).norm() / want.norm()) <= 2.5e-3


@pytest.mark.parametrize("L,h,heads,s,group", [(1, 64, 2, 40, 1), (1, 63, 3, 40, 1), (2, 162, 6, 33, 2), (2, 128, 2, 64, 2), (5, 64, 1, 128, 1), (1, 400, 5, 72, 2), (1, 512, 8, 128, 1)])
def test_stage_weight_gradients(L, h, heads, s, group):
    """The weight gradients of the stage are the products of the tensors it leaves: against the same stage in fp32 on the same (bf16) values."""
    grads = []
    for dtype in ("bf16", "f32"):
        c = StageConfig("case", L, h, heads, s, 2, 2, 4 * h, True, dtype, wgrad_group=group)
        dt = torch.bfloat16 if dtype == "bf16" else torch.float32
        g = torch.Generator(device="cuda").manual_seed(5)
        n = B.Stage(c, "cuda:0").params.numel()
        p = torch.empty(n, device="cuda").normal_(0, 0.03, generator=g).bfloat16()
        st = B.Stage(c, "cuda:0", params_flat=p.to(dt))
        xs = torch.empty(2, 2 * s, h, device="cuda").normal_(0, 1, generator=g).bfloat16().to(dt)
        ys, dxs = torch.empty_like(xs), torch.empty_like(xs)
        st.grad_accum_reset()
        for m in range(2):
            st.forward(m, xs[m], ys[m])
            st.backward_recompute(m, xs[m], dxs[m])
        st.grad_flush()
        grads.append(st.grads.double())
    assert float((grads[0] - grads[1]).norm() / grads[1].norm()) <= 2e-2   # bf16 activations between the layers
