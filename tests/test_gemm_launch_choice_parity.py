"""Products whose launch takes another kernel configuration than the one counted by rounds."""
import pytest
import torch

from paper_2111_04007_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("op,epi,M,N,K,choice,runs", [
    (0, 0, 6144, 3072, 64, 19, 24),       # three whole rounds of 192-wide tiles
    (0, 2, 2048, 5760, 192, 19, 24),
    (0, 1, 4096, 10240, 2304, 20, 17),    # three rounds of 256x256 for five of merged tiles
    (0, 2, 4096, 9216, 2304, 19, 17),
    (0, 0, 1024, 6912, 64, 20, 21),       # merged tiles turned
    (1, 3, 512, 9216, 128, 20, 21),
    (1, 0, 1536, 5120, 448, 20, 21),
    (1, 0, 2048, 5120, 3584, 18, 17),     # four waves
    (1, 3, 1024, 10240, 2304, 18, 17),
    (0, 0, 1920, 7680, 1024, 19, 23),     # sides of odd multiples of 128: the ragged form of the large tiles
    (0, 1, 4480, 6912, 1088, 20, 23),
    (0, 2, 6016, 4224, 1024, 19, 23),
    (1, 0, 1408, 10752, 1152, 19, 23),
    (1, 3, 1408, 10752, 1024, 19, 23),
])
def test_other_configurations_at_launch(op, epi, M, N, K, choice, runs):
    """The same bits as the named configuration, and a bf16 output's rounding (2^-9 in the norm, 2^-8 of the largest value) against fp64."""
    assert B.debug_gemm_choice(op, M, N, K) == choice
    g = torch.Generator(device="cuda").manual_seed(K)
    x, w, bias, aux = (torch.empty(s, device="cuda").normal_(0, d, generator=g).bfloat16()
                       for s, d in (((M, K), 1.0), ((N, K) if op == 0 else (K, N), K ** -0.5), ((N,), 1.0), ((M, N), 1.0)))
    outs = []
    for variant in (0, runs):
        out, u = torch.full((M, N), 7.0, device="cuda").bfloat16(), torch.full((M, N), 7.0, device="cuda").bfloat16()
        B.op_gemm(op, epi, x, w, out, bias=bias if op == 0 else None, aux_in=aux if epi >= 2 else None, aux_out=u if epi == 1 else None, variant=variant, M=M, N=N, K=K)
        outs.append((out, u))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    want = x.double() @ (w.double().t() if op == 0 else w.double())
    if op == 0:
        want += bias.double()
    if epi == 1:
        want = torch.nn.functional.gelu(want, approximate="tanh")
    elif epi == 2:
        want += aux.double()
    elif epi == 3:
        a = aux.double().requires_grad_()
        torch.nn.functional.gelu(a, approximate="tanh").backward(want)
        want = a.grad
    d = outs[0][0].double() - want
    assert float(d.norm() / want.norm()) <= 2.5e-3 and float(d.abs().max() / want.abs().max()) <= 2.0 ** -8
