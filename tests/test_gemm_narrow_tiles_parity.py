"""Forward products whose merged tiles are 192 wide: short reductions, every epilogue, each third of a tile."""
import pytest
import torch

from paper_2111_04007_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("epi", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", [(1024, 6144, 64), (1024, 6144, 128), (1024, 6144, 192), (2048, 3072, 448), (4096, 1536, 1536)])
def test_narrow_merged_tiles(epi, M, N, K):
    """Against fp32 products of the same operands; a bf16 output rounds by at most 2^-8 of itself, and its sum by far less."""
    assert B.debug_gemm_choice(B.OP_FWD, M, N, K) == 20
    g = torch.Generator(device="cuda").manual_seed(7)
    x, w, bias, res = (torch.empty(s, device="cuda").normal_(0, d, generator=g).bfloat16() for s, d in (((M, K), 1.0), ((N, K), 0.05), ((N,), 1.0), ((M, N), 1.0)))
    out, u = torch.full((M, N), 7.0, device="cuda").bfloat16(), torch.full((M, N), 7.0, device="cuda").bfloat16()
    B.op_gemm(B.OP_FWD, epi, x, w, out, bias=bias, aux_in=res if epi == 2 else None, aux_out=u if epi == 1 else None, M=M, N=N, K=K)
    want = x.double() @ w.double().t() + bias.double()
    pairs = [(out, want)]
    if epi == 1:
        pairs = [(u, want), (out, torch.nn.functional.gelu(want, approximate="tanh"))]
    elif epi == 2:
        pairs = [(out, want + res.double())]
    for got, ref in pairs:
        d = got.double() - ref
        for c in range(0, N, 32):   # the parts of a wave's 96 columns
            assert float(d[:, c:c + 32].norm() / ref[:, c:c + 32].norm()) <= 2.5e-3
        assert float(d.abs().max() / ref.abs().max()) <= 2.0 ** -8


def test_named_tile_width_is_what_runs():
    """20 is 256 wide and 24 is 192 wide also where the library would take the other: each refuses a width that is no multiple of its own."""
    M, K = 128, 64
    for variant, N, ok in ((20, 768, True), (24, 768, True), (20, 576, False), (24, 576, True), (20, 512, True), (24, 512, False)):
        g = torch.Generator(device="cuda").manual_seed(N)
        x, w, bias = (torch.empty(s, device="cuda").normal_(0, 1, generator=g).bfloat16() for s in ((M, K), (N, K), (N,)))
        out = torch.full((M, N), 7.0, device="cuda").bfloat16()
        if not ok:
            with pytest.raises(B.VarunaError) as ei:
                B.op_gemm(B.OP_FWD, 0, x, w, out, bias=bias, variant=variant, M=M, N=N, K=K)
            assert ei.value.code == B.EUNSUPPORTED
            continue
        B.op_gemm(B.OP_FWD, 0, x, w, out, bias=bias, variant=variant, M=M, N=N, K=K)
        want = x.double() @ w.double().t() + bias.double()
        assert float((out.double() - want).norm() / want.norm()) <= 2.5e-3   # a bf16 output's rounding
    with pytest.raises(B.VarunaError) as ei:   # the n-major products have no such tile
        B.op_gemm(B.OP_DGRAD, 0, torch.zeros(128, 64, device="cuda").bfloat16(), torch.zeros(64, 192, device="cuda").bfloat16(),
                  torch.zeros(128, 192, device="cuda").bfloat16(), variant=24, M=128, N=192, K=64)
    assert ei.value.code == B.EUNSUPPORTED
