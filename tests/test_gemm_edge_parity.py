"""The bf16 MFMA GEMM kernels on sizes that are no multiples of their tiles: every remainder, outputs next to the edge
untouched, no values from beyond a row's end."""
import pytest
import torch

from oracle import stage_oracle as O
from paper_2111_04007_amd import binding as B
from paper_2111_04007_amd.synth import to_f64
from tests.test_ops_parity import rnd

pytestmark = pytest.mark.gpu

SHAPES = [(129, 8, 8), (130, 136, 72), (8, 264, 56), (136, 128, 64), (264, 520, 200), (255, 256, 320), (513, 264, 448), (200, 1000, 840)]


@pytest.mark.parametrize("variant", [0, 22, 23])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_gemm_edge_rounding_accuracy(variant, M, N, K):
    """Output rounding 2^-9 / sqrt(3) = 1.1e-3 (bf16), 1e-5 for the fp32 accumulator.  The operands end exactly where a
    guard of NaNs begins: a value read past the end of a row or of the tensor and multiplied in would spread."""
    def guarded(shape, seed, scale=1.0):
        n = shape[0] * shape[1]
        buf = torch.full((n + 4096,), float("nan"), dtype=torch.bfloat16, device="cuda")
        buf[:n] = rnd(shape, "bf16", seed, scale).reshape(-1)
        return buf[:n].view(shape)

    x, w, wd = guarded((M, K), 1), guarded((N, K), 2, 0.05), guarded((K, N), 3, 0.05)
    bias, res = rnd((N,), "bf16", 4, 0.5), rnd((M, N), "bf16", 5)
    guard = torch.full((M * N + 4096,), 7.0, dtype=torch.bfloat16, device="cuda")
    out = guard[:M * N].view(M, N)
    B.op_gemm(B.OP_FWD, 2, x, w, out, bias=bias, aux_in=res, variant=variant, M=M, N=N, K=K)
    assert O.rel_l2(to_f64(out), to_f64(res) + O.linear_forward(to_f64(x), to_f64(w), to_f64(bias))) <= 2.5e-3
    B.op_gemm(B.OP_DGRAD, 0, x, wd, out, variant=variant, M=M, N=N, K=K)
    assert O.rel_l2(to_f64(out), to_f64(x) @ to_f64(wd)) <= 2.5e-3
    assert bool((guard[M * N:] == 7.0).all())
    Mw = (M + 7) // 8 * 8   # the weight gradient's M is a row length
    dy, xx = guarded((K, Mw), 6), guarded((K, N), 7)
    accg = torch.full((Mw * N + 4096,), 0.5, dtype=torch.float32, device="cuda")
    acc = accg[:Mw * N].view(Mw, N)
    B.op_gemm(B.OP_WGRAD, 0, dy, xx, acc, variant=variant, M=Mw, N=N, K=K)
    assert O.rel_l2(to_f64(acc), 0.5 + to_f64(dy).T @ to_f64(xx)) <= 1e-5
    for K1 in (K + 1, K + 5):   # a reduction of any length (tokens)
        dy, xx = guarded((K1, Mw), 8), guarded((K1, N), 9)
        acc.fill_(0.5)
        B.op_gemm(B.OP_WGRAD, 0, dy, xx, acc, variant=variant, M=Mw, N=N, K=K1)
        assert O.rel_l2(to_f64(acc), 0.5 + to_f64(dy).T @ to_f64(xx)) <= 1e-5
    assert bool((accg[Mw * N:] == 0.5).all())


@pytest.mark.parametrize("variant", [22, 23])
def test_gemm_edge_bit_stable_under_memory_contention(variant):
    """A k-tile must not be read before it has landed, also where loads of the last, partly filled one make no request."""
    side = torch.cuda.Stream()
    big = torch.empty(1 << 28, dtype=torch.uint8, device="cuda")
    big2 = torch.empty_like(big)
    M, N = 1000, 1400
    for K in (72, 136, 200, 1032):
        x, w, wd = rnd((M, K), "bf16", 40 + K), rnd((N, K), "bf16", 41 + K, 0.05), rnd((K, N), "bf16", 42 + K, 0.05)
        dy, xx, bias = rnd((K + 3, M), "bf16", 43 + K), rnd((K + 3, N), "bf16", 44 + K), rnd((N,), "bf16", 45 + K, 0.5)
        torch.cuda.synchronize()

        def products():
            o1 = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
            o2 = torch.empty_like(o1)
            o3 = torch.zeros((M, N), dtype=torch.float32, device="cuda")
            B.op_gemm(B.OP_FWD, 0, x, w, o1, bias=bias, variant=variant, M=M, N=N, K=K)
            B.op_gemm(B.OP_DGRAD, 0, x, wd, o2, variant=variant, M=M, N=N, K=K)
            B.op_gemm(B.OP_WGRAD, 0, dy, xx, o3, variant=variant, M=M, N=N, K=K + 3)
            return o1, o2, o3

        ref = products()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for _ in range(12):
                big2.copy_(big, non_blocking=True)
        outs = [products() for _ in range(8)]
        torch.cuda.synchronize()
        for o in outs:
            for got, want in zip(o, ref):
                assert torch.equal(got, want), (variant, K)


def test_stage_ragged_widths():
    """A whole bf16 step whose hidden size, MLP width and token count fit no tile (split weight gradients included)."""
    from paper_2111_04007_amd import synth
    from tests import parity_util as U
    for cfg in (synth.StageConfig("ragged-bf16-wide", 2, 5 * 64, 5, 200, 3, 2, 1288, True, "bf16", 0.02, seed=41),
                synth.StageConfig("ragged-bf16-g2", 1, 3 * 72, 3, 333, 2, 3, 864, False, "bf16", 0.02, seed=42, wgrad_group=2)):
        params = synth.make_params(cfg, perturb=0.05)
        xs, dys = synth.make_activations(cfg, cfg.n_micro_batches)
        st, ys, dxs = U.gpu_stage_step(cfg, params, xs, dys)
        U.compare_step(cfg, st, ys, dxs, U.oracle_stage_step(cfg, params, xs, dys), label=cfg.name)
        st.close()
