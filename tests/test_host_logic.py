"""CPU-only checks: the C-ABI library loads and exports what the header declares,
size/offset queries, argument validation (no GPU is touched by any of these),
and the FLOP cost model against the paper's throughput pairs."""
import ctypes as C
import os
import re

import pytest

from paper_2111_04007_amd import CONFIGS, binding as B, flops
from paper_2111_04007_amd.synth import StageConfig

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    lib = B.load()
    header = open(os.path.join(ROOT, "include", "varuna_stage.h")).read()
    declared = set(re.findall(r"\b(varuna_[a-z0-9_]+)\s*\(", header))
    assert declared, "no declarations parsed"
    assert declared == set(B.EXPORTS)
    for name in declared:
        assert hasattr(lib, name), name


def test_boundary_slot_size_matches_paper_example():
    """Design Overview: the stored input activation of the 2.5B GPT-2 (h=1920,
    s=1024, 16-bit) is 3.75 MB per example: one [s, h] tensor, nothing else."""
    cfg = StageConfig("x", 4, 1920, 20, 1024, 1, 1, 7680, True, "bf16")
    _, _, boundary, _ = B.query_sizes(cfg)
    assert boundary == 3_932_160 == int(3.75 * 2 ** 20)
    cfg8 = cfg.replace(micro_batch=4, n_micro_batches=16)
    assert B.query_sizes(cfg8)[2] == 3_932_160 * 4 * 16


@pytest.mark.parametrize("key", list(CONFIGS))
def test_param_layout(key):
    cfg = CONFIGS[key]
    h, f = cfg.hidden, cfg.mlp_hidden
    per_layer = 12 * h * h + 13 * h
    assert f == 4 * h
    pb, gb, _, wb = B.query_sizes(cfg)
    es = 4 if cfg.dtype == "f32" else 2
    assert pb == per_layer * cfg.n_layers * es
    assert gb == per_layer * cfg.n_layers * 4
    assert wb > 0
    want = [h, h, 3 * h * h, 3 * h, h * h, h, h, h, f * h, f, h * f, h]
    off = 0
    for l in range(cfg.n_layers):
        for i, n in enumerate(want):
            assert B.param_offset(cfg, l, i) == (off, n)
            off += n


def _expect(code, fn, *a):
    with pytest.raises(B.VarunaError) as ei:
        fn(*a)
    assert ei.value.code == code
    assert str(ei.value)


def test_config_validation():
    good = CONFIGS["C1"]
    _expect(B.EINVAL, B.query_sizes, good.replace(n_heads=3))
    _expect(B.EINVAL, B.query_sizes, good.replace(n_layers=0))
    _expect(B.EINVAL, B.query_sizes, good.replace(seq_len=-1))
    _expect(B.EUNSUPPORTED, B.query_sizes, good.replace(seq_len=1 << 20))
    _expect(B.EINVAL, B.param_offset, good, 2, 0)
    _expect(B.EINVAL, B.param_offset, good, 0, 12)
    lib = B.load()
    assert lib.varuna_stage_query_sizes(None, None, None, None, None) == B.EINVAL
    assert b"NULL" in lib.varuna_last_error()


def test_call_order_and_range_errors_without_gpu():
    """create/forward/backward argument and state checks return before any GPU work."""
    lib = B.load()
    cc = B.c_config(CONFIGS["C1"])
    h = C.c_void_p()
    fake = C.c_void_p(0x10000)   # aligned, never dereferenced on these paths
    assert lib.varuna_stage_create(C.byref(cc), None, fake, fake, fake, C.byref(h)) == B.EINVAL
    assert lib.varuna_stage_create(C.byref(cc), C.c_void_p(0x10010), fake, fake, fake, C.byref(h)) == B.EINVAL
    assert lib.varuna_stage_create(C.byref(cc), fake, fake, fake, fake, None) == B.EINVAL
    assert lib.varuna_stage_create(C.byref(cc), fake, fake, fake, fake, C.byref(h)) == B.OK
    assert lib.varuna_stage_forward(h, 4, fake, fake, None) == B.EINVAL
    assert lib.varuna_stage_forward(h, -1, fake, fake, None) == B.EINVAL
    assert lib.varuna_stage_forward(h, 0, None, fake, None) == B.EINVAL
    assert lib.varuna_stage_backward_recompute(h, 0, fake, fake, None) == B.ESTATE
    assert b"without a forward" in lib.varuna_last_error()
    assert lib.varuna_stage_backward_recompute(None, 0, fake, fake, None) == B.EINVAL
    assert lib.varuna_stage_grad_accum_reset(None, None) == B.EINVAL
    assert lib.varuna_stage_destroy(h) == B.OK
    assert lib.varuna_stage_destroy(None) == B.EINVAL


def test_op_argument_validation_without_gpu():
    lib = B.load()
    fake = C.c_void_p(0x10000)
    assert lib.varuna_op_gemm(B.BF16, 0, 0, 0, 0, 8, 8, fake, fake, fake, None, fake, None, None) == B.EINVAL
    assert lib.varuna_op_gemm(B.BF16, 0, 7, 0, 8, 8, 8, fake, fake, fake, None, fake, None, None) == B.EINVAL
    assert lib.varuna_op_gemm(B.BF16, 0, 2, 0, 8, 8, 8, fake, fake, fake, None, fake, None, None) == B.EINVAL
    assert lib.varuna_op_gemm(5, 0, 0, 0, 8, 8, 8, fake, fake, fake, None, fake, None, None) == B.EINVAL
    assert lib.varuna_op_attention_fwd(B.BF16, 0, 1, 0, 1, 64, 1, fake, fake, None, None) == B.EINVAL
    assert lib.varuna_op_attention_fwd(B.BF16, 0, 1, 1 << 20, 1, 64, 1, fake, fake, None, None) == B.EUNSUPPORTED
    assert lib.varuna_op_colreduce_scratch_bytes(4096, 1024) == 16 * 1024 * 4


def test_flop_model_reproduces_paper_throughput_pairs():
    """Evaluation: the 200B model (100 layers, h=12960, s=1024) ran at 0.022 ex/s/GPU
    = 27.3 TFLOP/s/GPU of useful work; 72*h^2 + 12*s*h FLOPs per token-layer
    reproduces that pair to a few percent."""
    per_ex = flops.model_flops_per_example(100, 12960, 1024)
    assert abs(per_ex * 0.022 / 1e12 - 27.3) / 27.3 < 0.03
    # stage accounting: 4 units of hardware work, 3 useful, forward = 1 (Background:
    # forward is a third of the iteration; recompute adds a third)
    cfg = CONFIGS["C5"]
    assert flops.step_flops_per_microbatch(cfg) == 4 * flops.forward_flops(cfg)
    assert flops.useful_flops_per_microbatch(cfg) == 3 * flops.forward_flops(cfg)
    dense = flops.forward_flops(cfg, causal_aware=False)
    T, h, s = cfg.tokens, cfg.hidden, cfg.seq_len
    assert dense == cfg.n_layers * (24.0 * T * h * h + 4.0 * T * s * h)
    assert abs(3 * dense / cfg.micro_batch - flops.model_flops_per_example(cfg.n_layers, h, s)) < 1e-3 * dense


def test_pick_micro_batch_rule():
    """Parametrized Simulation: the lowest m at which F(m)/m stops improving.  The paper's own
    datum (Job Morphing, "Problem setting and constraints": m=8 is 26 % better per example
    than m=4 for BERT-large) must move the pick past m=4."""
    from paper_2111_04007_amd.calibrate import pick_micro_batch
    ms = [1, 2, 4, 8, 16]
    assert pick_micro_batch(ms, [10.0, 7.0, 5.0, 5.0 / 1.26, 5.0 / 1.26 * 0.99]) == 8
    assert pick_micro_batch(ms, [3.0, 3.0, 3.0, 3.0, 3.0]) == 1            # flat: smallest m
    assert pick_micro_batch(ms, [5.0, 4.0, 3.0, 2.0, 1.0]) == 16           # still improving: largest
    assert pick_micro_batch([4, 1, 2], [1.0, 2.0, 1.02]) == 2              # order-free; 2 % is within the threshold
    assert pick_micro_batch(ms, [4.0, 3.0, 3.2, 2.5, 2.49]) == 8           # a non-monotone bump does not stop the search
    with pytest.raises(ValueError):
        pick_micro_batch([], [])


def test_grouped_rings_must_stay_addressable_with_32_bit_offsets():
    """bf16 path: G stacked micro-batches of the [T, f] weight-gradient operand must stay
    below 4 GiB (config 5: 128 MiB per slot, so G = 32 is the first group size refused)."""
    c5 = CONFIGS["C5"]
    assert B.query_sizes(c5.replace(wgrad_group=31))[3] > 0
    _expect(B.EUNSUPPORTED, B.query_sizes, c5.replace(wgrad_group=32))
    assert B.query_sizes(CONFIGS["C1"].replace(wgrad_group=64))[3] > 0


def test_gemm_kernel_choice_for_the_named_stage_shapes():
    """Which bf16 GEMM configuration the library picks (host-only query): 256x256 tiles where they
    fill the 256 CUs in whole rounds, 128x128 tiles otherwise, and merged 128x256 / 256x128 tiles
    where two 128x128 tiles per CU would share nothing and the merged form needs no more rounds."""
    FWD, DGRAD, WGRAD = 0, 1, 2
    T, h, f = 2048, 8192, 32768                                    # C5: everything on 256x256 tiles
    assert B.debug_gemm_choice(FWD, T, 3 * h, h) == 17 and B.debug_gemm_choice(FWD, T, h, f) == 17
    assert B.debug_gemm_choice(DGRAD, T, f, h) == 18 and B.debug_gemm_choice(DGRAD, T, h, 3 * h) == 18
    assert B.debug_gemm_choice(WGRAD, h, f, T) == 18 and B.debug_gemm_choice(WGRAD, 3 * h, h, 8 * T) == 18
    T, h, f = 2048, 3072, 12288                                    # C4
    assert B.debug_gemm_choice(FWD, T, 3 * h, h) == 19             # 1152 tiles: 2.25 rounds, elastic
    assert B.debug_gemm_choice(FWD, T, h, h) == 20                 # 384 tiles -> 192 merged, one round
    assert B.debug_gemm_choice(FWD, T, f, h) == 20                 # 1536 tiles -> 768 merged, 3 whole rounds
    assert B.debug_gemm_choice(DGRAD, T, h, f) == 20
    assert B.debug_gemm_choice(WGRAD, h, f, T) == 19                # weight gradients stay on 128x128
    T, h, f = 4096, 1920, 7680                                     # C3: 1920 = 15 x 128, only M is a multiple of 256
    assert B.debug_gemm_choice(FWD, T, h, h) == 21 and B.debug_gemm_choice(DGRAD, T, h, 3 * h) == 21
    assert B.debug_gemm_choice(FWD, T, f, h) == 17                 # 480 256x256 tiles: two rounds beat four of 128x128
    T, h, f = 4096, 1024, 4096                                     # C2
    assert B.debug_gemm_choice(FWD, T, h, h) == 19                 # 256 tiles: one workgroup per CU
    assert B.debug_gemm_choice(FWD, T, 3 * h, h) == 17             # 192 256x256 tiles: one round
    assert B.debug_gemm_choice(DGRAD, T, h, 3 * h) == 19
    assert B.debug_gemm_choice(FWD, 100, 128, 64) == -1            # one ragged tile: the small tiles
    assert B.debug_gemm_choice(7, 128, 128, 64) == -2


def test_named_weight_gradient_kernels_turn_the_grouped_launch_off():
    """A named configuration is what a step's weight gradients run on, so they may not go into a launch that has its own."""
    h, f, tokens = 1024, 4096, 4096
    assert B.debug_wgrad_group_choice(1, h, f, tokens) > 0 and B.debug_wgrad_group_choice(0, h, f, tokens) == -2
    try:
        for kw in ({"wgrad256": 12}, {"wgrad128": 14}):
            B.debug_set_gemm_kernels(**kw)
            assert B.debug_wgrad_group_choice(1, h, f, tokens) == 0
        B.debug_set_gemm_kernels(fwd256=12)
        assert B.debug_wgrad_group_choice(1, h, f, tokens) > 0
    finally:
        B.debug_set_gemm_kernels()


def test_gemm_kernel_choice_for_ragged_shapes():
    """Sizes that are no multiples of the tiles: 128x128 (22) or 256x256 (23) ragged tiles, small tiles on any addresses where rows are
    not whole 16-byte pieces."""
    FWD, DGRAD, WGRAD = 0, 1, 2
    T, h, f = 2000, 1600, 6400
    assert B.debug_gemm_choice(FWD, T, h, h) == 22 and B.debug_gemm_choice(DGRAD, T, h, f) == 22 and B.debug_gemm_choice(WGRAD, h, h, T) == 22
    assert B.debug_gemm_choice(FWD, T, f, h) == 23 and B.debug_gemm_choice(DGRAD, T, f, h) == 23 and B.debug_gemm_choice(WGRAD, f, h, T) == 23
    assert B.debug_gemm_choice(FWD, T, h, h + 1) == -1 and B.debug_gemm_choice(DGRAD, T, h + 4, h) == -1 and B.debug_gemm_choice(WGRAD, h + 4, h, T) == -1


def test_weight_gradient_group_choice():
    assert [B.debug_wgrad_group_choice(*a) for a in ((4, 1024, 4096, 128), (1, 1024, 4096, 4096), (1, 960, 3840, 192), (2, 768, 3072, 1000))] == [18, 19, 22, 23]
    assert B.debug_wgrad_group_choice(1, 512, 2048, 128) == 0          # fewer tiles than slots: split sums instead
    assert B.debug_wgrad_group_choice(2, 8192, 32768, 4096) == 0       # thousands of 256x256 tiles: nothing to gain
    assert B.debug_wgrad_group_choice(4, 1920, 7680, 4096) == 19 and B.debug_wgrad_group_choice(4, 1920, 7680, 32768) == 0


def test_weight_gradients_of_a_small_stage_share_a_launch_of_the_small_tiles():
    """Up to 128 tiles of 128x128 in all, counted with their ragged ones, and not where a weight-gradient configuration is named."""
    for layers, h, f, want in ((1, 64, 256, -1), (4, 64, 256, -1), (2, 256, 1024, -1), (3, 256, 1024, 0), (1, 384, 1536, -1), (1, 385, 1536, 0), (1, 512, 2048, 0), (1, 385, 1152, -1), (1, 385, 1153, 0)):
        assert B.debug_wgrad_group_choice(layers, h, f, 512) == want, (layers, h, f)
    try:
        B.debug_set_gemm_kernels(wgrad128=14)
        assert B.debug_wgrad_group_choice(2, 256, 1024, 512) == 0
    finally:
        B.debug_set_gemm_kernels()
