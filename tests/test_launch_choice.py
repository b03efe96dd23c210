"""Which configuration bf16 products and groups of weight gradients run on, where that is not the one counted by rounds of tiles alone, and the sizes just
beyond each line (host only; the dispatch and the query call the same function)."""
import pytest

from paper_2111_04007_amd import binding as B

FWD, DGRAD, WGRAD = 0, 1, 2


@pytest.mark.parametrize("op,epi,M,N,K,choice,runs", [
    (FWD, 0, 6144, 3072, 1536, 19, 24), (FWD, 0, 6144, 3840, 1536, 20, 20), (FWD, 0, 8192, 3072, 1536, 20, 20),      # 192-wide merged tiles: up to three rounds
    (FWD, 1, 6144, 3072, 1472, 19, 19), (FWD, 0, 2048, 9216, 64, 19, 19), (FWD, 2, 2048, 5760, 192, 19, 19), (FWD, 0, 2048, 3072, 3072, 20, 24),   # and long reductions
    (FWD, 1, 4096, 10240, 2304, 20, 17), (FWD, 1, 4096, 10240, 2240, 20, 21),                                   # 256x256: long reductions
    (FWD, 2, 4096, 9216, 2304, 19, 17), (FWD, 2, 4096, 9216, 2240, 19, 19),
    (FWD, 0, 1024, 6912, 64, 20, 21), (FWD, 0, 3072, 7680, 2560, 20, 20),                                       # merged tiles turned: clearly wide, whole groups of rows
    (DGRAD, 3, 512, 9216, 128, 20, 21), (DGRAD, 0, 1536, 5120, 448, 20, 21), (DGRAD, 0, 1536, 4096, 448, 20, 20), (DGRAD, 3, 2048, 4096, 12288, 20, 21), (DGRAD, 0, 2048, 4096, 12288, 20, 20),
    (DGRAD, 0, 2048, 5120, 3584, 18, 17), (DGRAD, 0, 2048, 5120, 3520, 18, 18), (DGRAD, 0, 3328, 4096, 3584, 18, 18),   # four waves: up to 200 workgroups, long reductions
    (DGRAD, 3, 1024, 10240, 2304, 18, 17), (DGRAD, 3, 1024, 10240, 2240, 18, 18),
    (FWD, 0, 1920, 7680, 1024, 19, 23), (FWD, 0, 1920, 7680, 960, 19, 19), (FWD, 1, 4480, 6912, 1088, 20, 23), (FWD, 2, 6016, 4224, 1024, 19, 23),   # odd multiples of 128
    (FWD, 1, 4096, 5760, 1920, 21, 21), (FWD, 0, 3200, 4992, 1664, 19, 19),
    (FWD, 2, 2304, 10880, 1792, 21, 21), (FWD, 0, 8064, 3072, 2816, 20, 20), (FWD, 1, 1920, 12800, 3200, 20, 23), (FWD, 0, 8832, 5632, 1472, 20, 23),   # against merged tiles in three rounds
    (DGRAD, 0, 1408, 10752, 1152, 19, 23), (DGRAD, 3, 1408, 10752, 1024, 19, 23), (DGRAD, 0, 2944, 9216, 2304, 19, 23), (DGRAD, 3, 2944, 9216, 2304, 19, 19),
    (WGRAD, 0, 1920, 7680, 512, 19, 23), (WGRAD, 0, 1920, 7680, 448, 19, 19), (WGRAD, 0, 7680, 1920, 576, 19, 23), (WGRAD, 0, 9984, 1152, 512, 19, 23),
    (WGRAD, 0, 384, 25600, 768, 19, 23), (WGRAD, 0, 384, 25472, 768, 19, 19), (WGRAD, 0, 8832, 2944, 512, 19, 19), (WGRAD, 0, 8832, 2944, 768, 19, 23), (WGRAD, 0, 6016, 7040, 640, 19, 23), (WGRAD, 0, 4480, 4480, 2048, 19, 19),
    (FWD, 0, 100, 128, 64, -1, -1), (FWD, 0, 2000, 1600, 1601, -1, -1), (FWD, 0, 2000, 6400, 1600, 23, 23), (WGRAD, 0, 8192, 8192, 2048, 18, 18),
])
def test_products(op, epi, M, N, K, choice, runs):
    assert B.debug_gemm_choice(op, M, N, K) == choice and B.debug_gemm_launch(op, epi, M, N, K) == runs


@pytest.mark.parametrize("layers,h,f,tokens,choice,runs", [
    (1, 1024, 4096, 2048, 19, 18), (1, 1024, 4096, 1984, 19, 19), (1, 1152, 3456, 2048, 19, 23), (1, 1152, 3456, 2047, 22, 22), (1, 1000, 4000, 2050, 22, 23),
    (1, 1000, 4000, 2000, 22, 22), (1, 1920, 7680, 4096, 19, 23), (2, 1600, 6400, 2048, 22, 22), (1, 896, 3584, 8192, 19, 19), (1, 256, 1024, 2048, -1, -1),
    (2, 8192, 32768, 4096, 0, 0), (2, 768, 3072, 1000, 23, 23),
])
def test_groups_of_weight_gradients(layers, h, f, tokens, choice, runs):
    assert B.debug_wgrad_group_choice(layers, h, f, tokens) == choice and B.debug_wgrad_group_launch(layers, h, f, tokens) == runs


def test_a_named_configuration_is_what_runs():
    try:
        B.debug_set_gemm_kernels(fwd128=14)
        assert B.debug_gemm_launch(FWD, 0, 1920, 7680, 1024) == 14
        B.debug_set_gemm_kernels(wgrad128=14)
        assert B.debug_gemm_launch(WGRAD, 0, 1920, 7680, 512) == 14 and B.debug_wgrad_group_launch(1, 1024, 4096, 2048) == 0
    finally:
        B.debug_set_gemm_kernels()


def test_what_is_no_product():
    for op, epi, M in ((3, 0, 128), (FWD, 3, 128), (DGRAD, 1, 128), (WGRAD, 4, 128), (FWD, 0, 0), (FWD, 0, 1 << 31)):
        assert B.debug_gemm_launch(op, epi, M, 128, 64) == -2
    assert B.debug_wgrad_group_launch(0, 1024, 4096, 2048) == -2
