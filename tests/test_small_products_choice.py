"""Which bf16 products go to the small shared-reduction tiles, and that a named configuration is what runs instead (host only)."""
import pytest

from paper_2111_04007_amd import binding as B


@pytest.mark.parametrize("op,M,N,K,small", [(0, 256, 1024, 64, True), (0, 384, 768, 8192, True), (0, 512, 1024, 64, True), (1, 512, 1024, 512, False), (1, 512, 1024, 1024, True),
                                            (2, 512, 1024, 1024, False), (2, 512, 1024, 2048, True), (0, 1024, 1024, 1024, False), (0, 1000, 1000, 1536, True),
                                            (2, 1024, 1024, 2048, False), (2, 1024, 1024, 4096, True), (0, 1152, 1024, 8192, False)])
def test_choice_of_few_tiles(op, M, N, K, small):
    assert (B.debug_gemm_choice(op, M, N, K) == -1) == small
    try:
        B.debug_set_gemm_kernels(fwd128=7, dgrad128=7, wgrad128=7)
        plain = M % 128 == 0 and N % 128 == 0
        assert B.debug_gemm_choice(op, M, N, K) == (7 if plain else 22)
    finally:
        B.debug_set_gemm_kernels()
    assert (B.debug_gemm_choice(op, M, N, K) == -1) == small
