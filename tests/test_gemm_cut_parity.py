"""Products on bf16 pieces: edges of steps, pieces and tiles, accuracy of an fp32 product, values at the ends of the range."""
import pytest
import torch

from paper_2111_04007_amd import binding as B

pytestmark = pytest.mark.gpu
DT = {"f32": torch.float32, "bf16": torch.bfloat16}


def rnd(shape, dtype, seed, std=1.0):
    return torch.empty(shape, dtype=torch.float32, device="cuda").normal_(0, std, generator=torch.Generator(device="cuda").manual_seed(seed)).to(DT[dtype])


def product(op, a, b, M, N, K, dtype):
    """The plain product of every layout: out, and the same in 64 bits."""
    if op == 0:
        bias = torch.zeros(N, dtype=DT[dtype], device="cuda")
        out = torch.full((M, N), 7.0, dtype=DT[dtype], device="cuda")
        B.op_gemm(op, 0, a, b, out, bias=bias, M=M, N=N, K=K)
        return out, a.double() @ b.double().t()
    if op == 1:
        out = torch.full((M, N), 7.0, dtype=DT[dtype], device="cuda")
        B.op_gemm(op, 0, a, b, out, M=M, N=N, K=K)
        return out, a.double() @ b.double()
    out = torch.zeros(M, N, device="cuda")
    B.op_gemm(op, 0, a, b, out, M=M, N=N, K=K)
    return out, a.double().t() @ b.double()


def operands(op, dtype, M, N, K, seed=1):
    a, b = {0: ((M, K), (N, K)), 1: ((M, K), (K, N)), 2: ((K, M), (K, N))}[op]
    return rnd(a, dtype, seed), rnd(b, dtype, seed + 1)


# a tile of each kind (32 on 8 waves, 32 on 4, 64 on 4, 64 on 1) with remainders of tile, 16-byte piece, step and share of the steps
SHAPES = [(1, 1, 1), (3, 2, 9), (33, 31, 17), (65, 7, 33), (63, 65, 1040), (41, 3, 1151), (31, 33, 255), (1, 257, 130), (481, 499, 161), (801, 803, 1025), (834, 833, 1089),
          (1000, 768, 1100), (1793, 1801, 1031), (2113, 2049, 67)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("op", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_every_remainder(dtype, op, M, N, K):
    """fp32 sums in several parts: 2e-7 and 5e-8 per root of K; a bf16 output adds its rounding (2^-9 / sqrt(3) and a margin)."""
    out, want = product(op, *operands(op, dtype, M, N, K), M, N, K, dtype)
    tol = 2.5e-3 if dtype == "bf16" and op < 2 else 2e-7 + 5e-8 * K ** 0.5
    assert float((out.double() - want).norm() / want.norm()) <= tol
    rows = (out.double() - want).norm(dim=1) / want.norm() * M ** 0.5
    assert float(rows.max()) <= 12 * tol   # no row or tile of its own error


@pytest.mark.parametrize("op", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", [(96, 70, 200), (96, 70, 1100), (1024, 1024, 1024), (2048, 2048, 1024)])
@pytest.mark.parametrize("scale", [1e-36, 1e-30, 1e30])
def test_small_and_large_values(op, M, N, K, scale):
    """Values whose last pieces would underflow, and large ones, keep the accuracy of an fp32 product (the products stay normal numbers)."""
    a, b = operands(op, "f32", M, N, K)
    a *= scale
    b *= min(1.0, 1e4 / scale) if scale > 1 else 1.0
    out, want = product(op, a, b, M, N, K, "f32")
    assert float((out.double() - want).norm() / want.norm()) <= 2e-7 + 5e-8 * K ** 0.5


@pytest.mark.parametrize("op", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", [(70, 65, 90), (70, 65, 1090), (1024, 1024, 1024), (2048, 2048, 1024)])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), torch.finfo(torch.float32).max, torch.finfo(torch.float32).min])
def test_values_at_the_end_of_the_range(op, M, N, K, value):
    """One such value reaches exactly its row or column, as in fp32 products: zeros of the other operand included."""
    a, b = operands(op, "f32", M, N, K)
    (a if op == 2 else a.t())[K // 2, M // 3] = value
    (b.t() if op == 0 else b)[K // 2, N // 4] = 0.0
    (b.t() if op == 0 else b)[K // 2, N // 2] = 2.0 ** -20
    out, want = product(op, a, b, M, N, K, "f32")
    want = want.float()   # rounds to infinity beyond the range; 64-bit products of finite values stay finite
    assert torch.equal(torch.isnan(out), torch.isnan(want)) and torch.equal(torch.isinf(out), torch.isinf(want))
    fin = torch.isfinite(want)
    assert torch.equal(out[~fin & ~torch.isnan(want)], want[~fin & ~torch.isnan(want)])
    rest = torch.arange(M, device="cuda") != M // 3
    d = (out[rest].double() - want[rest].double()).norm() / want[rest].double().norm()
    assert float(d) <= 2e-7 + 5e-8 * K ** 0.5
    # the row itself, element by element: an fp32 sum of K terms is off by at most K half units of the sum of their sizes
    ad, bd = (a.double().t() if op == 2 else a.double()), (b.double().t() if op == 0 else b.double())
    size = ad[M // 3].abs() @ bd.abs()
    off = (out[M // 3].double() - want[M // 3].double()).abs()
    assert bool((off <= K * 2.0 ** -24 * size)[fin[M // 3]].all())


@pytest.mark.parametrize("op", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", [(70, 65, 90), (70, 65, 1090), (512, 512, 2048), (1024, 1024, 1024), (2048, 2048, 1024)])
@pytest.mark.parametrize("place", ["row", "column", "pair", "small times large"])
def test_small_values_beside_others(op, M, N, K, place):
    """Values whose last bits no bf16 holds, in tiles whose sums are ordinary: one row, one column, one k of both operands, one whole operand.
    Every row and every column keeps the error of an fp32 product, relative to itself."""
    a, b = operands(op, "f32", M, N, K)
    at, bt = (a.t() if op == 2 else a), (b if op == 0 else b.t())   # [M, K], [N, K]
    if place == "row":
        at[M // 3] *= 1e-36
    elif place == "column":
        bt[N // 2] *= 1e-37
    elif place == "pair":
        at[:, K // 2] *= 1e-36
        bt[:, K // 2] *= 1e37
    else:
        a *= 1e-36
        b *= 1e30
    out, want = product(op, a, b, M, N, K, "f32")
    d = out.double() - want
    for dim in (0, 1):
        assert float((d.norm(dim=dim) / want.norm(dim=dim)).max()) <= 2e-7 + 5e-8 * K ** 0.5


@pytest.mark.parametrize("M,N,K", [(1801, 1801, 1000), (1801, 1801, 2000), (2049, 1601, 4000), (1201, 1101, 2000), (601, 601, 1000), (301, 255, 3000), (1801, 1801, 300), (1801, 1801, 129)])
@pytest.mark.parametrize("signs", ["both", "one"])
def test_error_of_a_bf16_weight_gradient(M, N, K, signs):
    """fp32 sums of exact products, on every kind of tile: no further from 64 bits than sums in fp32 products, whose measured errors stand
    here (values of both signs, which err more); a quarter as much again is allowed for, the error of a seed's values differs by a tenth."""
    a, b = operands(2, "bf16", M, N, K)
    if signs == "one":
        a, b = a.abs(), b.abs()
    out, want = product(2, a, b, M, N, K, "bf16")
    fp32_products = {129: 0.56e-7, 300: 0.70e-7, 1000: 0.92e-7, 2000: 1.20e-7, 3000: 1.46e-7, 4000: 1.69e-7}[K]
    assert float((out.double() - want).norm() / want.norm()) <= 1.25 * fp32_products


@pytest.mark.parametrize("op", [0, 1, 2])
@pytest.mark.parametrize("values", ["normal", "clustered"])
@pytest.mark.parametrize("K", [1, 2, 3, 16, 33])
def test_single_products_of_a_short_reduction(op, values, K):
    """Short sums show the rounding of their products.  1.0040206 * 1.0038986 has the largest terms of middle and last pieces, 2^-24 of the
    product; of K terms of one sign a result in fp32 is off by half a unit for each of its K roundings, and by no more."""
    M, N = 63, 65
    a, b = operands(op, "f32", M, N, K)
    if values == "clustered":
        a, b = (c * (1 + 1e-5 * x.clamp(-1, 1)) for c, x in ((1.0040206, a), (1.0038986, b)))
    else:
        a, b = a.abs(), b.abs()
    out, want = product(op, a, b, M, N, K, "f32")
    assert float(((out.double() - want).abs() / want).max()) <= 2.0 ** -24 * (K + 2.0 ** -8)   # (what is left out is below 2^-33)


@pytest.mark.parametrize("op", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", [(500, 2304, 1280), (1024, 1152, 1024), (1000, 1600, 1024), (1000, 768, 1276), (1000, 768, 1280), (1000, 3068, 1024), (1000, 3072, 1024)])
def test_whole_pieces_on_either_side_of_the_limits(op, M, N, K):
    out, want = product(op, *operands(op, "f32", M, N, K), M, N, K, "f32")
    assert float((out.double() - want).norm() / want.norm()) <= 2e-7 + 5e-8 * K ** 0.5   # as in every remainder


@pytest.mark.parametrize("op", [0, 1, 2])
@pytest.mark.parametrize("dtype,M,N,K", [("f32", 70, 65, 127), ("f32", 70, 65, 128), ("f32", 1101, 1103, 127), ("f32", 1101, 1103, 128), ("bf16", 1101, 1103, 64), ("bf16", 1101, 1103, 65), ("bf16", 999, 1003, 64), ("bf16", 1101, 1103, 256), ("bf16", 1101, 1103, 257), ("bf16", 1455, 1409, 200), ("f32", 1101, 1103, 255)])
def test_either_side_of_a_short_reduction(op, dtype, M, N, K):
    out, want = product(op, *operands(op, dtype, M, N, K), M, N, K, dtype)
    tol = 2.5e-3 if dtype == "bf16" and op < 2 else 2e-7 + 5e-8 * K ** 0.5   # as in every remainder
    assert float((out.double() - want).norm() / want.norm()) <= tol


@pytest.mark.parametrize("op", [0, 1, 2])
@pytest.mark.parametrize("dtype,M,N,K", [("bf16", 40, 24, 8), ("bf16", 8, 72, 31), ("bf16", 104, 336, 200), ("bf16", 720, 904, 1001), ("f32", 44, 20, 1025), ("f32", 444, 484, 1039), ("f32", 1000, 1024, 1290)])
def test_whole_rows_with_a_rest_of_k(op, dtype, M, N, K):
    """Last steps of operands whose k-rows are whole pieces, in tiles that end within the operand."""
    out, want = product(op, *operands(op, dtype, M, N, K), M, N, K, dtype)
    tol = 2.5e-3 if dtype == "bf16" and op < 2 else 2e-7 + 5e-8 * K ** 0.5   # as in every remainder
    assert float((out.double() - want).norm() / want.norm()) <= tol
