"""Register-operand tiles (problems of few tiles) through the public entry points.

Sizes sit where the tiles can go wrong: below, at and past a 32 x 32 and a 64 x 32 block,
K below, at and past one chunk of 16 and one turn of the four K waves (64), the largest
K and tile counts the rule gives them.  Integer inputs must come out bit for bit (every
partial sum is an integer below 2^24); U[-1, 1] inputs within 1e-5 normwise, the bar of
every float32 path.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1804_10694_amd import inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.fixture(scope="module")
def tg():
    from paper_1804_10694_amd import tgemm
    tgemm.set_policy("default")
    yield tgemm


SIZES = [(1, 1, 1), (31, 33, 15), (32, 32, 16), (33, 65, 17), (64, 64, 63), (65, 31, 64), (96, 100, 65),
         (130, 70, 129), (257, 255, 300), (700, 650, 700), (1060, 1060, 33), (40, 2500, 1100), (16, 16, 9000),
         (1600, 1600, 64), (1000, 1000, 1030)]


@pytest.mark.parametrize("shape", SIZES)
@pytest.mark.parametrize("dtype", ["f32", "x3"])
def test_few_tiles_exact_with_nan_around(tg, dtype, shape):
    # A, B, C inside wider buffers of NaN, at odd row strides: nothing outside reaches a sum and
    # nothing outside C is written.  |entries| <= 8: partial sums stay below 9000 * 64 < 2^24
    M, N, K = shape
    A, B, C0 = inputs.integer_inputs(M, N, K, seed=sum(shape), r=8)
    Ab, Bb, Cb = (inputs.padded(x, 3)[0].to(DEV) for x in (A, B, C0))
    tg.gemm(Ab[:, :K], Bb[:, :N], Cb[:, :N], 1.5, 0.5, dtype)
    got = Cb.cpu()
    np.testing.assert_array_equal(got[:, :N].numpy().astype(np.float64), oracle.gemm(A, B, C0, 1.5, 0.5))
    assert torch.isnan(got[:, N:]).all()


@pytest.mark.parametrize("shape", [(256, 256, 256), (700, 700, 4100), (1060, 1060, 1060), (33, 2000, 515)])
@pytest.mark.parametrize("dtype", ["f32", "x3"])
def test_few_tiles_within_tolerance(tg, dtype, shape):
    A, B, C0 = inputs.gemm_inputs(*shape, seed=11)
    C = C0.to(DEV)
    tg.gemm(A.to(DEV), B.to(DEV), C, 1.0, 1.0, dtype)
    again = C0.to(DEV)
    tg.gemm(A.to(DEV), B.to(DEV), again, 1.0, 1.0, dtype)
    assert torch.equal(C, again)  # the K waves' sums are added in a fixed order
    assert oracle.normwise_error(C.cpu().numpy(), oracle.gemm(A, B, C0, 1.0, 1.0)) <= 1e-5


def test_beta_zero_does_not_read_c_and_infinities_stay_in_their_rows(tg):
    A, B, C0 = inputs.integer_inputs(70, 90, 50, seed=5, r=8)
    A[3, 7] = float("inf")
    C = torch.full((70, 90), float("nan"), device=DEV)
    tg.gemm(A.to(DEV), B.to(DEV), C, 1.0, 0.0, "f32")
    rows = [i for i in range(70) if i != 3]
    ref = A[rows].double() @ B.double()
    np.testing.assert_array_equal(C.cpu()[rows].double().numpy(), ref.numpy())
    assert not torch.isfinite(C.cpu()[3][B[7] != 0]).any()


# labels: 9, 8 batch; 0, 5 rows; 2, 6 columns; 1, 3 contracted.  Every order of A, B and C that keeps one
# of its modes contiguous is read (or written) in place; the others go through copies
EXT = {9: 3, 8: 2, 0: 40, 5: 3, 2: 37, 6: 2, 1: 35, 3: 4}
ORDERS = [([9, 0, 1], [9, 1, 2], [9, 0, 2]), ([1, 9, 0], [9, 2, 1], [9, 0, 2]), ([9, 1, 0], [1, 9, 2], [0, 9, 2]),
          ([0, 9, 1], [2, 9, 1], [9, 2, 0]), ([1, 0, 9], [9, 1, 2], [9, 0, 2]), ([9, 0, 1], [9, 1, 2], [2, 0, 9]),
          ([8, 9, 0, 5, 1, 3], [1, 3, 8, 9, 2], [8, 9, 0, 5, 2]), ([9, 8, 0, 5, 1], [8, 9, 1, 2, 6], [8, 9, 0, 5, 2, 6]),
          ([1, 3, 0, 5], [2, 6, 1, 3], [0, 5, 2, 6]), ([0, 5, 3, 1], [2, 1, 3], [2, 0, 5]), ([1, 0], [1, 2], [0, 2]),
          ([0, 1], [2, 1], [2, 0]), ([9, 0], [9, 2], [9, 0, 2]), ([9, 1], [9, 2, 1], [9, 2]),
          ([1, 9, 0], [1, 9], [9, 0])]


@pytest.mark.parametrize("order", ORDERS, ids=lambda o: "_".join("".join(map(str, m)) for m in o))
@pytest.mark.parametrize("dtype", ["f32", "x3"])
def test_contraction_in_any_order_exact(tg, dtype, order):
    from oracle import contract as OT
    ma, mb, mc = order
    g = torch.Generator().manual_seed(17)
    A, B, C0 = (torch.randint(-8, 9, [EXT[m] for m in o], generator=g).float() for o in (ma, mb, mc))
    for alpha, beta in ((1.0, 0.0), (1.5, 0.5)):
        C = torch.full_like(C0, float("nan")) if beta == 0 else C0.clone()
        C = C.to(DEV)
        tg.contract(A.to(DEV), ma, B.to(DEV), mb, C, mc, alpha, beta, dtype)
        np.testing.assert_array_equal(C.cpu().numpy().astype(np.float64),
                                      OT.contract(A, ma, B, mb, mc, C0, alpha, beta))


@pytest.mark.parametrize("dims", [(256, 64, 64, 65), (16, 130, 200, 129), (1101, 33, 20, 128), (1100, 40, 64, 128)])
@pytest.mark.parametrize("dtype", ["f32", "x3"])
def test_strided_batch_exact(tg, dtype, dims):
    # on both sides of the tile counts where register tiles take a batch
    P, M, N, K = dims
    g = torch.Generator().manual_seed(18)
    A, B, C0 = (torch.randint(-8, 9, d, generator=g).float() for d in ((P, M, K), (P, K, N), (P, M, N)))
    C = C0.to(DEV)
    tg.gemm_batched_strided(A.to(DEV), B.to(DEV), C, 1.0, 1.0, dtype)
    ref = torch.bmm(A.double(), B.double()) + C0.double()
    np.testing.assert_array_equal(C.cpu().double().numpy(), ref.numpy())
