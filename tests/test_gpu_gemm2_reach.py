"""Back-to-back gemm with the longest rows of B and D that it takes (2^31 / 64 - 1 floats): the
last rows of a panel lie nearly 2^32 bytes past its first.  Small integers, bit-exact; the
padding of the rows holds NaN."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
LD = (2 ** 31 - 1) // 64


@pytest.fixture(scope="module")
def tg():
    from paper_1804_10694_amd import tgemm
    tgemm.set_policy("default")
    yield tgemm
    torch.cuda.empty_cache()


def _padded(rows, cols, ld):
    X = torch.full((rows, ld), float("nan"), device=DEV)
    X[:, :cols] = torch.randint(-3, 4, (rows, cols), device=DEV, dtype=torch.int8).float()
    return X[:, :cols]


@pytest.mark.parametrize("dtype", ["f32", "x3"])
@pytest.mark.parametrize("M,K,N1,N2", [(70, 37, 35, 9), (70, 32, 64, 140)])  # part panels and whole ones
def test_longest_rows(tg, dtype, M, K, N1, N2):
    A = torch.randint(-3, 4, (M, K), device=DEV, dtype=torch.int8).float()
    B, D = _padded(K, N1, LD), _padded(N1, N2, LD)
    E = torch.full((M, N2), float("nan"), device=DEV)
    tg.gemm2(A, B, D, E, relu=True, dtype=dtype)
    torch.cuda.synchronize()
    ref = torch.relu(A.double() @ B.double()) @ D.double()
    assert torch.equal(E.double(), ref)


def test_longer_rows_are_refused(tg):
    f = 0x10000
    assert tg.lib.tgemm_gemm2(4, 4, 4, 4, 1.0, f, 4, f, LD + 1, 0, f, 4, 0.0, f, 4, 0, None) == tg.NOT_SUPPORTED
    assert tg.lib.tgemm_gemm2(4, 4, 4, 4, 1.0, f, 4, f, 4, 0, f, LD + 1, 0.0, f, 4, 0, None) == tg.NOT_SUPPORTED
