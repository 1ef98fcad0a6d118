"""bf16 packed tiles that sum each K block of 128 by itself: as exact as the direct tiles.

Both add a K block's sum to the whole with one fused multiply-add; only the order inside a block
differs, so their errors against FP64 are alike (asserted: at most 1.25 times; a running sum over
8192 k is 3 times as far off).  Codes of small integers with power-of-two scales are exact, over
K that ends inside a block, inside a panel, and on both.
"""
import numpy as np
import pytest
import torch

import oracle
from oracle import precision as P
from paper_1804_10694_amd import inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.fixture(scope="module")
def tg():
    from paper_1804_10694_amd import tgemm
    tgemm.set_policy("default")
    yield tgemm
    tgemm.set_policy("default")


def _folded(tg):
    return [sid for sid, i in tg.schedules("bf16") if i["vec"] == 0 and (i["BM"], i["BN"], i["BK"]) == (128, 128, 64)]


def _bits(x):
    return torch.from_numpy(P.bf16_bits(x).view(np.int16)).to(DEV)


@pytest.mark.parametrize("shape", [(300, 260, 700), (129, 500, 128), (65, 70, 129), (40, 33, 50), (257, 130, 2049)],
                         ids=lambda s: "x".join(map(str, s)))
def test_exact_on_integers(tg, shape):
    M, N, K = shape
    A, B, C0 = inputs.integer_inputs(M, N, K, seed=81, r=8)
    g = np.random.default_rng(82)
    SA = (2.0 ** g.integers(-2, 3, P.scale_grid_shape(M, K))).astype(np.float32)
    SB = (2.0 ** g.integers(-2, 3, P.scale_grid_shape(K, N))).astype(np.float32)
    QA, QB = P.bf16_bits(A.numpy()), P.bf16_bits(B.numpy())
    ref = P.gemm_scaled_expected(QA, SA, QB, SB, C0.numpy(), 1.5, 0.5, "bf16")
    plain = oracle.gemm(A, B, C0, 1.5, 0.5)
    qa, qb, sa, sb = _bits(A.numpy()), _bits(B.numpy()), torch.from_numpy(SA).to(DEV), torch.from_numpy(SB).to(DEV)
    assert len(_folded(tg)) == 2
    for sid in _folded(tg):
        print(f"{shape} {tg.schedule_key(sid)}", flush=True)
        tg.set_policy(f"force:{sid}")
        C, D = C0.to(DEV), C0.to(DEV)
        tg.gemm_scaled(qa, sa, qb, sb, C, 1.5, 0.5, "bf16")
        tg.gemm(qa, qb, D, 1.5, 0.5, "bf16")
        torch.cuda.synchronize()
        tg.set_policy("default")
        np.testing.assert_array_equal(C.cpu().numpy().astype(np.float64), ref)
        np.testing.assert_array_equal(D.cpu().numpy().astype(np.float64), plain)


@pytest.mark.parametrize("M,N,scaled", [(300, 272, True), (300, 272, False), (1536, 2048, True)])
def test_as_exact_as_direct_tiles(tg, M, N, scaled):
    K = 8192
    g = torch.Generator(device=DEV)
    g.manual_seed(9)
    A, B = torch.randn(M, K, generator=g, device=DEV), torch.randn(K, N, generator=g, device=DEV)
    QA, SA = tg.quantize_tiles(A, "bf16")
    QB, SB = tg.quantize_tiles(B, "bf16")
    a, b = QA.view(torch.bfloat16).double(), QB.view(torch.bfloat16).double()
    if scaled:
        a = a * SA.double().repeat_interleave(128, 0)[:M].repeat_interleave(128, 1)[:, :K]
        b = b * SB.double().repeat_interleave(128, 0)[:K].repeat_interleave(128, 1)[:, :N]
    ref = a @ b

    def error(sid):
        tg.set_policy(f"force:{sid}")
        C = torch.empty(M, N, device=DEV)
        if scaled:
            tg.gemm_scaled(QA, SA, QB, SB, C, 1.0, 0.0, "bf16")
        else:
            tg.gemm(QA, QB, C, 1.0, 0.0, "bf16")
        torch.cuda.synchronize()
        tg.set_policy("default")
        return float((C.double() - ref).norm() / ref.norm())

    direct = error([sid for sid, i in tg.schedules("bf16") if i["vec"] == 4 and i["BM"] == 64][0])
    for sid in _folded(tg):
        e = error(sid)
        print(f"{M}x{N}x{K} scaled {scaled} {tg.schedule_key(sid)}: {e:.3e}, direct {direct:.3e}", flush=True)
        assert e <= 1.25 * direct
