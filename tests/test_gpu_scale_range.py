"""Scale products that lie far apart along K: the sums of one K block cannot stand in units of
another's product, and every result stays as exact as with products alike.

Rows and columns of every second scale tile keep the scale 1, the others follow a pattern of
exponents over the K blocks (A's and B's alike, so a product's exponent is their sum).  Every
second row of A has no codes in the first K block, so nothing large hides what the others sum to.
Every element within the bound of tests/scaled_bound.py.
"""
import numpy as np
import pytest
import torch

from oracle import precision as P
from scaled_bound import scaled_error_bound

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")

PATTERNS = {
    "down": [58, -40],          # products 2^116, then 2^-80 to the end
    "up": [-58, 40],
    "zigzag": [40, -40, 40, -40, 0],
    "drift": [20, 10, 0, -10, -20, -30],   # steps of 2^20, further and further from the first
    "under": [0, -80, 0, -80],  # products below float32: 0
    "near": [0, 11, 0, -11],    # within one unit
}


@pytest.fixture(scope="module")
def tg():
    from paper_1804_10694_amd import tgemm
    tgemm.set_policy("default")
    yield tgemm
    tgemm.set_policy("default")


def _inputs(M, N, K, dtype, pattern, seed):
    rng = np.random.default_rng(seed)
    A, B = rng.uniform(-1, 1, (M, K)), rng.uniform(-1, 1, (K, N))
    A[::2, :128] = 0.0
    enc = (lambda x: P.e4m3_encode(P.e4m3_rne_sat(x))) if dtype == "fp8" else \
        (lambda x: P.bf16_bits(P.bf16_rne(x.astype(np.float32))))
    nb = -(-K // 128)
    e = PATTERNS[pattern]
    e = np.array([e[min(k, len(e) - 1)] for k in range(nb)], dtype=np.float64)
    SA = np.ones(P.scale_grid_shape(M, K), np.float32)
    SB = np.ones(P.scale_grid_shape(K, N), np.float32)
    SA[1::2, :] = 2.0 ** e
    SB[:, 1::2] = (2.0 ** e)[:, None]
    return enc(A), SA, enc(B), SB


def _check(tg, shape, dtype, pattern, sids, alpha, beta):
    M, N, K = shape
    QA, SA, QB, SB = _inputs(M, N, K, dtype, pattern, M + N + K)
    C0 = np.random.default_rng(5).uniform(-1, 1, (M, N)).astype(np.float32)
    rows = np.arange(M) if M * N * K < 10 ** 9 else np.arange(0, M, 61)
    DA = P.decode(QA[rows], dtype) * np.repeat(SA.astype(np.float64), 128, 1)[rows // 128, :K]
    ref = alpha * (DA @ P.dequantize_tiles(P.decode(QB, dtype), SB, 128)) + beta * C0[rows]
    # and one rounding more of each K block's part and of C0; products and sums below
    # float32's normal numbers, 2^-126 each
    bound = scaled_error_bound(QA, SA, QB, SB, dtype, alpha=alpha, rows=rows) + 2.0 ** -24 * np.abs(ref) \
        + abs(beta) * np.abs(C0[rows]) * 2.0 ** -23 * (-(-K // 128)) + K * 2.0 ** -126
    dev = [torch.from_numpy(x.view(np.int16) if x.dtype == np.uint16 else x).to(DEV) for x in (QA, SA, QB, SB)]
    for sid in sids:
        print(f"{dtype} {shape} {pattern} {tg.schedule_key(sid) if sid is not None else 'rule'}", flush=True)
        tg.set_policy("default" if sid is None else f"force:{sid}")
        C = torch.from_numpy(C0).to(DEV)
        tg.gemm_scaled(*dev, C, alpha, beta, dtype)
        torch.cuda.synchronize()
        tg.set_policy("default")
        got = C.cpu().numpy()[rows].astype(np.float64)
        err = np.abs(got - ref)
        assert np.all(err <= bound), \
            f"{sid}: {np.sum(~(err <= bound))} elements past the bound, {np.sum(~np.isfinite(got))} not finite"


@pytest.mark.parametrize("pattern", list(PATTERNS))
@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
def test_every_packed_schedule(tg, dtype, pattern):
    sids = [None] + [sid for sid, info in tg.schedules(dtype) if info["vec"] == 0]
    _check(tg, (300, 390, 1000), dtype, pattern, sids, 1.5, 0.5)


@pytest.mark.parametrize("pattern", ["down", "zigzag", "drift"])
@pytest.mark.parametrize("shape", [
    (300, 700, 8000),     # ranges of three panels: units change inside a K block's range
    (1500, 2900, 1500),   # ranges of several K blocks, tiles shared by two and three of them
    (4100, 4100, 600),    # whole rounds, then ranges
], ids=lambda s: "x".join(map(str, s)))
def test_stream_k(tg, shape, pattern):
    sids = [sid for sid, info in tg.schedules("bf16") if info["split"]]
    assert sids
    _check(tg, shape, "bf16", pattern, sids, 1.0, 0.0)


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("shape", [(300, 200, 700), (1000, 900, 1500), (2048, 2048, 1024)],
                         ids=lambda s: "x".join(map(str, s)))
def test_quantised_operands(tg, dtype, shape):
    # float32 inputs whose K blocks lie far apart, through the quantiser
    M, N, K = shape
    e = 2.0 ** torch.tensor([60.0] + [-40.0] * (-(-K // 128) - 1), device=DEV).repeat_interleave(128)[:K]
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    A = (torch.rand(M, K, generator=g, device=DEV) * 2 - 1) * e
    A[::2, :128] = 0
    B = (torch.rand(K, N, generator=g, device=DEV) * 2 - 1) * e[:, None]
    QA, SA = tg.quantize_tiles(A, dtype)
    QB, SB = tg.quantize_tiles(B, dtype)
    C = torch.empty(M, N, device=DEV)
    tg.gemm_scaled(QA, SA, QB, SB, C, 1.0, 0.0, dtype)
    torch.cuda.synchronize()
    tol = {"bf16": 2e-2, "fp8": 6e-2}[dtype]  # the quantisation's own error
    ref = A.double() @ B.double()
    for rows in (slice(0, None, 2), slice(1, None, 2)):
        assert float((C[rows].double() - ref[rows]).norm() / ref[rows].norm()) <= tol
