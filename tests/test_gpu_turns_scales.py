"""Scales of the e4m3 tiles that take turns (256 x 256 packed schedules), against every other
packed schedule's bound.

Those tiles move their sums to another unit at a K block only where they have to: between powers
of two the exponents alone move, an unchanged product of mantissas moves nothing, anything else
divides.  The scales here go through every such step in both directions, another sequence in every
scale tile of a workgroup.  Every element within the bound of tests/scaled_bound.py.
"""
import numpy as np
import pytest
import torch

from oracle import precision as P
from scaled_bound import scaled_error_bound

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.fixture(scope="module")
def tg():
    from paper_1804_10694_amd import tgemm
    tgemm.set_policy("default")
    yield tgemm
    tgemm.set_policy("default")


def _scales(rows, cols, kind, axis, rng):
    """A scale grid whose sequence along K (axis) follows `kind`, shifted from line to line."""
    shape = P.scale_grid_shape(rows, cols)
    nk, lines = shape[axis], shape[1 - axis]
    seq = {
        # powers of two, others, an unchanged product of mantissas under another exponent, back
        "steps": [1.0, 4.0, 0.25, 1.5, 1.5, 3.0, 0.75, 1.0, 2.0, 1.25, 0.5, 1.25, 1.0],
        # products of mantissas of 2 and more (1.5 * 1.5, 1.75 * 1.75)
        "large": [1.5, 1.75, 1.5, 1.0, 1.75, 1.75, 8.0],
        # wide apart, powers of two and not
        "wide": [2.0 ** 60, 1.3 * 2.0 ** -40, 2.0 ** -60, 1.7 * 2.0 ** 50, 1.0],
    }.get(kind)
    S = np.empty((lines, nk), np.float32)
    for i in range(lines):
        S[i] = rng.uniform(0.3, 3.0, nk) if seq is None else [seq[(k + 2 * i) % len(seq)] for k in range(nk)]
        if kind == "random":  # half of them powers of two
            p = rng.random(nk) < 0.5
            S[i, p] = 2.0 ** rng.integers(-3, 4, int(p.sum()))
    return np.ascontiguousarray(S if axis == 1 else S.T)


@pytest.mark.parametrize("kind", ["steps", "large", "wide", "random"])
@pytest.mark.parametrize("shape", [(300, 390, 1700), (520, 260, 257), (256, 256, 100)],
                         ids=lambda s: "x".join(map(str, s)))
def test_scale_sequences(tg, shape, kind):
    M, N, K = shape
    rng = np.random.default_rng(K)
    QA = P.e4m3_encode(P.e4m3_rne_sat(rng.uniform(-1, 1, (M, K))))
    QB = P.e4m3_encode(P.e4m3_rne_sat(rng.uniform(-1, 1, (K, N))))
    SA, SB = _scales(M, K, kind, 1, rng), _scales(K, N, kind, 0, rng)
    ref = P.gemm_scaled_expected(QA, SA, QB, SB, None, 1.0, 0.0, "fp8")
    bound = scaled_error_bound(QA, SA, QB, SB, "fp8")
    dev = [torch.from_numpy(x).to(DEV) for x in (QA, SA, QB, SB)]
    packed = [sid for sid, info in tg.schedules("fp8") if info["vec"] == 0]
    assert any(tg.schedule_info(s)["BM"] == 256 and tg.schedule_info(s)["BN"] == 256 for s in packed)
    for sid in packed:
        print(f"fp8 {shape} {kind} {tg.schedule_key(sid)}", flush=True)
        tg.set_policy(f"force:{sid}")
        C = torch.full((M, N), float("nan"), device=DEV)
        tg.gemm_scaled(*dev, C, 1.0, 0.0, "fp8")
        torch.cuda.synchronize()
        tg.set_policy("default")
        err = np.abs(C.cpu().numpy().astype(np.float64) - ref)
        assert np.all(err <= bound), f"{sid}: {np.sum(~(err <= bound))} elements past the bound"
