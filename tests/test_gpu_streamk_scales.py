"""Stream-K forms of bf16 and e4m3 with scales that are not powers of two: the sum of a shared
tile does not depend on which of its workgroups finishes last.

The finisher adds its own sums from registers and the others' as they stored them; with scale
products that round, both have to round alike.  Bitwise-equal repeats, and every element within
the bound of tests/scaled_bound.py (plus one rounding for each range added).
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


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("shape", [(300, 270, 2100), (1100, 1400, 1153)], ids=lambda s: "x".join(map(str, s)))
def test_repeats_are_bitwise_equal(tg, dtype, shape):
    M, N, K = shape
    rng = np.random.default_rng(M)
    A, B = rng.uniform(-1, 1, (M, K)), rng.uniform(-1, 1, (K, N))
    enc = (lambda x: P.e4m3_encode(P.e4m3_rne_sat(x))) if dtype == "fp8" else \
        (lambda x: P.bf16_bits(P.bf16_rne(x.astype(np.float32))))
    QA, QB = enc(A), enc(B)
    SA = rng.uniform(0.3, 3.0, P.scale_grid_shape(M, K)).astype(np.float32)
    SB = rng.uniform(0.3, 3.0, P.scale_grid_shape(K, N)).astype(np.float32)
    rows = np.arange(0, M, 37)
    ref = (P.decode(QA[rows], dtype) * np.repeat(SA.astype(np.float64), 128, 1)[rows // 128, :K]) \
        @ P.dequantize_tiles(P.decode(QB, dtype), SB, 128)
    panels = -(-K // 64)
    bound = scaled_error_bound(QA, SA, QB, SB, dtype, rows=rows)
    bound += 2.0 ** -24 * panels * np.abs(ref).max()
    dev = [torch.from_numpy(x.view(np.int16) if x.dtype == np.uint16 else x).to(DEV) for x in (QA, SA, QB, SB)]
    sids = [sid for sid, info in tg.schedules(dtype) if info["split"]]
    assert sids
    for sid in sids:
        print(f"{dtype} {shape} {tg.schedule_key(sid)}", flush=True)
        tg.set_policy(f"force:{sid}")
        first = None
        for _ in range(30):
            C = torch.full((M, N), float("nan"), device=DEV)
            tg.gemm_scaled(*dev, C, 1.0, 0.0, dtype)
            torch.cuda.synchronize()
            first = C if first is None else first
            assert torch.equal(C, first)
        tg.set_policy("default")
        err = np.abs(first.cpu().numpy()[rows].astype(np.float64) - ref)
        assert np.all(err <= bound), f"{sid}: {np.sum(~(err <= bound))} elements past the bound"
