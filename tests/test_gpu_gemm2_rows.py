"""The back-to-back gemm over row counts of its two workgroup heights and edges of its panels.

E = alpha * act(A B) D + beta * E bit-exact against the FP64 oracle on small integers (bars
as in test_gpu_gemm2.py).  Rows: below one workgroup of 32 and of 64, and past whole rounds
(768 workgroups of 64 for N1 <= 128, 512 above) by a part of a 32-row workgroup, by half a
round and by more (all 64-row ones).  K and N1 around the 32-deep panels, fewer and more than
the ring holds; N2 around the 128- and 256-column chunks.
"""
import numpy as np
import pytest
import torch

from oracle import gemm2 as OG

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")

SHAPES = [
    (31, 1, 1, 1), (33, 31, 32, 128), (63, 32, 33, 129), (96, 33, 127, 255), (128, 95, 128, 257),
    (97, 129, 129, 384), (160, 257, 160, 385), (224, 300, 255, 513), (64, 64, 256, 640),
    (768 * 64 + 5, 33, 100, 130), (768 * 64 + 384 * 64 + 1, 20, 65, 7),
    (512 * 64 + 33, 40, 130, 140), (512 * 64 + 256 * 64, 33, 200, 9), (512 * 64 + 257 * 64 - 1, 16, 250, 33),
]


@pytest.mark.parametrize("dtype", ["f32", "x3"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_rows_and_panels(dtype, shape):
    from paper_1804_10694_amd import tgemm as tg
    M, K, N1, N2 = shape
    print(f"gemm2 rows {dtype} {shape}", flush=True)
    g = torch.Generator().manual_seed(sum(shape))
    A, B, D, E0 = (torch.randint(-4, 5, s, generator=g).float() for s in ((M, K), (K, N1), (N1, N2), (M, N2)))
    ref = OG.gemm2(A, B, D, E0, 1.5, 0.5, True)
    E = E0.to(DEV)
    tg.gemm2(A.to(DEV), B.to(DEV), D.to(DEV), E, 1.5, 0.5, True, dtype)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(E.cpu().numpy().astype(np.float64), ref)
