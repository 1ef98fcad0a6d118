"""f32 in-place 128 x 128 tiles whose last ones run as quarters of 64 x 64.

C = alpha*A*B + beta*C bit-exact on small integers against the FP64 oracle, and bitwise equal
to 64 x 64 tiles on U[-1, 1] inputs (both add every product in the order of k), around the
tile counts that decide: 256 and 257 tiles, 192 and 193 past a whole round, a ragged last
tile whose quarters lie partly or wholly outside C, and a sub-matrix at an odd offset.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1804_10694_amd import inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("shape", [
    (2048, 2048, 40),      # 256 tiles
    (300, 10960, 33),      # 3 x 86 = 258: quarters below row 300 are outside
    (4096, 1793, 17),      # 32 x 15 = 480: 224 over, whole tiles
    (1920, 3800, 19),      # 15 x 30 = 450: 194 over
    (2048, 3580, 50),      # 16 x 28 = 448: 192 over
    (2433, 3201, 16),      # 20 x 26 = 520, columns 3200 ..: one of 128
], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("offset", [0, 1])
def test_rest_tiles(shape, offset):
    from paper_1804_10694_amd import tgemm as tg
    tg.set_policy("default")
    M, N, K = shape
    ids = {i["BM"]: s for s, i in tg.schedules("f32") if i["inplace"]}

    def dev(x):
        buf = torch.zeros(x.shape[0], x.shape[1] + 3, device=DEV)
        v = buf[:, offset:offset + x.shape[1]]
        v.copy_(x)
        return v

    A, B, C0 = inputs.integer_inputs(M, N, K, seed=90)
    ref = oracle.gemm(A, B, C0, 1.5, 0.5)
    for sid in (None, ids[128]):
        print(f"rest {shape} offset {offset} schedule {sid}", flush=True)
        C = dev(C0)
        if sid is None:
            tg.gemm(dev(A), dev(B), C, 1.5, 0.5, "f32")
        else:
            tg.gemm_with_schedule(dev(A), dev(B), C, 1.5, 0.5, "f32", sid)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(C.cpu().numpy().astype(np.float64), ref)
    g = torch.Generator().manual_seed(91)
    A, B = dev(2 * torch.rand(M, K, generator=g) - 1), dev(2 * torch.rand(K, N, generator=g) - 1)
    out = [torch.full((M, N), float("nan"), device=DEV) for _ in range(2)]
    tg.gemm_with_schedule(A, B, out[0], 1.0, 0.0, "f32", ids[128])
    tg.gemm_with_schedule(A, B, out[1], 1.0, 0.0, "f32", ids[64])
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1])
