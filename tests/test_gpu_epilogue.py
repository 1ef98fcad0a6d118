"""The epilogue of the gemm kernels on blocks that end within M and on blocks that do not.

C = alpha*A*B + beta*C bit-exact on small integers against the FP64 oracle, at row counts
around the 32-row blocks and with row strides of C on both sides of the limits of its 32-bit
offsets (2^24 for a block's rows as scalar offsets, 2^25 for a row's range); every
kernel family of f32 and x3, and what lies beside C stays as it was.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1804_10694_amd import inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _one_of_each(tg, dtype):
    seen = {}
    for sid, i in tg.schedules(dtype):
        seen.setdefault((i["vec"], i["split"], i["inplace"], i["mfma"]), sid)
    return sorted(seen.values())


@pytest.mark.parametrize("dtype", ["f32", "x3"])
@pytest.mark.parametrize("M,ldc", [(31, 48), (32, 48), (64, 48), (300, 48), (33, (1 << 24) - 8), (64, (1 << 24) - 8),
                                   (64, 1 << 24), (35, 1 << 25)])
def test_block_rows_and_strides(dtype, M, ldc):
    from paper_1804_10694_amd import tgemm as tg
    tg.set_policy("default")
    N, K = 40, 24
    A, B, C0 = inputs.integer_inputs(M, N, K, seed=80 + M)
    Ad, Bd = A.to(DEV), B.to(DEV)
    buf = torch.empty((M - 1) * ldc + N + 8, device=DEV)
    wide = buf.as_strided((M, N + 8), (ldc, 1))
    for beta in (0.0, 0.5):
        ref = oracle.gemm(A, B, C0, 1.5, beta)
        for sid in [None] + _one_of_each(tg, dtype):
            print(f"epilogue {dtype} M={M} ldc={ldc} beta={beta} schedule {sid}", flush=True)
            wide.fill_(7.0)
            C = wide[:, :N]
            C.copy_(C0)
            if sid is None:
                tg.gemm(Ad, Bd, C, 1.5, beta, dtype)
            else:
                tg.gemm_with_schedule(Ad, Bd, C, 1.5, beta, dtype, sid)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(C.cpu().numpy().astype(np.float64), ref)
            assert (wide[:, N:] == 7.0).all()
