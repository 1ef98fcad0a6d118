"""tgemm_noalloc where packed bf16 and e4m3 operands do not fit its array: the rule's choice gives
way to direct tiles (sizes it took before it packed them), a schedule that a policy names is
refused."""
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


@pytest.mark.parametrize("dtype,M,N,K", [("bf16", 190000, 20, 330), ("fp8", 270000, 20, 420)])
def test_policy_choice_is_refused(tg, dtype, M, N, K):
    A, B, _ = inputs.integer_inputs(M, N, K, seed=77, r=8)
    enc = (lambda x: torch.from_numpy(P.e4m3_encode(x.numpy().astype(np.float64)))) if dtype == "fp8" else \
        (lambda x: torch.from_numpy(P.bf16_bits(x.numpy()).view(np.int16)))
    Ad, Bd, C = enc(A).to(DEV), enc(B).to(DEV), torch.zeros(M, N, device=DEV)
    sid = tg.select_schedule(M, N, K, dtype)[0]
    assert tg.schedule_info(sid)["vec"] == 0
    tg.gemm_noalloc(Ad, Bd, C, 1.0, 0.0, dtype)
    torch.cuda.synchronize()
    rows = np.arange(0, M, 997)
    np.testing.assert_array_equal(C.cpu().numpy()[rows].astype(np.float64),
                                  oracle.gemm_rows(A, B, None, 1.0, 0.0, rows))
    other = [s for s, i in tg.schedules(dtype) if i["vec"] == 0 and not i["split"] and s != sid][0]
    tg.set_policy(f"force:{other}")
    with pytest.raises(tg.TgemmError) as e:
        tg.gemm_noalloc(Ad, Bd, C, 1.0, 0.0, dtype)
    tg.set_policy("default")
    assert e.value.status == tg.SCRATCH_TOO_SMALL
