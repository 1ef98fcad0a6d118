"""Stream-K launches of more tiles than workgroups: whole rounds first, the rest in ranges.

C = alpha*A*B + beta*C bit-exact against the FP64 oracle on small integers (every partial
sum is an integer below 2^24, so neither the split nor the order of the sums changes it),
at tile counts around whole rounds (256 workgroups for 256 x 256 tiles, 512 for 128 x 256,
1024 for 128 x 128): none left, one, a sixteenth, an odd part of a round, one less than a round; and at
depths of one panel and of fewer panels than workgroups share.
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


def _codes(X, dtype):
    if dtype == "fp8":
        return torch.from_numpy(P.e4m3_encode(X.numpy().astype(np.float64)))
    return torch.from_numpy(P.bf16_bits(X.numpy()).view(np.int16))


@pytest.mark.parametrize("dtype", ["f32", "x3", "bf16", "fp8"])
@pytest.mark.parametrize("shape", [
    (4096, 4096, 33),     # 256, 512, 1024 tiles
    (100, 65700, 20),     # 257 of 256 x 256
    (4100, 4097, 150),    # 289, 33 x 17, 33 x 33
    (4090, 4350, 270),    # 272: 16 ranges a tile
    (7900, 4090, 100),    # 496, 992, 1984
], ids=lambda s: "x".join(map(str, s)))
def test_rounds_bit_exact_on_integers(tg, dtype, shape):
    M, N, K = shape
    A, B, C0 = inputs.integer_inputs(M, N, K, seed=70, r=8)
    ref = oracle.gemm(A, B, C0, 1.5, 0.5)
    Ad, Bd = (A.to(DEV), B.to(DEV)) if dtype in ("f32", "x3") else (_codes(A, dtype).to(DEV), _codes(B, dtype).to(DEV))
    for sid, info in tg.schedules(dtype):
        if not info["split"]:
            continue
        for _ in range(2):  # the counters are zero again after a launch
            print(f"stream-K rounds {tg.schedule_key(sid)} {shape}", flush=True)
            C = C0.to(DEV)
            tg.gemm_with_schedule(Ad, Bd, C, 1.5, 0.5, dtype, sid)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(C.cpu().numpy().astype(np.float64), ref, err_msg=tg.schedule_key(sid))


def test_shared_choice_without_workspace(tg):
    # the rule's stream-K choice, and what runs in its place where it can have no
    # workspace: on a stream first seen under capture, and in the call that allocates nothing
    dtype, (M, N, K) = "x3", (4096, 4352, 2000)
    A, B, C0 = inputs.integer_inputs(M, N, K, seed=71, r=8)
    assert tg.schedule_info(tg.select_schedule(M, N, K, dtype)[0])["split"] == 1
    ref = oracle.gemm(A, B, C0, 1.0, 0.5)
    Ad, Bd, Cd = A.to(DEV), B.to(DEV), C0.to(DEV)
    C = Cd.clone()
    tg.gemm(Ad, Bd, C, 1.0, 0.5, dtype)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(C.cpu().numpy().astype(np.float64), ref)
    C = Cd.clone()
    tg.gemm_noalloc(Ad, Bd, C, 1.0, 0.5, dtype)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(C.cpu().numpy().astype(np.float64), ref)
    C = Cd.clone()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        tg.gemm(Ad, Bd, C, 1.0, 0.5, dtype)
    for _ in range(3):
        C.copy_(Cd)
        graph.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(C.cpu().numpy().astype(np.float64), ref)
