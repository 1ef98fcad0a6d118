"""The network's fused kernels (few tiles) and the line to the gemm-by-gemm path, against the
FP64 oracle, at widths and row counts on both sides of a 32 x 32 tile and of a 64-deep turn
of the K waves.  Bars as for the other network tests: normwise 1e-4 for outputs and gradients
per layer, 1e-5 for the loss.
"""
import numpy as np
import pytest
import torch

import oracle
from oracle import mlp as O

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")

CASES = [([5, 1], 3), ([1, 1, 1], 1), ([3, 31, 65, 1], 33), ([22, 130, 40, 1], 1000), ([64, 32, 32, 1], 4097),
         ([17, 512, 512, 1], 63),
         ([8, 2048, 1], 65),       # 1024 tiles of 64 x 64: the last size of the fused kernels
         ([8, 2049, 1], 65),       # past it
         ([6, 64, 1], 65537)]      # past it by rows


@pytest.mark.parametrize("dims,rows", CASES)
def test_step_and_forward_match_oracle(dims, rows):
    from paper_1804_10694_amd import tgemm as tg
    r = np.random.default_rng(sum(dims) + rows)
    parts = []
    for i, o in zip(dims[:-1], dims[1:]):
        parts += [r.standard_normal(i * o) * np.sqrt(2.0 / i), r.standard_normal(o) * 0.1]
    p = np.concatenate(parts).astype(np.float32)
    X = r.standard_normal((rows, dims[0])).astype(np.float32)
    y = r.standard_normal(rows).astype(np.float32)
    P, Xd, yd = (torch.from_numpy(a).to(DEV) for a in (p, X, y))
    G, m, v = (torch.full_like(P, float("nan")), torch.zeros_like(P), torch.zeros_like(P))
    loss, work = torch.zeros(1, device=DEV), tg.mlp_workspace(dims, rows)
    work.fill_(float("nan"))
    out = tg.mlp_forward(dims, P, Xd, work=work)
    ref, _ = O.forward(p.astype(np.float64), dims, X.astype(np.float64))
    assert oracle.normwise_error(out.cpu().numpy(), ref) <= 1e-4
    work.fill_(float("nan"))
    tg.mlp_train_step(dims, P, G, m, v, 1, 0.0, Xd, yd, loss, work)
    L, g = O.gradients(p.astype(np.float64), dims, X.astype(np.float64), y.astype(np.float64))
    assert abs(loss.item() - L) <= 1e-5 * abs(L)
    got, off = G.cpu().numpy(), 0
    for i, o in zip(dims[:-1], dims[1:]):
        n = i * o + o
        assert oracle.normwise_error(got[off:off + n], g[off:off + n]) <= 1e-4
        off += n
    assert torch.equal(P.cpu(), torch.from_numpy(p))
