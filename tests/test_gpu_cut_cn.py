"""Crank-Nicolson steps of systems too long for one workgroup: the cut form's
segments with the unknowns of the cut rows in scratch, against the oracle;
while a graph is captured the sweeps run the same steps.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1909_04539_amd import sbs, workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def bands(kind, n, constant, seed):
    nb = 5 if kind == 5 else 3
    if constant:
        return np.array([0.2, -0.8, 2.2, -0.8, 0.2] if kind == 5 else [-0.4, 1.8, -0.4])[:, None] * np.ones(n)
    rng = np.random.default_rng(seed)
    B = rng.uniform(-1, 1, (nb, n))
    B[nb // 2] = np.sum(np.abs(np.delete(B, nb // 2, axis=0)), axis=0) + rng.uniform(1, 2, n)
    return B if kind == 13 else W.zero_outside(B)


# whole and ragged last segments and blocks, a last segment of one block, odd
# and tiny batches, several groups per workgroup
@pytest.mark.parametrize("kind,n,m", [(3, 2500, 64), (3, 5001, 333), (3, 2057, 2), (5, 2500, 130), (5, 4099, 77),
                                      (5, 2100, 20001), (13, 600, 50), (13, 2500, 129), (13, 1001, 20000), (13, 65, 70)])
@pytest.mark.parametrize("constant", [True, False])
@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-12), (torch.float32, 1e-5)])
def test_steps_match_oracle(kind, n, m, constant, dtype, tol):
    print(f"case kind={kind} n={n} m={m} constant={constant} dtype={dtype}", flush=True)
    B = bands(kind, n, constant, n + m)
    if constant and kind != 13:
        B = W.zero_outside(B)
    c = torch.from_numpy(np.random.default_rng(n * m).uniform(-1, 1, (n, m))).to(dtype)
    cols = np.unique(np.r_[0, m // 2, m - 1, np.random.default_rng(m).integers(0, m, 20)])
    with sbs.SharedLhs(kind, B) as h:
        x, g, s = c.to(DEV), c.to(DEV), torch.cuda.Stream()
        h.cn_step(x, 3)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            h.cn_step(g, 3)
        g.copy_(c.to(DEV))
        graph.replay()
        torch.cuda.synchronize()
    ref = oracle.cn_steps(kind, B, np.ascontiguousarray(c.double().numpy()[:, cols]), 3)
    for y in (x, g):
        got = y.double().cpu().numpy()[:, cols]
        err = np.max(np.max(np.abs(got - ref), axis=0) / np.max(np.abs(ref), axis=0))
        assert err <= tol, err
