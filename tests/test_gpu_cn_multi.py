"""Several Crank-Nicolson steps in one call: the partitioned kernels keep a
group's systems in registers between the steps, so five steps are the same,
bit for bit, as two steps and then three (the same kernel and arithmetic), and
match the oracle, as five calls of one step do (which may take another shape).
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
        B = np.array([0.2, -0.8, 2.2, -0.8, 0.2] if kind == 5 else [-0.4, 1.8, -0.4])[:, None] * np.ones(n)
    else:
        rng = np.random.default_rng(seed)
        B = rng.uniform(-1, 1, (nb, n))
        B[nb // 2] = np.sum(np.abs(np.delete(B, nb // 2, axis=0)), axis=0) + rng.uniform(1, 2, n)
    return B if kind == 13 else W.zero_outside(B)


# ragged and whole last blocks, one and several blocks, partial last groups,
# odd batches; each block length and one and two systems per lane; 65 periodic
# rows have no plan (one launch per step)
@pytest.mark.parametrize("kind,n,m", [(3, 17, 5), (3, 100, 130), (3, 1000, 77), (5, 40, 3), (5, 333, 200),
                                      (5, 1000, 8193), (5, 1024, 8192), (13, 96, 33), (13, 512, 1000), (13, 65, 70),
                                      (3, 700, 12001), (5, 2000, 129), (5, 2040, 4097), (3, 3000, 64), (3, 12, 2)])
@pytest.mark.parametrize("constant", [True, False])
@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-12), (torch.float32, 1e-5)])
def test_steps_in_one_call(kind, n, m, constant, dtype, tol):
    print(f"case kind={kind} n={n} m={m} constant={constant} dtype={dtype}", flush=True)
    B = bands(kind, n, constant, n + m)
    c = torch.from_numpy(np.random.default_rng(n * m).uniform(-1, 1, (n, m))).to(dtype)
    with sbs.SharedLhs(kind, B) as h:
        one, two, many = c.to(DEV), c.to(DEV), c.to(DEV)
        for _ in range(5):
            h.cn_step(one, 1)
        h.cn_step(two, 2)
        h.cn_step(two, 3)
        h.cn_step(many, 5)
        torch.cuda.synchronize()
    assert torch.equal(two, many)
    cols = np.unique(np.r_[0, m // 2, m - 1, np.random.default_rng(m).integers(0, m, 20)])
    ref = oracle.cn_steps(kind, B, np.ascontiguousarray(c.double().numpy()[:, cols]), 5)
    for x in (many, one):
        got = x.double().cpu().numpy()[:, cols]
        err = np.max(np.max(np.abs(got - ref), axis=0) / np.max(np.abs(ref), axis=0))
        assert err <= tol, err
