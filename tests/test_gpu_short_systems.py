"""Short systems in large batches, where a workgroup has few lanes: part of a
wave, whole waves with lanes that have no block, odd batches and partial last
groups; solves and Crank-Nicolson steps against the oracle, and nothing outside
the array is written."""
import numpy as np
import pytest
import torch

import oracle
from paper_1909_04539_amd import sbs
from test_cut_host import colrel, constant, dominant

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def run(kind, n, m, which, dtype, steps, tol):
    print(f"case kind={kind} n={n} m={m} {which} {dtype} steps={steps}", flush=True)
    B = dominant(kind, n, n) if which == "random" else constant(kind, n)
    guard = 63
    buf = torch.full((n * m + 2 * guard,), 7.25, dtype=dtype, device=DEV)
    x = buf[guard:guard + n * m].view(n, m)
    x.uniform_(-1, 1)
    cols = np.unique(np.r_[0, 1, 63, 64, m // 2, m - 3, m - 2, m - 1, np.random.default_rng(m).integers(0, m, 40)])
    at = torch.from_numpy(cols).to(DEV)
    rhs = x[:, at].double().cpu().numpy()
    with sbs.SharedLhs(kind, B) as h:
        h.cn_step(x, steps) if steps else h.solve(x)
        torch.cuda.synchronize()
    ref = oracle.cn_steps(kind, B, rhs, steps) if steps else oracle.solve(kind, B, rhs)
    assert colrel(x[:, at].double().cpu().numpy(), ref) <= tol
    assert torch.all(buf[:guard] == 7.25) and torch.all(buf[guard + n * m:] == 7.25)


# 1 to 13 blocks; batches on both sides of the lines between shapes
@pytest.mark.parametrize("kind,n", [(3, 17), (3, 33), (3, 72), (3, 130), (3, 200), (3, 300), (5, 17), (5, 33), (5, 57),
                                    (5, 84), (5, 130), (5, 200), (5, 400), (13, 48), (13, 96), (13, 160)])
@pytest.mark.parametrize("m", [3001, 8192, 65537, 131072])
@pytest.mark.parametrize("which", ["constant", "random"])
def test_fp64(kind, n, m, which):
    run(kind, n, m, which, torch.float64, 0, 1e-13)
    run(kind, n, m, which, torch.float64, 3, 1e-12)


@pytest.mark.parametrize("kind,n", [(3, 17), (3, 72), (3, 300), (5, 33), (5, 84), (5, 400), (13, 96)])
@pytest.mark.parametrize("m", [3001, 65537])
def test_fp32(kind, n, m):
    run(kind, n, m, "random", torch.float32, 0, 2e-5)
    run(kind, n, m, "random", torch.float32, 3, 2e-5)


# longer ones whose separators, one fewer than the blocks (as many, periodic),
# would lie a multiple of the LDS's banks apart
@pytest.mark.parametrize("kind,n", [(3, 512), (3, 1024), (3, 1010), (3, 2048), (13, 992), (13, 1024), (5, 1024)])
@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-12), (torch.float32, 2e-5)])
def test_separators_at_odd_strides(kind, n, dtype, tol):
    run(kind, n, 1501, "random", dtype, 2, tol)
    run(kind, n, 1501, "constant", dtype, 3, tol)
