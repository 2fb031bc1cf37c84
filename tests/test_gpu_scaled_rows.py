"""Matrices whose rows are scaled unevenly, right-hand sides with them: the
solution does not change, and solves on the GPU keep their digits (the windows
around a cut and the product with S^-1 drop entries by their effect on the
solution)."""
import numpy as np
import pytest
import torch

from paper_1909_04539_amd import sbs
from test_cut_host import colrel, dominant, matvec, scales

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("kind", [3, 5, 13])
@pytest.mark.parametrize("n", [1024, 2600])
@pytest.mark.parametrize("which", ["below", "above", "scattered"])
@pytest.mark.parametrize("K", [1e4, 1e12])
def test_solves(kind, n, which, K):
    m = 130
    x = np.random.default_rng(n).uniform(-1, 1, (n, m))
    for r in (128, 222, 250, 258):
        print(f"case kind={kind} n={n} {which} K={K} r={r}", flush=True)
        B = dominant(kind, n, r) * scales(n, which, K, r)
        b = torch.from_numpy(matvec(kind, B, x)).to(DEV)
        with sbs.SharedLhs(kind, B) as h:
            h.solve(b)
            torch.cuda.synchronize()
        assert colrel(b.cpu().numpy(), x) <= 2e-14
