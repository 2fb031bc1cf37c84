"""A NaN or infinity in one right-hand side: its own row's unknown is not finite,
and every other system's result is bit for bit what it is without it, in the
forms that keep systems whole and in the one that cuts them."""
import numpy as np
import pytest
import torch

from paper_1909_04539_amd import sbs
from test_cut_host import constant, dominant

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("kind", [3, 5, 13])
@pytest.mark.parametrize("n", [300, 1000, 2600])
@pytest.mark.parametrize("which", ["constant", "random"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("m", [130, 131])
def test_it_stays_in_its_system(kind, n, which, dtype, m):
    B = dominant(kind, n, n) if which == "random" else constant(kind, n)
    b = torch.from_numpy(np.random.default_rng(n).uniform(-1, 1, (n, m))).to(dtype).to(DEV)
    with sbs.SharedLhs(kind, B) as h:
        ref = h.solve(b.clone())
        for j in (0, 7, m - 1):
            others = [k for k in range(m) if k != j]
            for row in (0, 31, 200, 224, 225, 255, 256, 257, n // 2, n - 1):
                for value in (float("nan"), float("inf"), float("-inf")):
                    x = b.clone()
                    x[row, j] = value
                    h.solve(x)
                    assert not torch.isfinite(x[row, j]), (row, j, value)
                    assert torch.equal(x[:, others], ref[:, others]), (row, j, value)
