"""Plain solves of systems too long for one workgroup: the cut form (the
unknowns of a few rows first, from the rows of the inverse around them, then
the segments between them on their own) against the oracle, at ragged lengths
and last segments, odd batches, partial groups and unaligned rows, and for
periodic matrices of any length; nothing outside the right-hand sides is
written."""
import numpy as np
import pytest
import torch

import oracle
from paper_1909_04539_amd import sbs, workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = {torch.float64: 1e-12, torch.float32: 2e-5}


def matrix(kind, n, which):
    rng = np.random.default_rng(n)
    if kind == 13:
        s = {"constant": 0.5, "stiff": 20.0, "slow": 200.0}.get(which)
        if s is not None:
            return np.stack([np.full(n, -s), np.full(n, 1 + 2 * s), np.full(n, -s)])
        a, c = rng.uniform(-1, 1, n), rng.uniform(-1, 1, n)
        return np.stack([a, np.abs(a) + np.abs(c) + rng.uniform(1, 2, n), c])
    if which == "constant":
        return W.diffusion_bands(n, 0.5) if kind == 3 else W.hyperdiffusion_bands(n, 0.9)
    if which == "stiff":  # rows of the inverse 150 rows wide on either side
        return W.diffusion_bands(n, 20.0) if kind == 3 else W.hyperdiffusion_bands(n, 20.0)
    if which == "slow":   # wider than the windows kept: no cut form
        return W.diffusion_bands(n, 200.0) if kind == 3 else W.hyperdiffusion_bands(n, 2000.0)
    if kind == 3:
        return W.tri_dominant_bands(rng, n)
    B = rng.uniform(-1, 1, (5, n))
    B[2] = np.sum(np.abs(np.delete(B, 2, axis=0)), axis=0) + rng.uniform(1, 2, n)
    return W.zero_outside(B)


def colrel(x, ref):
    return float(np.max(np.max(np.abs(x - ref), axis=0) / np.max(np.abs(ref), axis=0)))


@pytest.mark.parametrize("kind,n,which", [
    (3, 3001, "random"), (3, 5141, "random"), (3, 8192, "constant"), (3, 5000, "stiff"), (3, 5000, "slow"),
    (5, 1541, "random"), (5, 2001, "random"), (5, 5140, "constant"), (5, 5143, "random"), (5, 5000, "stiff"),
    (5, 5000, "slow"), (13, 513, "random"), (13, 514, "random"), (13, 1000, "constant"), (13, 1027, "random"),
    (13, 2600, "random"), (13, 2001, "stiff"), (13, 4999, "random"), (13, 3001, "slow")])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("m", [1, 2, 3, 33, 64, 513])
def test_cut_solves_match_oracle(kind, n, which, dtype, m):
    print(f"case kind={kind} n={n} {which} m={m} {dtype}", flush=True)
    B = matrix(kind, n, which)
    rhs = np.random.default_rng(n + m).uniform(-1, 1, (n, m))
    guard = 257  # an odd offset: rows start at odd elements
    buf = torch.full((n * m + 2 * guard,), 7.25, dtype=dtype, device=DEV)
    x = buf[guard:guard + n * m].view(n, m)
    x.copy_(torch.from_numpy(rhs))
    rhs = x.cpu().double().numpy()
    with sbs.SharedLhs(kind, B) as h:
        h.solve(x)
        torch.cuda.synchronize()
    tol = TOL[dtype] * (100 if which in ("stiff", "slow") and dtype == torch.float32 else 1)
    assert colrel(x.cpu().double().numpy(), oracle.solve(kind, B, rhs)) <= tol
    assert torch.all(buf[:guard] == 7.25) and torch.all(buf[guard + n * m:] == 7.25)


def test_cut_solve_of_a_batch_that_fills_the_chip():
    # several groups per workgroup, odd batch, sampled columns
    for kind, n, m, which in ((5, 2001, 20001, "random"), (3, 8192, 4097, "constant")):
        B = matrix(kind, n, which)
        x = torch.rand((n, m), dtype=torch.float64, device=DEV) * 2 - 1
        cols = np.unique(np.r_[0, 1, 31, 32, 33, m - 34, m - 2, m - 1, np.random.default_rng(3).integers(0, m, 60)])
        at = torch.from_numpy(cols).to(DEV)
        rhs = x[:, at].cpu().numpy()
        with sbs.SharedLhs(kind, B) as h:
            h.solve(x)
            torch.cuda.synchronize()
        assert colrel(x[:, at].cpu().numpy(), oracle.solve(kind, B, rhs)) <= 1e-12
