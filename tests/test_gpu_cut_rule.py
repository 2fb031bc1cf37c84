"""Batches on both sides of the lines where AUTO leaves the whole-system forms
for the cut form: the general sweeps' results to the rounding of the type."""
import numpy as np
import pytest
import torch

from paper_1909_04539_amd import sbs, workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("kind,n", [(3, 1025), (3, 1728), (3, 1729), (3, 2048), (3, 2049), (5, 1024), (5, 1025),
                                    (5, 1600), (5, 2048), (5, 2049)])
@pytest.mark.parametrize("m", [1, 2, 127, 128, 1501, 4097])
@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-13), (torch.float32, 1e-5)])
def test_auto_matches_the_sweeps(kind, n, m, dtype, tol):
    print(f"case kind={kind} n={n} m={m} dtype={dtype}", flush=True)
    B = W.diffusion_bands(n, 0.5) if kind == 3 else W.hyperdiffusion_bands(n, 0.5)
    b = torch.from_numpy(np.random.default_rng(n + m).uniform(-1, 1, (n, m))).to(dtype)
    with sbs.SharedLhs(kind, B) as h:
        x = h.solve(b.to(DEV)).cpu().double()
        y = h.solve(b.to(DEV), variant=sbs.VARIANT_STREAM).cpu().double()
    # diagonally dominant systems (condition below 20): some tens of roundings
    err = float(((x - y).abs().amax(0) / y.abs().amax(0)).max())
    assert err <= tol, err
