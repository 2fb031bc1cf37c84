"""Mixed-precision solves on short overlapping segments (two workgroups per
CU), of matrices that one workgroup could hold whole and longer ones, at batch
sizes on both sides of the one that fills the GPU, against the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1909_04539_amd import sbs, workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# one row past the one-workgroup sizes (256 and 224), whole and ragged blocks,
# the largest single workgroups, and the first sizes past them
@pytest.mark.parametrize("kind,n", [(3, 257), (3, 289), (3, 400), (3, 481), (3, 512), (3, 513), (3, 1025),
                                    (5, 225), (5, 289), (5, 400), (5, 449), (5, 512), (5, 513), (5, 1025)])
@pytest.mark.parametrize("m,sweeps", [(3, 2), (16384, 2), (16385, 2), (70, 1)])
def test_refined_on_short_segments(kind, n, m, sweeps):
    print(f"case kind={kind} n={n} m={m} sweeps={sweeps}", flush=True)
    B = W.diffusion_bands(n, 0.5) if kind == 3 else W.hyperdiffusion_bands(n, 0.3)
    b = np.random.default_rng(n + m).uniform(-1, 1, (n, m)).astype(np.float32)
    with sbs.SharedLhs(kind, B) as h:
        x = h.solve_refined(torch.from_numpy(b).to(DEV), sweeps=sweeps)
        torch.cuda.synchronize()
    cols = np.unique(np.r_[0, m // 2, m - 1, np.random.default_rng(m).integers(0, m, 30)])
    got = x.cpu().numpy()[:, cols]
    ref = oracle.refine_reference(kind, B, np.ascontiguousarray(b[:, cols]))
    # FP32 solves; each correction brings the error down by their relative error
    err = np.max(np.max(np.abs(got - ref), axis=0) / np.max(np.abs(ref), axis=0))
    assert err <= (1e-12 if sweeps == 2 else 1e-9), err
