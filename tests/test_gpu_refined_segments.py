"""Mixed-precision solves of matrices that take several segments (overlapping
runs of rows solved independently, one workgroup with one wave per 32-row
block each), and served FP32 requests, whose tiles are such segments, against
the FP64 oracle of the promoted right-hand sides."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_1909_04539_amd import sbs, workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# FP32 arithmetic: the solution of the truncated FP32 factor; the corrections
# bring the FP64 residual down by the FP32 solve's relative error each
TOL = {0: 2e-5, 1: 1e-9, 2: 1e-12, 3: 1e-12}


def matrix(kind, n, which):
    rng = np.random.default_rng(n)
    if which == "slow":  # inverse decays over hundreds of rows: no segments
        return W.zero_outside(np.stack([-np.ones(n), np.full(n, 2.01), -np.ones(n)]))
    if which == "constant":
        return W.diffusion_bands(n, 0.5) if kind == 3 else W.hyperdiffusion_bands(n, 1.0)
    if kind == 3:
        return W.tri_dominant_bands(rng, n)
    B = rng.uniform(-1, 1, (5, n))
    B[2] = np.sum(np.abs(np.delete(B, 2, axis=0)), axis=0) + rng.uniform(1, 2, n)
    return W.zero_outside(B)


def colrel(x, ref):
    return float(np.max(np.max(np.abs(x - ref), axis=0) / np.max(np.abs(ref), axis=0)))


# one row past the one-workgroup sizes (560 and 512 rows), the largest two
# segments, three, ragged and many; partial groups of systems
@pytest.mark.parametrize("kind,n", [(3, 561), (3, 992), (3, 993), (3, 2900), (3, 8192), (5, 513), (5, 800),
                                    (5, 865), (5, 1500), (5, 5003), (3, 20011)])
@pytest.mark.parametrize("which", ["random", "constant"])
@pytest.mark.parametrize("m,sweeps", [(1, 2), (65, 0), (130, 1), (64, 3)])
def test_refined_by_segments(kind, n, which, m, sweeps):
    print(f"case kind={kind} n={n} {which} m={m} sweeps={sweeps}", flush=True)
    B = matrix(kind, n, which)
    b = np.random.default_rng(n + m).uniform(-1, 1, (n, m)).astype(np.float32)
    with sbs.SharedLhs(kind, B) as h:
        t = torch.from_numpy(b).to(DEV)
        x = h.solve_refined(t, sweeps=sweeps)
        torch.cuda.synchronize()
        assert torch.equal(t.cpu(), torch.from_numpy(b))
    assert colrel(x.cpu().numpy(), oracle.refine_reference(kind, B, b)) <= TOL[sweeps]


def test_slowly_decaying_inverse_keeps_the_other_forms():
    n, m = 3000, 70
    B = matrix(3, n, "slow")
    b = np.random.default_rng(1).uniform(-1, 1, (n, m)).astype(np.float32)
    with sbs.SharedLhs(3, B) as h:
        x = h.solve_refined(torch.from_numpy(b).to(DEV), sweeps=3)
        torch.cuda.synchronize()
    # condition number 400: the FP32 solve leaves up to 400 * 1e-5 of the
    # error per correction, three of them leave FP64 rounding
    assert colrel(x.cpu().numpy(), oracle.refine_reference(3, B, b)) <= 1e-10


def test_served_requests_by_segments():
    # one and several segments, both workgroup sizes, systems that fill no
    # whole group of 64, and a matrix without segments
    mats = [(3, 64, "random"), (3, 65, "random"), (3, 256, "constant"), (3, 257, "random"), (3, 513, "random"),
            (5, 100, "random"), (5, 448, "constant"), (5, 449, "random"), (5, 2000, "constant"), (3, 6000, "random"),
            (3, 3000, "slow")]
    L = sbs.lib()
    srv = ctypes.c_void_p()
    assert L.sbs_server_create(1 << 30, 2, 0, ctypes.byref(srv)) == 0
    hs, reqs = [], []
    for k, (kind, n, which) in enumerate(mats):
        B = matrix(kind, n, which)
        h = sbs.SharedLhs(kind, B)
        i = ctypes.c_int32()
        assert L.sbs_server_register(srv, h.handle, ctypes.byref(i)) == 0
        hs.append(h)
        for m in (1, 64, 200):
            b = np.random.default_rng(100 * k + m).uniform(-1, 1, (n, m)).astype(np.float32)
            reqs.append((kind, B, which, i.value, b, torch.from_numpy(b).to(DEV)))
    torch.cuda.synchronize()
    tickets = []
    for kind, B, which, i, b, t in reqs:
        tk = ctypes.c_uint64()
        assert L.sbs_server_submit(srv, i, t.data_ptr(), t.shape[1], sbs.SBS_F32, ctypes.byref(tk)) == 0
        tickets.append(tk)
    for (kind, B, which, i, b, t), tk in zip(reqs, tickets):
        print(f"case served kind={kind} n={b.shape[0]} m={b.shape[1]} {which}", flush=True)
        assert L.sbs_server_wait(srv, tk, 30_000_000, None, None) == 0
        out = torch.empty(b.shape, dtype=torch.float64, device=DEV)
        assert L.sbs_server_fetch(srv, tk, out.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        assert L.sbs_server_release(srv, tk) == 0
        err = colrel(out.cpu().numpy(), oracle.refine_reference(kind, B, b))
        assert err <= (1e-6 if which == "slow" else 1e-12), (kind, b.shape, which, err)
    assert L.sbs_server_destroy(srv) == 0
    for h in hs:
        h.close()
