"""The solver's work as its users have it done, for timing and for checking.

Every case goes through the package's public entry points: plain solves in
place (tridiagonal, pentadiagonal, periodic; FP64 and FP32), Crank-Nicolson
steps, ADI steps, mixed-precision solves, and requests served by the request
loop.  A program keeps the factored matrix (one handle for many right-hand
sides); right-hand sides live on the GPU and are solved in place, as in a
time-stepping loop.

Matrices
  hyper    the Crank-Nicolson matrix of hyperdiffusion, constant bands
           (s, -4s, 1 + 6s, -4s, s), truncated ends
  diff     the Crank-Nicolson matrix of diffusion, constant bands
           (-s, 1 + 2s, -s), truncated or periodic
  var      the same operators with a coefficient that varies along the axis
           (I + D^T K D and I + D2^T K D2, K drawn from the seed): every row
           is different, constants are kept, so repeated solves in place
           neither grow nor vanish
  random   the diagonally dominant tridiagonal recipe with a weak margin
"""
import ctypes
import math

import numpy as np
import torch

from paper_1909_04539_amd import sbs, workloads as W

KINDS = {"tri": sbs.SBS_TRI, "penta": sbs.SBS_PENTA, "periodic": sbs.SBS_TRI_PERIODIC}
DTYPES = {"f64": torch.float64, "f32": torch.float32}


def listed():
    return [
        # one small batch: a single latency-bound solve of 1024 short systems
        dict(name="tri 256x1024", op="solve", kind="tri", bands="var", n=256, m=1024, dtype="f64", s=0.8),
        # the benchmark's batch of hyperdiffusion steps
        dict(name="hyper 1024x65536", op="solve", kind="penta", bands="hyper", n=1024, m=65536, dtype="f64", s=0.5),
        # a matrix without constant bands, sizes that divide nothing
        dict(name="penta var 2001x20001", op="solve", kind="penta", bands="var", n=2001, m=20001, dtype="f64", s=0.5),
        # the longest systems the serving set draws, a few thousand of them
        dict(name="tri var 8192x4096", op="solve", kind="tri", bands="var", n=8192, m=4096, dtype="f64", s=0.5),
        # long systems, few right-hand sides
        dict(name="hyper 5000x500", op="solve", kind="penta", bands="hyper", n=5000, m=500, dtype="f64", s=0.3),
        # single precision throughout
        dict(name="tri f32 700x100000", op="solve", kind="tri", bands="var", n=700, m=100000, dtype="f32", s=0.5),
        # a periodic axis whose length is no multiple of anything
        dict(name="periodic 1000x10000", op="solve", kind="periodic", bands="var", n=1000, m=10000, dtype="f64", s=0.5),
        # time stepping, both of the paper's schemes
        dict(name="cn hyper 1024x65536", op="cn", kind="penta", bands="hyper", n=1024, m=65536, dtype="f64", s=0.5,
             steps=8),
        dict(name="cn periodic 512x6000", op="cn", kind="periodic", bands="diff", n=512, m=6000, dtype="f64", s=0.5,
             steps=20),
        # one alternating-direction step of a square grid
        dict(name="adi 2048x2048", op="adi", ny=2048, nx=2048, s=0.5),
        # mixed precision at the size where storage matters
        dict(name="refined 512x1048576", op="refined", kind="tri", bands="random", n=512, m=1 << 20, sweeps=2),
        # a burst of requests over many matrices, half FP32 and half FP64
        dict(name="serve 192", op="serve", matrices=16, requests=192, m_max=4096, trace=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choices(["solve", "cn", "adi", "refined", "serve"], [10, 4, 2, 3, 1])[0]
    if op == "adi":
        return dict(op="adi", ny=_log(rng, 64, 4096), nx=_log(rng, 64, 4096), s=round(rng.uniform(0.1, 1.0), 3))
    if op == "serve":
        return dict(op="serve", matrices=rng.randint(4, 16), requests=rng.randint(16, 192), m_max=_log(rng, 256, 4096),
                    trace=rng.randint(2, 1 << 20))
    n = _log(rng, 48, 8192)
    m = _log(rng, 64, min(1 << 20, max(128, (1 << 26) // n)))
    if op == "refined":
        return dict(op="refined", kind=rng.choice(["tri", "penta"]), bands=rng.choice(["var", "hyper"]), n=n, m=m,
                    sweeps=rng.randint(1, 3), s=round(rng.uniform(0.1, 1.0), 3))
    kind = rng.choice(["tri", "tri", "penta", "penta", "periodic"])
    constant = "hyper" if kind == "penta" else "diff"
    c = dict(op=op, kind=kind, bands=rng.choice([constant, "var"]), n=n, m=m,
             dtype=rng.choice(["f64", "f64", "f64", "f32"]), s=round(rng.uniform(0.1, 1.0), 3))
    if op == "cn":
        c["steps"] = rng.randint(1, 12)
    return c


# ---------------------------------------------------------------- matrices
def _bands(case, seed):
    kind, which, n = case["kind"], case["bands"], case["n"]
    rng = np.random.default_rng([seed, 1])
    if which == "random":
        return W.tri_dominant_bands(rng, n, (0.05, 0.5))
    s = case["s"]
    if which in ("hyper", "diff") and kind == "penta":
        return W.hyperdiffusion_bands(n, s)
    if which in ("hyper", "diff"):
        B = W.diffusion_bands(n, s)
        if kind == "periodic":
            B[0, 0] = B[2, n - 1] = -s
        return B
    if kind == "penta":
        # I + D2^T K D2, D2 the second difference on interior points
        k = np.zeros(n + 4)  # weight of the stencil centred at row i is k[i + 2]
        k[3:n + 1] = s * rng.uniform(0.5, 1.5, max(n - 2, 0))
        km, k0, kp = k[1:n + 1], k[2:n + 2], k[3:n + 3]
        B = np.stack([km, -2 * (km + k0), 1 + km + 4 * k0 + kp, -2 * (k0 + kp), kp])
        return W.zero_outside(B)
    k = s * rng.uniform(0.5, 1.5, n + 1)  # weight of the link between rows i - 1 and i is k[i]
    k[n] = k[0]
    if kind == "tri":
        k[0] = k[n] = 0.0
    return np.stack([-k[:n], 1 + k[:n] + k[1:], -k[1:]])


def _uniform(shape, dtype, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.empty(shape, dtype=dtype, device="cuda").uniform_(-1.0, 1.0, generator=g)


def _field(ny, nx, seed):
    """A smooth field of 8 Fourier modes plus a little noise, on the GPU."""
    rng = np.random.default_rng([seed, 3])
    ys = torch.arange(ny, dtype=torch.float64, device="cuda")[:, None] * (2 * math.pi / ny)
    xs = torch.arange(nx, dtype=torch.float64, device="cuda")[None, :] * (2 * math.pi / nx)
    F = 1e-3 * _uniform((ny, nx), torch.float64, seed + 1)
    for _ in range(8):
        k, l = int(rng.integers(1, 17)), int(rng.integers(1, 17))
        F += float(rng.uniform(0.5, 1.5)) * torch.sin(k * xs + l * ys + float(rng.uniform(0, 2 * math.pi)))
    return F


def _serving(case):
    """The matrices and request sizes of a served burst (fixed by the case)."""
    lhs = W.serving_lhs_set(seed=case["trace"], count=case["matrices"])
    trace = W.serving_trace(1e6, case["requests"], seed=case["trace"], n_lhs=case["matrices"], m_max=case["m_max"])
    return lhs, trace


class _Server:
    """A request loop with its registered matrices, released with the state."""

    def __init__(self, budget, handles):
        self.lib = sbs.lib()
        self.p = ctypes.c_void_p()
        _ok(self.lib.sbs_server_create(budget, 0, 0, ctypes.byref(self.p)))
        self.handles = handles  # alive until the server is gone
        self.ids = []
        for h in handles:
            i = ctypes.c_int32()
            _ok(self.lib.sbs_server_register(self.p, h.handle, ctypes.byref(i)))
            self.ids.append(i.value)

    def __del__(self):
        if self.p:
            self.lib.sbs_server_destroy(self.p)


def _ok(status):
    if status != 0:
        raise RuntimeError(sbs.sbs_status_str(status))


# ---------------------------------------------------------------- one pass
def prepare(case, seed):
    op = case["op"]
    if op == "adi":
        ny, nx, s = case["ny"], case["nx"], case["s"]
        grid = _field(ny, nx, seed)
        return dict(op=op, hy=sbs.SharedLhs(sbs.SBS_TRI, W.diffusion_bands(ny, s)),
                    hx=sbs.SharedLhs(sbs.SBS_TRI, W.diffusion_bands(nx, s)), grid=grid, work=torch.empty_like(grid))
    if op == "serve":
        lhs, trace = _serving(case)
        handles = [sbs.SharedLhs(l.kind, l.bands) for l in lhs]
        rhs = [_uniform((lhs[r.lhs].n, r.m), torch.float32 if r.fp32 else torch.float64, 1000 * seed + r.rid)
               for r in trace]
        out = torch.empty(sum(lhs[r.lhs].n * r.m for r in trace), dtype=torch.float64, device="cuda")
        views, at = [], 0
        for t in rhs:
            views.append(out[at:at + t.numel()])
            at += t.numel()
        torch.cuda.synchronize()  # the right-hand sides are there before the server reads them
        return dict(op=op, srv=_Server(8 << 30, handles), which=[r.lhs for r in trace], rhs=rhs, out=out, views=views)
    h = sbs.SharedLhs(KINDS[case["kind"]], _bands(case, seed))
    n, m = case["n"], case["m"]
    if op == "refined":
        return dict(op=op, h=h, b=_uniform((n, m), torch.float32, seed), sweeps=case["sweeps"],
                    x=torch.empty((n, m), dtype=torch.float64, device="cuda"),
                    work=torch.empty(sbs.sbs_refined_workspace_bytes(h.handle, m), dtype=torch.uint8, device="cuda"))
    x = _uniform((n, m), DTYPES[case["dtype"]], seed)
    return dict(op=op, h=h, x=x, steps=case.get("steps", 0))


def run(state):
    op = state["op"]
    if op == "solve":
        return state["h"].solve(state["x"])
    if op == "cn":
        return state["h"].cn_step(state["x"], state["steps"])
    if op == "adi":
        return sbs.sbs_adi_step(state["hy"].handle, state["hx"].handle, state["grid"], state["work"])
    if op == "refined":
        return state["h"].solve_refined(state["b"], state["sweeps"], x=state["x"], work=state["work"])
    # served: submit the burst, wait for each request, copy its result out, give its memory back
    srv, lib = state["srv"], sbs.lib()
    stream = torch.cuda.current_stream()
    tickets = []
    for k, t in zip(state["which"], state["rhs"]):
        tk = ctypes.c_uint64()
        code = sbs.SBS_F32 if t.dtype == torch.float32 else sbs.SBS_F64
        _ok(lib.sbs_server_submit(srv.p, srv.ids[k], t.data_ptr(), t.shape[1], code, ctypes.byref(tk)))
        tickets.append(tk)
    x, lat = ctypes.c_void_p(), ctypes.c_double()
    for tk, v in zip(tickets, state["views"]):
        _ok(lib.sbs_server_wait(srv.p, tk, -1, ctypes.byref(x), ctypes.byref(lat)))
        _ok(lib.sbs_server_fetch(srv.p, tk, v.data_ptr(), stream.cuda_stream))
    stream.synchronize()  # a request is released once its copy is done
    for tk in tickets:
        _ok(lib.sbs_server_release(srv.p, tk))
    return state["out"]


# ---------------------------------------------------------------- its work
def work(case):
    op = case["op"]
    if op == "adi":
        u = case["ny"] * case["nx"]
        return dict(bytes=16 * u, flops=10 * u)
    if op == "serve":
        lhs, trace = _serving(case)
        b = f = 0
        for r in trace:
            u = lhs[r.lhs].n * r.m
            per = 5 if lhs[r.lhs].kind == W.TRI else 9
            b += u * (12 if r.fp32 else 16)
            f += u * per
        return dict(bytes=b + 8 * sum(l.kind * l.n for l in lhs), flops=f)
    u = case["n"] * case["m"]
    per = {"tri": 5, "periodic": 7, "penta": 9}[case["kind"]]
    fac = 8 * case["n"] * (5 if case["kind"] == "penta" else 3)
    if op == "refined":
        return dict(bytes=12 * u + fac, flops=u * (per + case["sweeps"] * (2 * per + 2)))
    elem = 8 if case["dtype"] == "f64" else 4
    if op == "cn":
        return dict(bytes=2 * elem * u + fac, flops=case["steps"] * 2 * u * per)
    return dict(bytes=2 * elem * u + fac, flops=u * per)


# ---------------------------------------------------------------- in 64 bits
def _solve64(kind, B, X):
    """X <- A^{-1} X by elimination without pivoting, row by row, in FP64."""
    n = B.shape[1]
    if kind == "periodic":
        # A = A' + u v^T, A' without corners
        Bp = np.array(B, dtype=np.float64)
        b0, a0, cl = B[1, 0], B[0, 0], B[2, n - 1]
        Bp[1, 0] = 2 * b0
        Bp[1, n - 1] = B[1, n - 1] + a0 * cl / b0
        u = torch.zeros((n, 1), dtype=torch.float64, device=X.device)
        u[0, 0], u[n - 1, 0] = -b0, cl
        X = _solve64("tri", Bp, X)
        z = _solve64("tri", Bp, u)
        vy = X[0] - (a0 / b0) * X[n - 1]
        vz = float(z[0, 0] - (a0 / b0) * z[n - 1, 0])
        return X.addcmul_(z, vy[None, :] / (1 + vz), value=-1.0)
    B = B.tolist()
    if kind == "tri":
        a, b, c = B
        den, up = [b[0]], []
        for i in range(1, n):
            up.append(c[i - 1] / den[i - 1])
            den.append(b[i] - a[i] * up[i - 1])
        X[0].div_(den[0])
        for i in range(1, n):
            X[i].sub_(X[i - 1], alpha=a[i]).div_(den[i])
        for i in range(n - 2, -1, -1):
            X[i].sub_(X[i + 1], alpha=up[i])
        return X
    a, b, c, d, e = B
    al, ga, de, be = [0.0] * n, [0.0] * n, [0.0] * n, [0.0] * n
    for i in range(n):
        g1, d1 = (ga[i - 1], de[i - 1]) if i >= 1 else (0.0, 0.0)
        g2, d2 = (ga[i - 2], de[i - 2]) if i >= 2 else (0.0, 0.0)
        eps = a[i] if i >= 2 else 0.0
        be[i] = (b[i] if i >= 1 else 0.0) - eps * g2
        al[i] = c[i] - eps * d2 - be[i] * g1
        ga[i] = ((d[i] if i < n - 1 else 0.0) - be[i] * d1) / al[i]
        de[i] = (e[i] if i < n - 2 else 0.0) / al[i]
        if i >= 2:
            X[i].sub_(X[i - 2], alpha=eps)
        if i >= 1:
            X[i].sub_(X[i - 1], alpha=be[i])
        X[i].div_(al[i])
    for i in range(n - 2, -1, -1):
        X[i].sub_(X[i + 1], alpha=ga[i])
        if i + 2 < n:
            X[i].sub_(X[i + 2], alpha=de[i])
    return X


def _matvec64(kind, B, X):
    """A X in FP64."""
    n, h = B.shape[1], B.shape[0] // 2
    Bt = torch.from_numpy(np.ascontiguousarray(B)).to(X.device)
    Y = Bt[h][:, None] * X
    for k in range(2 * h + 1):
        off = k - h
        if off == 0:
            continue
        lo, hi = max(0, -off), min(n, n - off)
        if hi > lo:
            Y[lo:hi].addcmul_(Bt[k, lo:hi, None], X[lo + off:hi + off])
    if kind == "periodic":
        Y[0].add_(X[n - 1], alpha=float(B[0, 0]))
        Y[n - 1].add_(X[0], alpha=float(B[2, n - 1]))
    return Y


def exact(case, seed):
    op = case["op"]
    if op == "adi":
        ny, nx, s = case["ny"], case["nx"], case["s"]
        G = _solve64("tri", W.diffusion_bands(ny, s), _field(ny, nx, seed))
        return _solve64("tri", W.diffusion_bands(nx, s), G.t().contiguous()).t().contiguous()
    if op == "serve":
        lhs, trace = _serving(case)
        got = [None] * len(trace)
        for q, l in enumerate(lhs):
            mine = [r for r in trace if r.lhs == q]
            if not mine:
                continue
            X = torch.cat([_uniform((l.n, r.m), torch.float32 if r.fp32 else torch.float64,
                                    1000 * seed + r.rid).double() for r in mine], dim=1)
            X = _solve64("tri" if l.kind == W.TRI else "penta", l.bands, X)
            for r, x in zip(mine, X.split([r.m for r in mine], dim=1)):
                got[r.rid] = x.reshape(-1)
        return torch.cat(got)
    n, m = case["n"], case["m"]
    if op == "refined":
        return _solve64(case["kind"], _bands(case, seed), _uniform((n, m), torch.float32, seed).double())
    B = _bands(case, seed)
    X = _uniform((n, m), DTYPES[case["dtype"]], seed).double()
    for _ in range(case.get("steps", 0)):
        X = _solve64(case["kind"], B, 2 * X - _matvec64(case["kind"], B, X))
    return X if op == "cn" else _solve64(case["kind"], B, X)
