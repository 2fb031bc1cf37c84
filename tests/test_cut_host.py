"""The cut form of plain solves and the segments of mixed-precision solves, on
the CPU: the tables that build_partitions uploads are run step for step by
tests/host/cut_emulate.cpp, built with g++ and the address and undefined
behaviour sanitizers, and compared with the oracle: ragged lengths, wrapped
windows, segments that share a plan, and matrices whose rows are scaled
unevenly (the solution of a system does not change when a row and its
right-hand sides are multiplied by the same factor)."""
import os
import shutil
import struct
import subprocess

import numpy as np
import pytest

import oracle
import test_partition_host as P
from paper_1909_04539_amd import workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1909_04539_amd", "csrc")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if not shutil.which("g++") or not os.path.isdir("/opt/rocm/include/hip"):
        pytest.skip("needs g++ and the HIP headers")
    out = str(tmp_path_factory.mktemp("cut") / "cut_emulate")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-omit-frame-pointer", "-pthread",
           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           os.path.join(CSRC, "partition.cpp"), os.path.join(HERE, "host", "mock_device.cpp"),
           os.path.join(HERE, "host", "cut_emulate.cpp"), "-o", out]
    subprocess.run(cmd, check=True)
    return out


def run(exe, tmp_path, kind, B, rhs):
    """(segments, cuts, x) of the cut form, (segments, x) of the refined one; x None where there is none."""
    n, m = rhs.shape
    src, dst = str(tmp_path / "in.bin"), str(tmp_path / "out.bin")
    with open(src, "wb") as f:
        f.write(struct.pack("<iqq", kind, n, m))
        f.write(np.ascontiguousarray(B, dtype=np.float64).tobytes())
        f.write(np.ascontiguousarray(rhs, dtype=np.float64).tobytes())
    r = subprocess.run([exe, src, dst], capture_output=True, text=True, timeout=120,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=1", UBSAN_OPTIONS="halt_on_error=1"))
    assert r.returncode == 0, r.stderr
    with open(dst, "rb") as f:
        def column():
            return np.frombuffer(f.read(8 * n * m), dtype=np.float64).reshape(n, m)
        Q, cuts = struct.unpack("<2i", f.read(8))
        x = column() if Q else None
        (nseg,) = struct.unpack("<i", f.read(4))
        y = column() if nseg else None
    return (Q, cuts, x), (nseg, y)


def colrel(x, ref):
    return float(np.max(np.max(np.abs(x - ref), axis=0) / np.max(np.abs(ref), axis=0)))


def dominant(kind, n, seed):
    rng = np.random.default_rng(seed)
    nb = 5 if kind == 5 else 3
    B = rng.uniform(-1, 1, (nb, n))
    B[nb // 2] = np.sum(np.abs(np.delete(B, nb // 2, axis=0)), axis=0) + rng.uniform(1, 2, n)
    return B if kind == 13 else W.zero_outside(B)


def constant(kind, n, s=0.5):
    if kind == 5:
        return W.hyperdiffusion_bands(n, s)
    B = W.diffusion_bands(n, s)
    if kind == 13:
        B[0, 0] = B[2, n - 1] = -s
    return B


def matvec(kind, B, X):
    """A X; the rows' sums in long double, rounded once."""
    n, h = B.shape[1], B.shape[0] // 2
    Y = np.zeros(X.shape, dtype=np.longdouble)
    for k in range(2 * h + 1):
        off = k - h
        if kind == 13:
            Y += B[k][:, None].astype(np.longdouble) * np.roll(X, -off, axis=0)
        else:
            lo, hi = max(0, -off), min(n, n - off)
            Y[lo:hi] += B[k, lo:hi, None].astype(np.longdouble) * X[lo + off:hi + off]
    return Y.astype(np.float64)


@pytest.mark.parametrize("kind,n", [(3, 257), (3, 258), (3, 300), (3, 513), (3, 1029), (3, 2500), (3, 8192), (5, 257),
                                    (5, 258), (5, 259), (5, 520), (5, 1027), (5, 2001), (5, 5000), (13, 513), (13, 514),
                                    (13, 515), (13, 1000), (13, 1027), (13, 2600), (13, 4999)])
@pytest.mark.parametrize("which", ["random", "constant"])
def test_tables_solve_like_the_oracle(exe, tmp_path, kind, n, which):
    B = dominant(kind, n, n) if which == "random" else constant(kind, n)
    rhs = np.random.default_rng(n).uniform(-1, 1, (n, 2)).astype(np.float32).astype(np.float64)
    (Q, cuts, x), (nseg, y) = run(exe, tmp_path, kind, B, rhs)
    if kind == 13 and n < 514:
        assert Q == 0  # shorter than the windows of a periodic matrix
    else:
        assert Q >= 2 and cuts == (Q if kind == 13 else Q - 1)
        assert colrel(x, oracle.solve(kind, B, rhs)) <= 1e-13
    assert (nseg > 0) == (kind != 13)
    if nseg:
        assert colrel(y, oracle.refine_reference(kind, B, rhs.astype(np.float32))) <= 1e-12


@pytest.mark.parametrize("kind", [3, 5, 13])
def test_slowly_decaying_inverse_has_no_cut_form(exe, tmp_path, kind):
    B = constant(kind, 2600, 2000.0)
    (Q, _, _), _ = run(exe, tmp_path, kind, B, np.ones((2600, 1)))
    assert Q == 0


# The first cut of 2500 or 2600 tridiagonal rows is at 224 .. 256, of the
# pentadiagonal ones likewise: rows around there get one large coefficient (a
# value imposed through the diagonal), or the rows up to there are scaled.
def scales(n, which, K, r):
    d = np.ones(n)
    if which == "below":
        d[:r] = K
    elif which == "above":
        d[r:] = K
    else:
        d[r::7] = K
    return d


@pytest.mark.parametrize("kind", [3, 5, 13])
@pytest.mark.parametrize("which", ["below", "above", "scattered"])
@pytest.mark.parametrize("K", [1e4, 1e8, 1e15])
def test_scaled_rows(exe, tmp_path, kind, which, K):
    # x is uniform, the right-hand sides are A x: |A^-1| |A| is below 10, so the
    # rounding of the right-hand sides and of the solve move x by some 1e-15
    n = 2600
    x = np.random.default_rng(n).uniform(-1, 1, (n, 2))
    for r in (200, 222, 240, 250, 258):
        d = scales(n, which, K, r)
        for B in (constant(kind, n), dominant(kind, n, r)):
            (Q, _, got), _ = run(exe, tmp_path, kind, B * d, matvec(kind, B * d, x))
            assert Q >= 2
            assert colrel(got, x) <= 2e-14, (r, colrel(got, x))


@pytest.mark.parametrize("kind", [3, 5, 13])
@pytest.mark.parametrize("K", [1e6, 1e12, 1e16])
def test_imposed_values(exe, tmp_path, kind, K):
    # a value imposed through a large diagonal entry and right-hand side
    n = 2600
    x = np.random.default_rng(n).uniform(-1, 1, (n, 2))
    for r in (200, 215, 235, 245, 250):
        B = constant(kind, n)
        B[B.shape[0] // 2, r] = K
        (Q, _, got), _ = run(exe, tmp_path, kind, B, matvec(kind, B, x))
        assert Q >= 2
        assert colrel(got, x) <= 2e-14, (r, colrel(got, x))


# The separator plans of the whole matrix drop entries of S^-1 in the same way.
part_exe = P.exe


@pytest.mark.parametrize("kind,n", [(3, 1024), (5, 1024), (13, 1024), (3, 300), (5, 333)])
@pytest.mark.parametrize("which", ["below", "above", "scattered"])
@pytest.mark.parametrize("K", [1e8, 1e15])
def test_scaled_rows_in_separator_plans(part_exe, tmp_path, kind, n, which, K):
    x = np.random.default_rng(n).uniform(-1, 1, (n, 2))
    for r in (100, 128, 160):
        B = constant(kind, n) * scales(n, which, K, r)
        found = 0
        for lb, *_, got in P.run_sep(part_exe, tmp_path, kind, B, matvec(kind, B, x)):
            if lb:
                found += 1
                assert colrel(got, x) <= 2e-14, (lb, r, colrel(got, x))
        assert found >= 2


# Tiny pivots at the rows that start a 16-row block: the recurrences on the
# whole matrix never meet them, a plan cut there loses digits.  Where those rows
# are large, a right-hand side that is uniform in every row leaves their
# unknowns too small to tell; A x of a uniform x does not.
def tiny_pivots_in_large_rows(n, rows, K):
    B = P.tiny_block_pivot_bands(n)
    B[1, 16::16] = np.where(np.arange(16, n, 16) < rows, 1e-9, 3.0)
    B[:, :rows] *= K
    return B


@pytest.mark.parametrize("n", [256, 1000, 2600])
def test_plans_that_lose_the_unknowns_of_large_rows_are_dropped(exe, part_exe, tmp_path, n):
    B = tiny_pivots_in_large_rows(n, min(n // 2, 200), 1e14)
    x = np.random.default_rng(n).uniform(-1, 1, (n, 2))
    b = matvec(3, B, x)
    assert colrel(oracle.solve(3, B, b), x) <= 2e-13
    (Q, _, got), (nseg, y) = run(exe, tmp_path, 3, B, b)
    plans, seps = P.run_all(part_exe, tmp_path, 3, B, b)
    for lb, *_, z in [(Q, got)] + plans + seps:
        if lb:
            assert colrel(z, x) <= 2e-13, lb
