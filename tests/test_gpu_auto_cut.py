"""Which solves and Crank-Nicolson calls AUTO cuts into segments (sbs_auto_cut),
and single steps that run that way against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1909_04539_amd import sbs
from test_cut_host import colrel, constant, dominant

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def matrix(kind, n, which):
    return dominant(kind, n, n) if which == "random" else constant(kind, n, 2000.0 if which == "slow" else 0.5)


# past 2048 rows always, unless the inverse decays too slowly for the windows;
# one system has no pair; a periodic matrix without whole blocks has no other
# partitioned form; short matrices are one segment
@pytest.mark.parametrize("kind,n,which,m,cut", [
    (3, 2049, "constant", 64, True), (3, 3001, "random", 2, True), (3, 3001, "random", 1, False),
    (5, 2500, "constant", 513, True), (5, 5143, "random", 64, True), (13, 2600, "random", 33, True),
    (13, 1027, "constant", 64, True), (3, 5000, "slow", 64, False), (5, 5000, "slow", 64, False),
    (13, 3001, "slow", 64, False), (3, 256, "random", 4096, False), (5, 600, "constant", 64, False)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_solves(kind, n, which, m, cut, dtype):
    x = torch.zeros((n, m), dtype=dtype, device=DEV)
    with sbs.SharedLhs(kind, matrix(kind, n, which)) as h:
        got = sbs.sbs_auto_cut(h.handle, x)
    assert (got is not None) == cut, got
    if cut:
        segments, S = got
        assert 1 < segments <= n // 128 + 1 and S in (8, 16, 32, 64, 128)


# 1025 to 2048 rows by where the rows start: at multiples of 128 bytes (whole
# lines), between them, or at multiples of 128 KiB; a last round of workgroups
# that the cut form makes one of, and one it does not; up to 1024 rows
@pytest.mark.parametrize("kind,n,which,m,cut", [
    (3, 1500, "constant", 20000, False), (3, 2048, "random", 10000, False), (3, 1500, "constant", 25000, True),
    (3, 1500, "constant", 16384, True), (3, 1100, "constant", 20000, True), (5, 1300, "constant", 20000, False),
    (5, 1300, "constant", 25000, True), (5, 1500, "random", 10000, True), (3, 1800, "constant", 4400, False),
    (5, 1800, "constant", 4400, True), (5, 1024, "constant", 65536, True), (5, 1024, "constant", 60000, False),
    (5, 1000, "constant", 65536, False), (3, 1000, "constant", 65536, True), (5, 961, "constant", 49152, False)])
def test_large_batches(kind, n, which, m, cut):
    x = torch.empty((n, m), dtype=torch.float64, device=DEV)
    with sbs.SharedLhs(kind, matrix(kind, n, which)) as h:
        assert (sbs.sbs_auto_cut(h.handle, x) is not None) == cut


@pytest.mark.parametrize("kind,n,m", [(3, 2057, 1501), (3, 2500, 1100), (3, 5001, 333), (5, 2100, 5000), (5, 2500, 130),
                                      (5, 4099, 77), (13, 600, 50), (13, 1001, 129), (13, 2500, 2)])
@pytest.mark.parametrize("which", ["constant", "random"])
@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-12), (torch.float32, 1e-5)])
def test_one_step(kind, n, m, which, dtype, tol):
    print(f"case kind={kind} n={n} m={m} {which} {dtype}", flush=True)
    B = matrix(kind, n, which)
    c = torch.from_numpy(np.random.default_rng(n * m).uniform(-1, 1, (n, m))).to(dtype)
    with sbs.SharedLhs(kind, B) as h:
        x = c.to(DEV)
        assert sbs.sbs_auto_cut(h.handle, x, cn_steps=1) is not None
        h.cn_step(x, 1)
        torch.cuda.synchronize()
    cols = np.unique(np.r_[0, m // 2, m - 1, np.random.default_rng(m).integers(0, m, 20)])
    ref = oracle.cn_steps(kind, B, np.ascontiguousarray(c.double().numpy()[:, cols]), 1)
    assert colrel(x.double().cpu().numpy()[:, cols], ref) <= tol


# one launch of the pair form where the cut form's two cost more; the large
# batches beside those it keeps are cut
@pytest.mark.parametrize("kind,n,which,m,cut", [
    (3, 2500, "constant", 64, False), (3, 2500, "constant", 512, False), (3, 2500, "constant", 1024, True),
    (13, 2112, "constant", 4000, False), (13, 4096, "constant", 512, True), (3, 1030, "random", 500, False),
    (3, 1030, "random", 4096, False), (3, 1030, "random", 16000, True), (3, 1300, "random", 64, False),
    (3, 1300, "random", 1000, True), (13, 1728, "random", 8000, False), (3, 300, "random", 70000, False),
    (3, 800, "random", 32768, False), (3, 1000, "random", 20000, True), (5, 1030, "random", 64, True)])
def test_one_step_keeps_the_pair_form(kind, n, which, m, cut):
    x = torch.zeros((n, m), dtype=torch.float64, device=DEV)
    with sbs.SharedLhs(kind, matrix(kind, n, which)) as h:
        assert (sbs.sbs_auto_cut(h.handle, x, cn_steps=1) is not None) == cut


# rounds of workgroups of the two forms: as many (whole blocks keep the pair form,
# a ragged last one does not), fewer of the cut form's; FP32 while the pair form's are one round
@pytest.mark.parametrize("n,m,dtype,cut", [
    (1472, 6000, torch.float64, False), (1472, 5000, torch.float64, True), (1472, 12000, torch.float64, False),
    (1472, 10000, torch.float64, True), (1472, 20000, torch.float64, True), (1216, 6000, torch.float64, True),
    (1471, 6000, torch.float64, True), (1599, 8000, torch.float64, False), (1406, 4096, torch.float32, True),
    (1207, 1100, torch.float32, False), (1553, 1100, torch.float32, True),
    (1408, 3000, torch.float32, False), (1408, 4096, torch.float32, False), (1408, 4400, torch.float32, True),
    (1100, 2000, torch.float32, True), (1600, 1100, torch.float32, False), (1600, 3000, torch.float32, True)])
def test_one_step_by_rounds(n, m, dtype, cut):
    x = torch.zeros((n, m), dtype=dtype, device=DEV)
    with sbs.SharedLhs(3, matrix(3, n, "random")) as h:
        assert (sbs.sbs_auto_cut(h.handle, x, cn_steps=1) is not None) == cut


# pentadiagonal constant bands where no pair form fits
@pytest.mark.parametrize("n,m,cut", [(1750, 4096, False), (1792, 4096, False), (1800, 4096, True), (2048, 20000, True)])
def test_one_step_of_constant_pentadiagonal_bands(n, m, cut):
    x = torch.zeros((n, m), dtype=torch.float64, device=DEV)
    with sbs.SharedLhs(5, constant(5, n)) as h:
        assert (sbs.sbs_auto_cut(h.handle, x, cn_steps=1) is not None) == cut


# FP32 solves: a whole round of the pair form's workgroups, and seven segments
@pytest.mark.parametrize("kind,n,m,cut", [(3, 1950, 777, True), (3, 1950, 6000, True), (3, 1950, 8192, False),
                                          (13, 1920, 4096, False), (3, 1920, 5000, True),
                                          (3, 1950, 8300, True), (13, 1792, 1000, False), (3, 1800, 1000, True), (5, 1536, 500, True)])
def test_fp32_beside_the_pair_form(kind, n, m, cut):
    x = torch.zeros((n, m), dtype=torch.float32, device=DEV)
    with sbs.SharedLhs(kind, matrix(kind, n, "random")) as h:
        assert (sbs.sbs_auto_cut(h.handle, x) is not None) == cut


def test_several_steps_keep_the_systems_whole_where_they_can():
    # steps of a call are the same arithmetic however a caller groups them
    x = torch.zeros((4000, 64), dtype=torch.float64, device=DEV)
    with sbs.SharedLhs(3, constant(3, 4000)) as h:
        assert sbs.sbs_auto_cut(h.handle, x, cn_steps=1) is not None
        assert sbs.sbs_auto_cut(h.handle, x, cn_steps=2) is None
    with sbs.SharedLhs(3, constant(3, 6000)) as h:  # no whole form fits
        y = torch.zeros((6000, 64), dtype=torch.float64, device=DEV)
        assert sbs.sbs_auto_cut(h.handle, y, cn_steps=2) is not None


def test_bad_arguments():
    L = sbs.lib()
    x = torch.zeros((300, 8), dtype=torch.float64, device=DEV)
    import ctypes
    a, b = ctypes.c_int32(), ctypes.c_int32()
    with sbs.SharedLhs(3, constant(3, 300)) as h:
        ok = (h.handle, 8, sbs.SBS_F64, x.data_ptr(), 0, ctypes.byref(a), ctypes.byref(b))
        assert L.sbs_auto_cut(*ok) == 0
        for k, bad in ((0, None), (1, 0), (2, 7), (4, -1), (5, None), (6, None)):
            assert L.sbs_auto_cut(*[bad if i == k else v for i, v in enumerate(ok)]) == 1


@pytest.mark.parametrize("kind,n,m", [(5, 3124, 3736), (3, 2336, 6001), (13, 2600, 2000)])
def test_short_last_segment(kind, n, m):
    # the last segment (28, 23 and 29 rows) takes more workgroups than its rows alone give it
    B = constant(kind, n)
    x = np.random.default_rng(n).uniform(-1, 1, (n, m))
    t = torch.from_numpy(x).to(DEV)
    with sbs.SharedLhs(kind, B) as h:
        assert sbs.sbs_auto_cut(h.handle, t) is not None
        h.solve(t)
        torch.cuda.synchronize()
    cols = np.unique(np.r_[0, 1, 127, 128, m // 2, m - 2, m - 1, np.random.default_rng(m).integers(0, m, 40)])
    ref = oracle.solve(kind, B, np.ascontiguousarray(x[:, cols]))
    assert colrel(t.cpu().numpy()[:, cols], ref) <= 1e-13
