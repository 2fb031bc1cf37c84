"""Completion of served tiles that a workgroup of several waves solves: a tile's
count may go down only when every wave's results are where the host and the
rest of the GPU read them.  A missing wait shows only now and then in results,
so it is looked for in the gfx950 listing of the kernel, built here from source:
each wave waits for its own stores before the workgroup's barrier, and the wave
that takes one from the count waits for the write-back of its L2 first."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1909_04539_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    if not os.path.exists(build.hipcc()) and not shutil.which(build.hipcc()):
        pytest.skip("needs hipcc")
    out = str(tmp_path_factory.mktemp("asm") / "refine.s")
    subprocess.run([build.hipcc(), *build.HIP_FLAGS, "-I", build.INCLUDE, "-I", build.CSRC, "--offload-device-only", "-S",
                    os.path.join(build.CSRC, "refine.hip"), "-o", out], check=True)
    with open(out) as f:
        return f.read()


@pytest.mark.parametrize("kind", [3, 5])
def test_results_are_written_back_before_the_count_goes_down(listing, kind):
    body = re.search(r"^_ZN\S*k_refine_tilesILi%dE[^\n]*:[^\n]*$(.*?)s_endpgm" % kind, listing, re.M | re.S).group(1)
    ops = [m.group(1) for m in re.finditer(r"^\s+((?:s_waitcnt|s_barrier|global_|buffer_)[^;\n]*)", body, re.M)]
    at = [i for i, op in enumerate(ops) if op.startswith("global_atomic_add") and "sc1" in op]
    assert len(at) == 1  # the request's count, at system scope (the tile counter is at device scope)
    i = at[0] - 1

    def waits(op):
        return op.startswith("s_waitcnt") and "vmcnt(0)" in op

    assert waits(ops[i]), ops[i]                                # the write-back has completed
    assert ops[i - 1].startswith("buffer_wbl2 sc0 sc1"), ops[i - 1]
    i -= 2
    while not ops[i].startswith("s_barrier"):
        assert not ops[i].startswith("global_store"), ops[i]
        i -= 1
    before = i - 1
    while not waits(ops[before]):                               # every wave's stores, before the barrier
        assert not ops[before].startswith(("global_store", "s_barrier")), ops[before]
        before -= 1
    assert any(op.startswith("global_store") for op in ops[:before])
