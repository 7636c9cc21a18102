"""Host arithmetic of the matrix-core passes (csrc/mfma_plan.h), compiled with g++
into a small shared library: how a launch splits its work."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = """
#include "mfma_plan.h"
using namespace cox;
extern "C" {
void dense(int64_t nblk, int64_t nstage, int64_t ncu, int64_t words, int64_t room, int64_t* out)
{
    const DensePlan d = dense_plan(nblk, nstage, ncu, words, room);
    out[0] = d.nfull;
    out[1] = d.ksplit;
}
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SRC)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2010_16114_amd", "csrc"), "-o", str(d / "plan.so"), str(d / "plan.cpp")],
                   check=True)
    return ctypes.CDLL(str(d / "plan.so"))


def _dense(plan, *args):
    out = (ctypes.c_int64 * 2)()
    plan.dense(*[ctypes.c_int64(a) for a in args], out)
    return out[0], out[1]


@pytest.mark.parametrize("nblk", [1, 7, 255, 256, 257, 391, 1563])
@pytest.mark.parametrize("nstage", [1, 2, 15, 16, 782, 7813])
@pytest.mark.parametrize("words", [256 * 96, 512 * 48])
def test_dense_product_split(plan, nblk, nstage, words):
    """Every split stays within the room for its sums and gives each share a stage; with
    no compute-unit count, or no room, every block runs whole."""
    for ncu in (0, 64, 256):
        for room in (0, words, 12 << 20):
            nfull, k = _dense(plan, nblk, nstage, ncu, words, room)
            assert 0 <= nfull <= nblk and 1 <= k <= min(16, nstage)
            assert nblk - nfull == (nblk % ncu if ncu else 0)
            assert k == 1 or (nblk > nfull and k * (nblk - nfull) * words <= room)
            if ncu == 0 or room == 0:
                assert k == 1
    # 391 blocks on 256 compute units: 135 left over, in shares that shorten the second round
    if nblk == 391 and nstage == 782:
        assert _dense(plan, nblk, nstage, 256, words, 12 << 20)[1] > 1
