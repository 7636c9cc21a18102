"""Host arithmetic of the matrix-core passes (csrc/mfma_plan.h), compiled with g++
into a small shared library: how a launch splits its work, and that no int32 sum can wrap."""
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
int xtr(int64_t ntail, int64_t nstage, int64_t slots, int64_t ptail, int B, int64_t room)
{
    return xtr_split(ntail, nstage, slots, ptail, B, room);
}
int64_t max_sum() { return kMfmaMaxSum; }
int64_t shares(int64_t nstage, int64_t stage) { return min_shares(nstage, stage); }
int64_t xroom(int64_t n, int64_t p, int64_t ncu) { return xtr_room(n, p, ncu); }
int64_t droom(int64_t n, int64_t p) { return dense_room(n, p); }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SRC)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2010_16114_amd", "csrc"), "-o", str(d / "plan.so"), str(d / "plan.cpp")],
                   check=True)
    lib = ctypes.CDLL(str(d / "plan.so"))
    i64 = ctypes.c_int64
    lib.xtr.argtypes = [i64, i64, i64, i64, ctypes.c_int, i64]
    lib.shares.argtypes = [i64, i64]
    lib.xroom.argtypes = [i64, i64, i64]
    lib.droom.argtypes = [i64, i64]
    lib.max_sum.restype = lib.shares.restype = lib.xroom.restype = lib.droom.restype = i64
    return lib


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


def test_sums_stay_in_int32(plan):
    """The extreme limbs are -128 and 127, the largest count 2: a run of the longest
    length fits int32, and it is not far below what int32 holds."""
    m = plan.max_sum()
    assert m % 128 == 0 and -2**31 <= -128 * 2 * m and 127 * 2 * m < 2**31
    assert -128 * 2 * (m + 256) < -2**31


@pytest.mark.parametrize("terms", [1, 128, 2**23 - 128, 2**23 - 127, 2**23, 2**23 + 512, 2**24 + 64, 2**27 + 1, 2**30,
                                   2**31 - 1])
def test_long_sums_are_split(plan, terms):
    """Whatever the split, no share of a sum is longer than int32 holds.  Shares take
    floor or ceil(stages / shares) stages.  A problem of so many columns (subjects) has
    at most 288e9 / terms subjects (columns): their sums fit the room that set-up gives
    them, and without that room the plan says so."""
    m, other = plan.max_sum(), max(1, min(200_000, 288 * 10**9 // terms))
    for stage in (64, 128):
        nstage = -(-terms // stage)
        k = plan.shares(nstage, stage)
        assert -(-nstage // k) * stage <= m and (k == 1 or -(-nstage // (k - 1)) * stage > m)
    nstage, k = -(-terms // 64), plan.shares(-(-terms // 64), 64)
    for sub, words in ((256, 256 * 96), (512, 512 * 48)):
        rows = -(-other // 512) * 512
        nblk, room = -(-other // sub), max(min(12 << 20, 16 * rows * 96), k * rows * 96 if k > 1 else 0)
        nfull, ks = _dense(plan, nblk, nstage, 256, words, room)
        assert ks >= 1 and -(-nstage // ks) * 64 <= m and (k == 1 or nfull == 0)
        if k > 1:
            assert _dense(plan, nblk, nstage, 256, words, 0)[1] == 0
    nstage, k = -(-terms // 128), plan.shares(-(-terms // 128), 128)
    nblk = -(-other // 256)
    ntail, room = (nblk, max(min(6 * 256 * 256, 16 * other), k * other)) if k > 1 else (nblk % 256, 6 * 256 * 256)
    ks = plan.xtr(ntail, nstage, 256, min(other, ntail * 256), 64, room)
    assert ks >= 1 and -(-nstage // ks) * 128 <= m
    if k > 1:
        assert plan.xtr(ntail, nstage, 256, other, 64, 0) == 0


@pytest.mark.parametrize("n,p,shares", [(400_000, 500_000, 3), (400_000, 62_500, 1), (200_000, 50_000, 5),
                                        (3001, 701, 12)])
def test_room_of_the_plans(plan, n, p, shares):
    """Within the room that a handle gives it X~' R splits its last round as it was
    measured best; the dense product always finds room to run."""
    nblk, nstage = -(-p // 256), -(-n // 128)
    ntail = nblk % 256
    assert plan.xtr(ntail, nstage, 256, p - (nblk - ntail) * 256, 64, plan.xroom(n, p, 256)) == shares
    for sub, words in ((256, 256 * 96), (512, 512 * 48)):
        assert _dense(plan, -(-n // sub), -(-p // 64), 256, words, plan.droom(n, p))[1] >= 1
