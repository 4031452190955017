"""Which workgroup takes which tile (scc_deal.h): the header itself, built for the host, gives every pair of column tile and row
group to one workgroup, and every column tile to one of a persistent grid's; and the reciprocal's quotient with its one correction,
recomputed here, is exact over the whole range of indexes."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2101_00745_amd import build

SOURCE = """
#include "scc_deal.h"
using namespace scc;
static Deal make(int form, long long outer, int inner)
{
    return form == 0 ? make_deal(outer, inner) : form == 1 ? make_runs(outer, inner) : in_eighths(make_runs(outer, inner));
}
// pairs of the workgroups 8*from ... 8*to - 1 as outer * inner_count + inner, -1 without work; returns slots of an XCD.  runs: 0 or 1
extern "C" int deal(int form, int runs, long long outer, int inner, int from, int to, long long* pairs)
{
    const Deal d = make(form, outer, inner);
    for (int bid = 8 * from; bid < 8 * to && bid < 8 * d.chunk; ++bid) {
        int o, i;
        const bool work = runs ? dealt<true>(d, bid, o, i) : dealt<false>(d, bid, o, i);
        pairs[bid - 8 * from] = !work ? -1 : (o < 0 || i < 0 || i >= inner) ? -2 : (long long)o * inner + i;
    }
    return d.chunk;
}
// tiles that `lanes` workgroups of each XCD take, in turn; returns their number
extern "C" int persistent(long long outer, int lanes, int* tiles)
{
    const Deal d = make_runs(outer, 1);
    int n = 0;
    for (int xcd = 0; xcd < 8; ++xcd)
        for (int lane = 0; lane < lanes; ++lane)
            for (int i = lane; i < tiles_of(d, xcd); i += lanes) tiles[n++] = nth_tile(d, xcd, i);
    return n;
}
"""
OUTERS = [1, 2, 7, 8, 9, 127, 128, 129, 143, 144, 255, 256, 257, 383, 384, 391, 512, 518, 1000, 1024, 1151, 1152, 2047, 5000]


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    folder = tmp_path_factory.mktemp("deal")
    source, lib = str(folder / "deal.cpp"), str(folder / "deal.so")
    with open(source, "w") as f:
        f.write(SOURCE)
    subprocess.run([os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__=1", "-I", build.CSRC,
                    "-I", os.path.join(build.rocm_root(), "include"), source, "-o", lib], check=True)
    h = ctypes.CDLL(lib)
    h.deal.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_longlong, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    h.persistent.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_void_p]
    return h


# a body without runs reads any deal as one in eighths (form 1 with runs 0)
@pytest.mark.parametrize("form,runs", [(0, 1), (1, 1), (2, 1), (2, 0), (1, 0)])
def test_every_pair_once(host, form, runs):
    for inner in (1, 2, 3, 5, 8, 12, 17):
        for outer in OUTERS:
            chunk = (outer * inner + 7) // 8
            pairs = np.full(8 * chunk, -3, dtype=np.int64)
            assert host.deal(form, runs, outer, inner, 0, chunk, pairs.ctypes.data) == chunk
            assert pairs.min() >= -1
            assert np.array_equal(np.sort(pairs[pairs >= 0]), np.arange(outer * inner)), (outer, inner)


@pytest.mark.parametrize("inner", [1, 3, 40, 1023])
def test_large_grids(host, inner):
    """2**28 - 1 workgroups at most, some of them: in range, no pair twice, and those of an XCD's run on neighbouring tiles."""
    outer = (2**28 - 1) // inner
    chunk = (outer * inner + 7) // 8
    seen = []
    for at in (0, chunk // 3, min(chunk - 6000, outer // 128 * 16 * inner - 1500), chunk - 3000):      # the last two: where the runs end, and the end
        pairs = np.full(8 * 3000, -3, dtype=np.int64)
        assert host.deal(0, 1, outer, inner, at, at + 3000, pairs.ctypes.data) == chunk
        assert pairs.min() >= -1 and pairs.max() < outer * inner
        seen.append(pairs[pairs >= 0])
        assert len(seen[-1]) >= 8 * 3000 - 8
        ahead = pairs.reshape(-1, 8)[1:] - pairs.reshape(-1, 8)[:-1]
        assert np.mean(ahead == 1) > 0.93                    # 15 of 16 tiles of a run
    seen = np.concatenate(seen)
    assert len(np.unique(seen)) == len(seen)


@pytest.mark.parametrize("lanes", [1, 2, 3, 8, 32])
def test_persistent_workgroups_take_every_tile_once(host, lanes):
    for outer in OUTERS + [128 * 17 + 1, 128 * 40 - 1]:
        tiles = np.full(outer + 64, -1, dtype=np.int32)
        assert host.persistent(outer, lanes, tiles.ctypes.data) == outer
        assert np.array_equal(np.sort(tiles[:outer]), np.arange(outer)), outer


@pytest.mark.parametrize("inner", [1, 2, 3, 7, 12, 255, 256, 257, 1000, 65535, 65536, 65537, 2**30, 2**31 - 1])
def test_quotient_is_exact(inner):
    recip = 2**32 - 1 if inner == 1 else 2**32 // inner          # make_runs
    some = np.random.default_rng(0).integers(0, 2**31, 20000)
    ends = np.arange(1, 2000, dtype=np.int64) * inner
    at = np.concatenate([np.arange(2000), some, ends, ends - 1, [2**31 - 1]])
    at = at[at < 2**31]
    tile = (at.astype(np.uint64) * np.uint64(recip) >> np.uint64(32)).astype(np.int64)
    rest = at - tile * inner
    more = rest >= inner
    assert np.array_equal(tile + more, at // inner) and np.array_equal(rest - more * inner, at % inner)
