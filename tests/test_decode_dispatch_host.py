"""What fa_decode_blocks launches (CPU): a child process loads two recording
functions in the place of the library's decode launchers and calls the entry
point, so its choice of tile, split and workgroups shows without a GPU."""
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RECORD = r"""
#include "%(root)s/paper_2409_00184_amd/csrc/fa_internal.hpp"
extern "C" { long long rec[9]; }
namespace fa {
static hipError_t put(const DecodeLaunch &a, int kernel, int waves, int grid) {
    const long long r[9] = {kernel, a.rows, waves, grid, a.xsegs, a.nitems, a.xcost, a.nt_store, a.slab};
    for (int i = 0; i < 9; ++i) rec[i] = r[i];
    return hipSuccess;
}
hipError_t launch_decode_sep(const DecodeLaunch &a, int w, int g, hipStream_t) { return put(a, 0, w, g); }
hipError_t launch_decode_mfma(const DecodeLaunch &a, int w, int g, hipStream_t) { return put(a, 1, w, g); }
}
"""

CHILD = r"""
import ctypes, json, sys
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
vp, i32 = ctypes.c_void_p, ctypes.c_int32
lib.fa_decode_blocks.argtypes = [vp, i32, vp, vp, ctypes.c_int, vp, ctypes.c_uint32, vp, vp, vp, i32, vp, vp]
out = []
for c in json.load(sys.stdin):
    res, tune = (i32 * 3)(*c["res"]), (i32 * 6)(*c["tune"])
    groups = c.get("groups", 0)
    p = ctypes.c_void_p(4096)  # never read by the host
    st = lib.fa_decode_blocks(p, c["nblocks"], p, p, c.get("dtype", 0), res, c["mask"], tune,
                              p if groups else None, p if groups else None, groups, p, None)
    v = (ctypes.c_longlong * 9).in_dll(rec, "rec")
    out.append([st] + list(v))
json.dump(out, sys.stdout)
"""
KEYS = ("status", "kernel", "rows", "waves", "grid", "xsegs", "nitems", "xcost", "nt_store", "slab")


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    import paper_2409_00184_amd as fa
    d = tmp_path_factory.mktemp("record")
    src, so = d / "record.cpp", d / "record.so"
    src.write_text(RECORD % dict(root=ROOT))
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-w", "-fPIC",
                    "-shared", str(src), "-o", str(so)], check=True)

    def run(cases):
        r = subprocess.run([sys.executable, "-c", CHILD, str(so), fa.library_path()], check=True,
                           input=json.dumps(cases), capture_output=True, text=True)
        return [dict(zip(KEYS, x)) for x in json.loads(r.stdout)]
    return run


def _items(nblocks, res, rows):
    return nblocks * -(-res[1] // rows) * -(-res[2] // 64)


SHAPES = [(1, (64, 64, 64)), (64, (64, 64, 64)), (512, (64, 64, 64)), (5000, (64, 64, 64)),
          (300, (61, 47, 53)), (40, (96, 80, 48)), (9000, (17, 9, 5)), (200, (250, 7, 130)), (3, (2, 2, 2))]


@pytest.mark.parametrize("mask", [1, 14, 15, 15 | 0x100])
def test_given_grid_is_not_exceeded(launches, mask):
    """tune.grid is an upper bound of the workgroups, with and without a plan, and
    one below the item count runs whole items."""
    cases = []
    for nblocks, res in SHAPES:
        for kernel, dtype in ((0, 0), (1, 1)):
            for rows in ((0, 4, 8, 16) if kernel == 0 else (0, 16)):
                n = _items(nblocks, res, rows or 8)
                for grid in {1, 7, max(1, n // 2), max(1, n - 1), n, n + 1, 2 * n, 8 * n, 1 << 20, 1 << 21}:
                    tune = [rows, 0, grid, kernel, 0, 0]
                    cases.append(dict(nblocks=nblocks, res=res, mask=mask, tune=tune, dtype=dtype))
                    if rows:
                        cases.append(dict(cases[-1], groups=min(n, grid)))
    for c, r in zip(cases, launches(cases)):
        assert r["status"] == 0, c
        grid = c["tune"][2]
        assert 0 < r["grid"] <= min(grid, 1 << 20), (c, r)
        if "groups" in c:
            assert r["grid"] == c["groups"] * r["xsegs"], (c, r)
        else:
            assert r["nitems"] == _items(c["nblocks"], c["res"], r["rows"]) * r["xsegs"], (c, r)
        if grid < _items(c["nblocks"], c["res"], r["rows"]):
            assert r["xsegs"] == 1, (c, r)


def test_rows_without_a_plan(launches):
    """Rows left open: eight for one channel, for eight given waves, for a large
    batch split along x and for one of small grids, else four; never more waves
    than rows by default."""
    cases = [(dict(nblocks=500, res=(64, 64, 40), mask=3, tune=[0, 8, 0, 0, 0, 0]), 8, 8),
             (dict(nblocks=500, res=(64, 64, 40), mask=3, tune=[0, 4, 0, 0, 0, 0]), 4, 4),
             (dict(nblocks=500, res=(64, 64, 40), mask=3, tune=[0, 0, 0, 0, 0, 0]), 4, 4),
             (dict(nblocks=500, res=(64, 64, 40), mask=1, tune=[0, 0, 0, 0, 0, 0]), 8, 8),
             (dict(nblocks=512, res=(64, 64, 64), mask=15, tune=[0, 0, 0, 0, 0, 0]), 8, 8),
             (dict(nblocks=512, res=(64, 64, 64), mask=14, tune=[0, 0, 0, 0, 0, 0]), 4, 4),
             (dict(nblocks=8192, res=(32, 32, 32), mask=15, tune=[0, 0, 0, 0, 0, 0]), 8, 8),
             (dict(nblocks=8, res=(32, 32, 32), mask=15, tune=[0, 0, 0, 0, 0, 0]), 4, 4)]
    for (c, rows, waves), r in zip(cases, launches([c for c, _, _ in cases])):
        assert (r["status"], r["rows"], r["waves"]) == (0, rows, waves), (c, r)


def test_store_kind(launches):
    """store = 0: non-temporal by the bytes of a row of the layout that is
    written, a record's being four times a planar row's; store = 1: ordinary."""
    wanted = {15: {64, 96, 32, 16, 12, 4, 28}, 1: {64, 96, 32, 16, 12, 4, 28},
              15 | 0x100: {64, 96, 32, 16, 12, 4, 28, 36, 40, 48, 72, 62, 18}}
    cases = [dict(nblocks=100, res=(64, 64, rz), mask=mask, tune=[0, 0, 0, 0, 0, store])
             for mask in wanted for store in (0, 1)
             for rz in (4, 12, 13, 16, 18, 28, 32, 36, 40, 48, 53, 62, 64, 72, 96)]
    for c, r in zip(cases, launches(cases)):
        rz, store = c["res"][2], c["tune"][5]
        nt = store == 0 and rz in wanted[c["mask"]]
        assert r["nt_store"] == int(nt), (c, r)


def test_more_segments_than_a_launch_holds(launches):
    """Batches whose segments come to more than 2^20 workgroups run whole items,
    several to a workgroup above 2^20 items."""
    cases = [dict(nblocks=n, res=res, mask=15, tune=[0] * 6, groups=groups)
             for n, res, groups in ((40000, (64, 64, 64), 0), (40000, (64, 64, 64), 320000),
                                    (30000, (64, 64, 64), 0), (2 << 20, (8, 8, 8), 0))]
    r = launches(cases)
    assert [x["status"] for x in r] == [0] * 4
    assert [(x["xsegs"], x["grid"]) for x in r] == [(1, 320000), (1, 320000), (4, 960000), (1, 1 << 20)]
    assert r[3]["nitems"] == 2 << 20
