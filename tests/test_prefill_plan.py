"""The prefill launch's host-checkable parts (csrc/prefill_plan.h), built with
the host compiler: every grid is covered exactly once, also one whose
workgroups have no 31-bit id; and the choice of the kernel at its lines."""

import ctypes
import itertools
import os
import shutil
import subprocess

import pytest

from paper_2609_33536_amd import build

SOURCE = """
#include "prefill_plan.h"
extern "C" void place(uint32_t bx, uint32_t by, uint32_t gx, uint32_t gy, int tiles, int hkv, int batch, int spread,
                      int* out) {
  const ekv::PrefillPlace p = ekv::place_workgroup(bx, by, gx, gy, tiles, hkv, batch, spread != 0);
  out[0] = p.seq, out[1] = p.kv_head, out[2] = p.tile;
}
extern "C" int spreads(int64_t groups, int64_t rows, int64_t most_rows) {
  return ekv::spread_tiles(groups, rows, most_rows);
}
extern "C" int divides(int64_t workgroups, int64_t columns, int max_len, int stated) {
  return ekv::divide_units(workgroups, columns, max_len, stated != 0);
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("g++ or the HIP headers missing")
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SOURCE)
    p = subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", "-ftrapv", "-D__HIP_PLATFORM_AMD__",
                        "-I/opt/rocm/include", f"-I{build.CSRC}", "plan.cpp", "-o", "plan.so"], cwd=d,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout[-3000:]
    return ctypes.CDLL(str(d / "plan.so"))


def _place(plan, bx, by, gx, gy, tiles, hkv, batch, spread=False):
    out = (ctypes.c_int * 3)()
    plan.place(bx, by, gx, gy, tiles, hkv, batch, int(spread), out)
    return tuple(out)


@pytest.mark.parametrize("tiles,hkv,batch", itertools.product([1, 2, 7], [1, 2, 3, 8, 16], [1, 3, 16]))
def test_every_tile_once(plan, tiles, hkv, batch):
    gx, gy = tiles * hkv, batch
    for spread in (False, True):
        got = {_place(plan, bx, by, gx, gy, tiles, hkv, batch, spread) for by in range(gy) for bx in range(gx)}
        assert got == set(itertools.product(range(batch), range(hkv), range(tiles)))


@pytest.mark.parametrize("hkv,batch", [(1, 16), (1, 64), (2, 8), (4, 16), (3, 16), (1, 18), (2, 3), (6, 2)])
def test_spread_tiles_lie_on_all_xcds(plan, hkv, batch):
    """16 tiles of every (sequence, KV head) on the 8 XCDs (workgroup ids go round robin): two on each where the
    number of groups is a multiple of 8 (unspread: all 16 on one), else at most twice that on any."""
    tiles, groups = 16, hkv * batch
    assert plan.spreads(ctypes.c_int64(groups), ctypes.c_int64(1), ctypes.c_int64(2))
    xcds = {}
    for i in range(tiles * groups):
        s, h, t = _place(plan, i % (tiles * hkv), i // (tiles * hkv), tiles * hkv, batch, tiles, hkv, batch, True)
        xcds.setdefault((s, h), []).append(i % 8)
    most = 2 if groups % 8 == 0 else 4
    assert all(max(x.count(i) for i in range(8)) <= most for x in xcds.values())


@pytest.mark.parametrize("groups,rows,most,spread", [(64, 7, 8, False), (64, 6999, 8000, True), (32, 7, 8, False),
                                                     (30, 8, 8, True), (31, 1, 8, False), (65, 1, 8, False)])
def test_choice_of_the_order(plan, groups, rows, most, spread):
    assert bool(plan.spreads(ctypes.c_int64(groups), ctypes.c_int64(rows), ctypes.c_int64(most))) == spread


@pytest.mark.parametrize("tiles,hkv,batch", [(16384, 8, 16384), (1 << 18, 8, 65535), (1 << 21, 3, 65535)])
def test_grids_beyond_31_bits(plan, tiles, hkv, batch):
    gx, gy = tiles * hkv, batch
    assert gx * gy >= 1 << 31 and gx * 256 < 1 << 32
    seen = set()
    for by in (0, 1, batch // 2, batch - 1):
        for bx in (0, 1, hkv - 1, hkv, gx // 2, gx - hkv, gx - 1):
            s, h, t = _place(plan, bx, by, gx, gy, tiles, hkv, batch)
            assert s == by and (h, t) == (bx % hkv, tiles - 1 - bx // hkv) and 0 <= t < tiles
            seen.add((s, h, t))
    assert len(seen) == 4 * len({0, 1, hkv - 1, hkv, gx // 2, gx - hkv, gx - 1})


@pytest.mark.parametrize("workgroups,columns,max_len,stated,split", [
    (1, 64, 32, True, False), (1, 65, 32, True, True), (1, 64, 33, True, True), (1, 64, 32, False, True),   # one unit
    (1, 4096, 16, False, True), (256, 4096, 16, False, True),                       # they fit the chip at once
    (257, 64, 511, True, False), (257, 64, 512, False, True), (512, 64, 512, True, True), (513, 64, 8192, True, False),
    (513, 32, 1024, True, True), (2048, 32, 8192, True, True), (2049, 32, 8192, True, False),
    (513, 32, 1023, True, False), (513, 33, 8192, True, False),
    (513, 32, 8192, False, False), (4096, 32, 8192, False, False),                  # only the table's width: no claim
    (1 << 40, 1 << 30, 1 << 30, True, False)])
def test_choice_of_the_kernel(plan, workgroups, columns, max_len, stated, split):
    plan.divides.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int]
    assert bool(plan.divides(workgroups, columns, max_len, stated)) == split
