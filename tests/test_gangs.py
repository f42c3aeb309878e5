"""Tiles in gangs: which launches have them, and that their runs are every chunk once."""
import ctypes
import os
import subprocess

import pytest

from paper_2502_06728_amd import build

DRIVER = r"""
#include "tiled_launch.h"
extern "C" int run_log2(int s, int k, int val, int idx_bytes, int R, int adam) {
    return deto::run_log2(s, k, val, idx_bytes, R ? deto::decompress_run_bytes(s, k, R, adam != 0) : deto::kRunBytes);
}
extern "C" int gangs(int s, int k, int val, int lg, int adam, int amsgrad, int classes) {
    deto::KParams p = {};
    p.s = s; p.k = k; p.val_dtype = val; p.idx_u8 = val != 0; p.run_lg = lg; p.adam = adam; p.amsgrad = amsgrad;
    return deto::decompress_gangs(p, classes);
}
// how often a chunk is in a tile
extern "C" void cover(int64_t tiles, int lg, int* times) {
    for (int64_t t = 0; t < tiles; ++t) {
        const deto::TileRows rows = deto::tile_rows(t, tiles, lg);
        for (uint32_t r = 0; r < 64; ++r) ++times[rows.first + rows.chunk(r)];
    }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("gangs")
    (d / "gangs.hip").write_text(DRIVER)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950",
                    "--cuda-host-only", "-std=c++17", "-O1", "-fPIC", "-shared", "-I", build.CSRC,
                    "-o", str(d / "gangs.so"), str(d / "gangs.hip")], check=True, capture_output=True)
    return ctypes.CDLL(str(d / "gangs.so"))


@pytest.mark.parametrize("tiles", [1, 31, 32, 33, 63, 64, 100])
def test_every_chunk_is_in_one_tile(lib, tiles):
    for lg in range(7):
        times = (ctypes.c_int * (64 * tiles))()
        lib.cover(ctypes.c_int64(tiles), lg, times)
        assert set(times) == {1}


# (s, k, values, bytes of an index, R (0: compress), AdamW, log2 of a run's chunks; 6: no gangs)
@pytest.mark.parametrize("s,k,val,idx,R,adam,want", [
    (64, 32, 0, 4, 0, 0, 3), (64, 4, 0, 4, 0, 0, 3), (64, 2, 0, 4, 0, 0, 4), (64, 1, 0, 4, 0, 0, 6), (32, 16, 0, 4, 0, 0, 4),
    (32, 4, 0, 4, 0, 0, 4), (32, 2, 0, 4, 0, 0, 4), (32, 4, 3, 1, 0, 0, 6), (64, 32, 2, 1, 0, 0, 3), (16, 4, 0, 4, 0, 0, 5),
    (128, 16, 0, 4, 0, 0, 2), (96, 12, 0, 4, 0, 0, 6), (192, 24, 0, 4, 0, 0, 6), (256, 32, 0, 4, 0, 0, 6), (64, 32, 0, 0, 0, 0, 3),
    (64, 32, 0, 4, 4, 0, 3), (64, 16, 0, 4, 4, 0, 4), (64, 8, 0, 4, 4, 0, 3), (64, 8, 0, 4, 16, 0, 6), (64, 4, 0, 4, 4, 0, 6),
    (32, 4, 0, 4, 4, 0, 4), (64, 4, 0, 4, 4, 1, 3), (64, 4, 0, 4, 32, 1, 4), (64, 8, 0, 4, 16, 1, 3), (128, 32, 0, 4, 4, 0, 3),
    (64, 16, 2, 1, 4, 1, 3)])
def test_runs(lib, s, k, val, idx, R, adam, want):
    assert lib.run_log2(s, k, val, idx, R, adam) == want


@pytest.mark.parametrize("s,k,val,lg,adam,amsgrad,classes,want", [
    (64, 32, 0, 3, 0, 0, 4, 1), (64, 32, 0, 6, 0, 0, 4, 0), (64, 32, 0, 3, 0, 0, 0, 0), (64, 30, 0, 3, 0, 0, 4, 0),
    (64, 32, 2, 3, 0, 0, 4, 0), (64, 32, 2, 3, 1, 0, 4, 1), (64, 32, 2, 3, 1, 0, 2, 0), (64, 32, 0, 3, 1, 1, 4, 0),
    (16, 4, 0, 5, 0, 0, 2, 0), (128, 32, 0, 3, 0, 0, 4, 1)])
def test_decompress_gangs(lib, s, k, val, lg, adam, amsgrad, classes, want):
    assert lib.gangs(s, k, val, lg, adam, amsgrad, classes) == want
