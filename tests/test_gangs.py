"""Tiles in gangs: which launches have them, and that their runs are every chunk once."""
import ctypes
import os
import subprocess

import pytest

from paper_2502_06728_amd import build
from tests import test_gpu_gangs as on_gpu

DRIVER = r"""
#include "tiled_launch.h"
extern "C" int run_log2(int s, int k, int val, int idx_bytes, int R, int adam) {
    return deto::run_log2(s, k, val, idx_bytes, R ? deto::decompress_run_bytes(s, k, R, adam != 0) : deto::kRunBytes);
}
static deto::KParams params(int s, int k, int R, int val, int adam) {
    deto::KParams p = {};
    p.s = s; p.k = k; p.R = R; p.val_dtype = val; p.idx_u8 = val != 0; p.adam = adam != 0; p.amsgrad = adam == 2;
    return p;
}
// transmitted indices: -1 in a row, else workgroups per CU
extern "C" int gangs(int s, int k, int R, int val, int u8, int adam, int bf16, int64_t n) {
    deto::KParams p = params(s, k, R, val, adam);
    p.idx_u8 = u8;
    p.run_lg = deto::decompress_run_log2(p, n, true, bf16 != 0);
    const int classes = deto::decompress_classes(p, n, bf16 != 0, deto::lane_decompress(p));
    return deto::decompress_gangs(p, n, bf16 != 0, classes) ? deto::decompress_gang_workgroups(p, n, bf16 != 0) : -1;
}
extern "C" int scheme_lg(int s, int k, int R, int val, int bf16, int64_t n) {
    deto::KParams p = params(s, k, R, val, 0);
    p.scheme = 2; p.use_dct = 1;
    return deto::decompress_run_log2(p, n, false, bf16 != 0);
}
extern "C" int compress_lg(int s, int k, int64_t n) { return deto::compress_run_log2(params(s, k, 1, 0, 0), n); }
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


def test_compress_from_2_to_the_20_on(lib, monkeypatch):
    monkeypatch.delenv("DETO_SMALL_SHARD_TILES")
    line = 1 << 20
    assert lib.compress_lg(32, 8, ctypes.c_int64(line)) == 6 and lib.compress_lg(32, 8, ctypes.c_int64(line + 1)) == 4
    monkeypatch.setenv("DETO_SMALL_SHARD_TILES", "0")                     # (no shard is small)
    assert lib.compress_lg(32, 8, ctypes.c_int64(line)) == 4


F32, F16, SIGNS = 0, 2, 3
SGD, ADAM, AMSGRAD = 0, 1, 2


# (s, k, R, values, optimizer, bf16 parameters, elements, -1 in a row or workgroups per CU in gangs), both sides of lines
@pytest.mark.parametrize("s,k,R,val,opt,bf16,n,want", [
    # AdamW: a quarter of the chunk or two replicas; 16-bit values at chunk 64 and 128 up to R*k = s
    (64, 16, 4, F32, ADAM, 1, 1 << 23, -1), (64, 16, 4, F32, ADAM, 1, (1 << 23) + 1, 0), (64, 16, 4, F32, ADAM, 0, (1 << 24) + 1, 3),
    (64, 12, 3, F32, ADAM, 1, 1 << 27, -1), (64, 12, 2, F32, ADAM, 1, 1 << 27, 3), (64, 16, 4, F32, AMSGRAD, 1, 1 << 27, -1),
    (64, 15, 4, F32, ADAM, 1, 1 << 27, -1), (128, 32, 4, F32, ADAM, 1, 1 << 25, 0), (128, 32, 4, F32, ADAM, 1, 1 << 26, 3),
    (128, 32, 5, F32, ADAM, 1, 1 << 26, 0), (32, 8, 4, F32, ADAM, 0, 1 << 26, 5), (32, 8, 4, F32, ADAM, 1, 1 << 26, 0),
    (64, 16, 4, F16, ADAM, 1, (1 << 23) + 1, 4), (64, 16, 4, F16, ADAM, 0, (1 << 23) + 1, 3), (64, 16, 5, F16, ADAM, 1, 1 << 26, -1),
    (128, 64, 2, F16, ADAM, 1, 1 << 26, 3), (128, 64, 3, F16, ADAM, 1, 1 << 26, -1), (32, 16, 2, F16, ADAM, 1, 1 << 26, -1),
    (64, 32, 2, SIGNS, ADAM, 1, 1 << 26, -1), (128, 64, 2, SIGNS, ADAM, 1, 1 << 26, -1), (96, 24, 4, F32, ADAM, 1, 1 << 26, -1),
    # plain update, fp32 values
    (64, 32, 2, F32, SGD, 1, 1 << 25, -1), (64, 32, 2, F32, SGD, 1, (1 << 25) + 1, 4), (64, 32, 4, F32, SGD, 1, 1 << 26, 3),
    (64, 32, 2, F32, SGD, 0, (1 << 23) + 1, 0), (64, 32, 1, F32, SGD, 0, 1 << 26, 0),
    (64, 16, 2, F32, SGD, 0, 1 << 24, 0), (64, 16, 2, F32, SGD, 0, (1 << 24) + 1, -1), (64, 20, 2, F32, SGD, 0, 1 << 24, -1),
    (64, 16, 2, F32, SGD, 1, 1 << 24, -1), (64, 16, 1, F32, SGD, 0, 1 << 26, 0),
    (64, 16, 1, F32, SGD, 1, 1 << 26, -1), (64, 12, 8, F32, SGD, 0, 1 << 26, -1), (64, 32, 4, F16, SGD, 0, 1 << 26, -1),
    (32, 16, 4, F32, SGD, 1, 1 << 26, -1), (32, 16, 5, F32, SGD, 1, 1 << 26, 4), (32, 8, 1, F32, SGD, 0, 1 << 26, 0),
    (128, 32, 4, F32, SGD, 0, 1 << 25, -1), (128, 32, 4, F32, SGD, 0, 1 << 26, 0), (128, 32, 5, F32, SGD, 0, 1 << 26, 3),
    (128, 32, 4, F32, SGD, 1, 1 << 26, -1), (128, 32, 5, F32, SGD, 1, 1 << 26, 3), (128, 28, 8, F32, SGD, 1, 1 << 26, -1)])
def test_decompress_gangs(lib, s, k, R, val, opt, bf16, n, want):
    assert lib.gangs(s, k, R, val, val != F32, opt, bf16, ctypes.c_int64(n)) == want


def test_the_shapes_of_the_tests_on_the_gpu_run_in_gangs(lib):
    for s, k, R, bf16 in on_gpu.PLAIN:
        assert lib.gangs(s, k, R, F32, 0, SGD, bf16, ctypes.c_int64(on_gpu.plain_size(s))) >= 0
    for s, k, R, val, u8, bf16 in on_gpu.ADAMW:
        assert lib.gangs(s, k, R, val, u8, ADAM, bf16, ctypes.c_int64(on_gpu.adamw_size(s))) >= 0


@pytest.mark.parametrize("s,k,R,val,bf16,n,want", [
    (64, 32, 1, F32, 1, 1 << 24, 6), (64, 32, 1, F32, 1, (1 << 24) + 1, 3), (64, 32, 1, F32, 0, 1 << 26, 6),
    (64, 32, 1, F16, 1, 1 << 26, 6), (64, 16, 15, F32, 1, 1 << 26, 6), (64, 16, 16, F32, 1, 1 << 26, 4),
    (32, 16, 1, F32, 1, 1 << 26, 4), (32, 8, 64, F32, 1, 1 << 26, 6)])
def test_decompress_gangs_of_coefficients(lib, s, k, R, val, bf16, n, want):
    assert lib.scheme_lg(s, k, R, val, bf16, ctypes.c_int64(n)) == want
