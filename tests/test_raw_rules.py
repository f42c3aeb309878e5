"""Which launches the streaming kernels of Striding and Random take, at both sides of the lines."""
import ctypes
import os
import subprocess

import pytest

from paper_2502_06728_amd import build

DRIVER = r"""
#include "tiled_launch.h"
static deto::KParams params(int s, int k, int R, int val, int adam) {
    deto::KParams p = {};
    p.s = s; p.k = k; p.R = R; p.val_dtype = val; p.idx_u8 = val != 0; p.scheme = 2; p.adam = adam;
    return p;
}
extern "C" int takes(int s, int k, int val, int bf16, int64_t n) {
    return deto::raw_decompress(params(s, k, 2, val, 0), n, bf16 != 0);
}
extern "C" int takes_signs(int s, int k, int R, int bf16, int adam, int64_t n) {
    return deto::raw_decompress(params(s, k, R, 3, adam), n, bf16 != 0);
}
extern "C" int compress_quads(int s, int k) { return deto::raw_compress_quads(params(s, k, 1, 0, 0)); }
extern "C" int quads(int s, int k, int R, int val, int adam, int64_t n) {
    return deto::raw_decompress_quads(params(s, k, R, val, adam), n);
}
extern "C" int built(int s, int q, int adam) {
#define X(S, Q) if (s == S && q == Q) return 1;
    DETO_RAW_DECOMPRESS_LIST(X)
#undef X
#define X(S, Q) if (s == S && q == Q) return !adam;
    DETO_RAW_DECOMPRESS_PLAIN_LIST(X)
#undef X
    return 0;
}
extern "C" int workgroups(int s, int k, int scheme, int val, int adam, int bf16, int64_t n) {
    deto::KParams p = params(s, k, 2, val, adam);
    p.scheme = scheme;
    return deto::raw_decompress_workgroups(p, n, bf16 != 0);
}
extern "C" int compresses(int s, int k, int scheme, int64_t n) {
    deto::KParams p = params(s, k, 1, 0, 0);
    p.scheme = scheme;
    return deto::raw_compress(p, n);
}
extern "C" int compress_workgroups(int s, int k, int scheme, int val, int bf16, int64_t n) {
    deto::KParams p = params(s, k, 1, val, 0);
    p.scheme = scheme;
    return deto::raw_compress_workgroups(p, n, bf16 != 0);
}
extern "C" int compress_built(int s, int q) {
#define X(S, Q) if (s == S && q == Q) return 1;
    DETO_RAW_COMPRESS_LIST(X)
#undef X
    return 0;
}
"""
SIZES = (1, 1 << 17, 1 << 22, (1 << 22) + 1, 1 << 23, (1 << 23) + 1, 1 << 25, 1 << 26, (1 << 26) + 1, 1 << 30)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("raw")
    (d / "raw.hip").write_text(DRIVER)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950",
                    "--cuda-host-only", "-std=c++17", "-O1", "-fPIC", "-shared", "-I", build.CSRC,
                    "-o", str(d / "raw.so"), str(d / "raw.hip")], check=True, capture_output=True)
    return ctypes.CDLL(str(d / "raw.so"))


def test_every_choice_is_built(lib):
    for s in (16, 32, 64, 96, 128, 192, 256):
        for k in range(1, s // 2 + 1):
            assert lib.compress_built(s, lib.compress_quads(s, k))
            for R in (1, 2, 7, 8, 15, 16, 64):
                for adam in (0, 1):
                    for n in SIZES:
                        for val in (0, 3):
                            assert lib.built(s, lib.quads(s, k, R, val, adam, ctypes.c_int64(n)), adam)


@pytest.mark.parametrize("s,k,val,bf16,n,want", [
    # a lane per chunk: small launches, and large ones of bf16 parameters
    (64, 8, 0, 0, 1 << 17, 0), (64, 8, 0, 0, (1 << 17) + 1, 1), (128, 16, 0, 0, 64, 1), (64, 8, 0, 1, 1 << 26, 1),
    (64, 8, 0, 1, (1 << 26) + 1, 0), (64, 8, 0, 0, 1 << 30, 1), (64, 8, 2, 1, 1 << 23, 1), (64, 8, 2, 1, (1 << 23) + 1, 0),
    (64, 8, 2, 0, (1 << 23) + 1, 1), (32, 8, 0, 1, (1 << 23) + 1, 0), (64, 7, 0, 1, 1 << 30, 1), (128, 16, 2, 1, 1 << 30, 1)])
def test_decompress_rule(lib, s, k, val, bf16, n, want):
    assert lib.takes(s, k, val, bf16, ctypes.c_int64(n)) == want


@pytest.mark.parametrize("s,k,R,bf16,adam,n,want", [
    # two-bit signs: more entries than the chunk has, where a lane per chunk serves them
    (32, 16, 6, 1, 0, 1 << 27, 0), (32, 16, 7, 1, 0, 1 << 27, 1), (64, 32, 2, 1, 0, 1 << 27, 0), (64, 32, 3, 1, 0, 1 << 27, 1),
    (32, 8, 4, 1, 0, 1 << 27, 0), (32, 8, 5, 1, 0, 1 << 27, 1), (32, 1, 32, 1, 0, 1 << 27, 0), (32, 1, 33, 1, 0, 1 << 27, 1),
    (32, 16, 2, 0, 0, 1 << 27, 1), (32, 4, 2, 0, 0, 1 << 23, 0), (32, 4, 3, 1, 0, 1 << 23, 1), (32, 4, 2, 0, 0, (1 << 23) + 1, 1),
    (32, 4, 1, 0, 1, 1 << 20, 1), (32, 3, 1, 0, 0, 1 << 20, 1), (32, 16, 2, 1, 1, 1 << 27, 1), (64, 2, 1, 1, 0, 1 << 27, 1)])
def test_decompress_rule_of_signs(lib, s, k, R, bf16, adam, n, want):
    assert lib.takes_signs(s, k, R, bf16, adam, ctypes.c_int64(n)) == want


# (s, k, R, values, AdamW, elements, pieces a thread)
@pytest.mark.parametrize("s,k,R,val,adam,n,want", [
    (64, 8, 2, 0, 0, 1 << 22, 2), (64, 8, 2, 0, 0, (1 << 22) + 1, 4), (64, 8, 16, 0, 0, 1 << 20, 2), (64, 8, 16, 0, 0, (1 << 20) + 1, 4),
    (64, 8, 8, 0, 0, 1 << 23, 4), (64, 8, 8, 0, 0, (1 << 23) + 1, 8), (64, 8, 7, 0, 0, 1 << 24, 4), (16, 8, 64, 0, 0, 1 << 24, 4),
    (64, 8, 1, 3, 0, 1 << 24, 8), (64, 8, 1, 3, 0, 1 << 23, 4), (256, 16, 1, 3, 0, 1 << 24, 4), (16, 8, 1, 3, 0, 1 << 24, 4),
    (64, 8, 2, 0, 1, 1 << 26, 2), (64, 8, 2, 0, 1, (1 << 26) + 1, 4), (128, 32, 2, 0, 1, 1 << 23, 2), (128, 32, 2, 0, 1, 1 << 24, 4),
    (64, 4, 16, 3, 1, 1 << 24, 4), (64, 4, 15, 3, 1, 1 << 24, 2), (64, 4, 16, 0, 1, 1 << 24, 2), (32, 16, 16, 3, 1, 1 << 24, 4), (96, 8, 2, 0, 0, 1 << 22, 3),
    (96, 8, 2, 0, 0, 1 << 23, 6), (192, 8, 2, 0, 1, 1 << 23, 3), (192, 8, 2, 0, 1, 1 << 24, 6), (256, 64, 4, 0, 0, 1 << 24, 8),
    (256, 64, 3, 0, 0, 1 << 24, 4), (256, 64, 4, 0, 1, 1 << 24, 4)])
def test_pieces_of_a_thread(lib, s, k, R, val, adam, n, want):
    assert lib.quads(s, k, R, val, adam, ctypes.c_int64(n)) == want


def test_compress_rule(lib):
    for s, k, scheme, want in ((96, 25, 2, 0), (96, 24, 2, 1), (96, 25, 1, 1), (64, 32, 2, 1), (256, 128, 2, 0)):
        assert lib.compresses(s, k, scheme, ctypes.c_int64(1 << 16)) == want
        assert lib.compresses(s, k, scheme, ctypes.c_int64((1 << 16) + 1)) == 1


def test_workgroups_per_cu(lib):
    for val, adam, bf16, n, want in ((0, 0, 0, 1 << 25, 0), (0, 0, 0, (1 << 25) + 1, 5), (0, 0, 1, 1 << 27, 0), (0, 1, 1, 1 << 26, 3),
                                     (0, 1, 0, (1 << 26) + 1, 0), (3, 1, 0, 1 << 26, 3), (3, 1, 1, 1 << 26, 0), (2, 1, 0, 1 << 25, 0)):
        assert lib.workgroups(64, 8, 2, val, adam, bf16, ctypes.c_int64(n)) == want
    # AdamW (fp32 parameters, bf16): none where Random's shuffle is long for the workgroup's elements
    for s, k, scheme, f32, bf16 in ((64, 20, 2, 3, 3), (64, 21, 2, 3, 0), (64, 32, 1, 3, 3), (64, 32, 2, 3, 0), (128, 64, 2, 3, 3),
                                    (256, 78, 2, 3, 0), (256, 79, 2, 0, 0), (256, 128, 1, 3, 3), (96, 30, 2, 3, 3), (96, 31, 2, 3, 0)):
        for on_bf16, want in ((0, f32), (1, bf16)):
            assert lib.workgroups(s, k, scheme, 0, 1, on_bf16, ctypes.c_int64(1 << 26)) == want
    # compress (fp32 gradients, bf16): more where Random's shuffle is long for the workgroup's elements
    for s, k, scheme, val, f32, bf16 in ((64, 32, 1, 0, 4, 5), (64, 25, 2, 3, 4, 5), (64, 26, 2, 3, 6, 0), (64, 26, 2, 2, 5, 6),
                                         (64, 32, 2, 0, 5, 5), (96, 48, 2, 3, 6, 0), (96, 48, 2, 2, 4, 5), (128, 64, 2, 0, 4, 5),
                                         (192, 59, 2, 1, 5, 6), (192, 60, 2, 1, 0, 0), (192, 38, 2, 1, 4, 5), (192, 39, 2, 0, 5, 5),
                                         (256, 78, 2, 3, 6, 0), (256, 79, 2, 0, 0, 0), (256, 128, 1, 0, 4, 5), (256, 51, 2, 0, 4, 5)):
        for on_bf16, want in ((0, f32), (1, bf16)):
            assert lib.compress_workgroups(s, k, scheme, val, on_bf16, ctypes.c_int64(1 << 24)) == 0
            assert lib.compress_workgroups(s, k, scheme, val, on_bf16, ctypes.c_int64((1 << 24) + 1)) == want
