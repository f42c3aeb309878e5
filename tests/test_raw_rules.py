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
extern "C" int quads(int s, int k, int R, int adam, int64_t n) {
    return deto::raw_decompress_quads(params(s, k, R, 0, adam), n);
}
extern "C" int built(int s, int q) {
#define X(S, Q) if (s == S && q == Q) return 1;
    DETO_RAW_DECOMPRESS_LIST(X)
#undef X
    return 0;
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
                        assert lib.built(s, lib.quads(s, k, R, adam, ctypes.c_int64(n)))


@pytest.mark.parametrize("s,k,val,bf16,n,want", [
    (64, 8, 0, 0, 1 << 17, 0), (64, 8, 0, 0, (1 << 17) + 1, 1), (128, 16, 0, 0, 64, 1), (64, 7, 0, 1, 1 << 23, 1),
    (64, 7, 0, 1, (1 << 23) + 1, 0), (128, 16, 3, 1, 1 << 30, 1), (64, 8, 0, 1, 1 << 26, 1), (64, 8, 0, 1, (1 << 26) + 1, 0),
    (64, 8, 0, 0, 1 << 30, 1), (64, 8, 2, 1, (1 << 23) + 1, 0), (64, 8, 2, 0, (1 << 23) + 1, 1), (32, 8, 0, 1, (1 << 23) + 1, 0)])
def test_decompress_rule(lib, s, k, val, bf16, n, want):
    assert lib.takes(s, k, val, bf16, ctypes.c_int64(n)) == want


@pytest.mark.parametrize("s,k,R,bf16,adam,n,want", [
    (32, 16, 15, 1, 0, 1 << 27, 0), (32, 16, 16, 1, 0, 1 << 27, 1), (32, 1, 31, 1, 0, 1 << 27, 0), (32, 1, 32, 1, 0, 1 << 27, 1),
    (32, 2, 16, 1, 0, 1 << 24, 0), (32, 2, 17, 1, 0, 1 << 24, 1), (32, 2, 16, 1, 0, (1 << 24) + 1, 1), (64, 4, 16, 1, 0, 1 << 24, 1),
    (64, 2, 32, 1, 0, 1 << 24, 0), (64, 2, 32, 1, 0, (1 << 24) + 1, 1),
    (64, 5, 1, 0, 0, 1 << 24, 1), (64, 3, 15, 0, 0, 1 << 24, 1), (64, 3, 16, 0, 0, 1 << 24, 0), (64, 3, 22, 0, 0, 1 << 24, 1),
    (32, 1, 32, 0, 0, 1 << 24, 0), (64, 1, 64, 0, 0, 1 << 24, 1), (64, 2, 32, 0, 0, 1 << 24, 0), (16, 1, 17, 0, 0, 1 << 24, 1),
    (64, 3, 64, 1, 1, 1 << 24, 0), (64, 5, 47, 1, 1, 1 << 24, 1), (64, 7, 48, 0, 1, 1 << 24, 0), (32, 5, 48, 0, 1, 1 << 24, 1),
    (64, 4, 64, 0, 1, 1 << 24, 1), (64, 3, 16, 0, 0, 1 << 23, 1)])
def test_decompress_rule_of_signs(lib, s, k, R, bf16, adam, n, want):
    assert lib.takes_signs(s, k, R, bf16, adam, ctypes.c_int64(n)) == want
