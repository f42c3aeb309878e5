"""The rules that choose a kernel by sizes and types (csrc/tiled_launch.h), compiled for the host and
asked at both sides of the lines that they draw."""
import ctypes
import os
import subprocess

import pytest

from paper_2502_06728_amd import build

F32, F16, SIGNS = 0, 2, 3
TOPK, STRIDE, RANDOM = 0, 1, 2

DRIVER = r"""
#include "tiled_launch.h"
static deto::KParams params(const int* a) {
    deto::KParams p = {};
    p.s = a[0]; p.k = a[1]; p.R = a[2]; p.val_dtype = a[3]; p.idx_u8 = a[3] != 0;
    p.scheme = a[4]; p.use_dct = a[5]; p.adam = a[6];
    return p;
}
extern "C" int few(const int* a, int64_t chunks) { return deto::few_chunks(params(a), chunks); }
extern "C" int few_decompress(const int* a, int64_t chunks) {
    return deto::few_chunks_decompress(params(a), chunks, a[4] == 0);
}
extern "C" int stream_first(const int* a, int64_t) { return deto::stream_before_classes(params(a)); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("dispatch")
    (d / "rules.hip").write_text(DRIVER)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950",
                    "--cuda-host-only", "-std=c++17", "-O1", "-fPIC", "-shared", "-I", build.CSRC,
                    "-o", str(d / "rules.so"), str(d / "rules.hip")], check=True, capture_output=True)
    lib = ctypes.CDLL(str(d / "rules.so"))

    def call(name, s, k, count, R=2, val=F32, scheme=TOPK, dct=None, adam=0, *more):
        dct = scheme == TOPK if dct is None else dct
        a = (ctypes.c_int * 7)(s, k, R, val, scheme, int(dct), adam)
        return getattr(lib, name)(a, ctypes.c_int64(count), *more)

    return call


@pytest.mark.parametrize("s,k,val,scheme,dct", [(64, 21, SIGNS, TOPK, True), (256, 32, F32, RANDOM, False),
                                                (128, 16, F16, STRIDE, True), (32, 4, F32, TOPK, True)])
def test_less_than_a_tile_goes_to_the_general_kernels(rules, s, k, val, scheme, dct):
    for R in (1, 64):
        for adam in (0, 1):
            assert rules("few_decompress", s, k, 63, R, val, scheme, dct, adam)
            assert rules("few_decompress", s, k, 1, R, val, scheme, dct, adam)
    assert rules("few", s, k, 63, 1, val, scheme, dct)


def test_a_round_of_chunks_without_a_transform_goes_to_the_general_kernels(rules):
    # compress: up to a round of single-wavefront workgroups; a long shuffle less
    for scheme, k, limit in ((STRIDE, 64, 5120), (RANDOM, 16, 5120), (RANDOM, 64, 2048)):
        assert rules("few", 128, k, limit, 1, SIGNS, scheme, False)
        assert not rules("few", 128, k, limit + 1, 1, SIGNS, scheme, False)
        assert not rules("few", 128, k, 1000, 1, SIGNS, scheme, True)
    # decompress: a few replicas at the larger chunk sizes
    for adam, limit in ((0, 2560), (1, 4096)):
        for s, R, few in ((96, 2, True), (256, 7, True), (64, 2, False), (256, 8, False)):
            assert bool(rules("few_decompress", s, 8, limit, R, F16, RANDOM, False, adam)) == few
            assert not rules("few_decompress", s, 8, limit + 1, R, F16, RANDOM, False, adam)
            assert not rules("few_decompress", s, 8, limit, R, F16, RANDOM, True, adam)
    # top-k: signs of many replicas only
    assert rules("few_decompress", 128, 42, 2560, 16, SIGNS)
    assert not rules("few_decompress", 128, 42, 2561, 16, SIGNS)
    assert not rules("few_decompress", 128, 42, 2560, 2, SIGNS)
    assert not rules("few_decompress", 128, 42, 2560, 16, F16)


def test_adamw_striding_streams_at_the_larger_chunks_only(rules):
    for s, adam, stream in ((64, 0, True), (32, 1, False), (64, 1, False), (96, 1, True), (192, 1, True)):
        assert bool(rules("stream_first", s, s // 8, 0, 2, F32, STRIDE, False, adam)) == stream
