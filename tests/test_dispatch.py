"""The rules that choose a kernel by sizes and types (csrc/tiled_launch.h), compiled for the host and
asked at both sides of the lines that they draw."""
import ctypes
import os
import subprocess

import pytest

from paper_2502_06728_amd import build

F32, F16, SIGNS = 0, 2, 3
TOPK, STRIDE, RANDOM = 0, 1, 2
RAW = (RANDOM, False)                                    # Random on the momentum itself

DRIVER = r"""
#include "tiled_launch.h"
static deto::KParams params(const int* a) {
    deto::KParams p = {};
    p.s = a[0]; p.k = a[1]; p.R = a[2]; p.val_dtype = a[3]; p.idx_u8 = a[3] != 0;
    p.scheme = a[4]; p.use_dct = a[5]; p.adam = a[6];
    return p;
}
extern "C" int few(const int*, int64_t chunks) { return deto::few_chunks(chunks); }
extern "C" int few_decompress(const int* a, int64_t chunks) {
    return deto::few_chunks_decompress(params(a), chunks, a[4] == 0);
}
extern "C" int direct(const int* a, int64_t chunks) {
    return deto::direct_compress(params(a)) && !deto::few_direct(params(a), chunks);
}
// (of the kernels that the launch runs on: tiles in gangs or in a row)
static int compress_wgs_of(const int* a, int64_t tiles, bool bf16) {
    deto::CompressLaunch l = {};
    l.p = params(a);
    l.tiles = tiles;
    l.grad_bf16 = bf16;
    l.p.run_lg = deto::compress_run_log2(l.p, tiles * 64 * l.p.s);
    return deto::launch_workgroups(l);
}
extern "C" int compress_wgs(const int* a, int64_t t) { return compress_wgs_of(a, t, false); }
extern "C" int compress_wgs_bf16(const int* a, int64_t t) { return compress_wgs_of(a, t, true); }
static int decompress_wgs_of(const int* a, int64_t n, bool bf16) {
    deto::DecompressLaunch l = {};
    l.p = params(a);
    l.n = n;
    l.param_bf16 = bf16;
    l.idx = a[4] == 0 ? a : nullptr;
    l.p.run_lg = deto::decompress_run_log2(l.p, n, l.idx != nullptr, bf16);
    const int classes = l.idx ? deto::decompress_classes(l.p, n, bf16, deto::lane_decompress(l.p))
                              : deto::scheme_classes(l.p, n, bf16, deto::lane_scheme(l.p));
    return deto::launch_workgroups(l, classes);
}
extern "C" int decompress_wgs(const int* a, int64_t n) { return decompress_wgs_of(a, n, true); }
extern "C" int decompress_wgs_f32(const int* a, int64_t n) { return decompress_wgs_of(a, n, false); }
extern "C" int spare(const int* a, int64_t wgs) { return deto::spare_lds(static_cast<int>(wgs), a[0]); }
extern "C" int lane(const int* a, int64_t) { return deto::lane_decompress(params(a)); }
extern "C" int classes(const int* a, int64_t n, int bf16) {
    return deto::decompress_classes(params(a), n, bf16, deto::lane_decompress(params(a)));
}
extern "C" int lane_scheme(const int* a, int64_t) { return deto::lane_scheme(params(a)); }
extern "C" int scheme_classes(const int* a, int64_t n, int bf16) {
    return deto::scheme_classes(params(a), n, bf16, deto::lane_scheme(params(a)));
}
extern "C" int counts(const int* a, int64_t) { return deto::count_signs(params(a)); }
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
    assert rules("few", s, k, 63, 1, val, scheme, dct) and not rules("few", s, k, 64, 1, val, scheme, dct)


def test_few_chunks_of_many_replicas_signs_go_to_the_general_kernels(rules):
    assert rules("few_decompress", 128, 42, 2560, 16, SIGNS)
    assert not rules("few_decompress", 128, 42, 2561, 16, SIGNS)
    assert not rules("few_decompress", 128, 42, 2560, 2, SIGNS)
    assert not rules("few_decompress", 128, 42, 2560, 16, F16)


@pytest.mark.parametrize("s,val,few", [(16, SIGNS, 4096), (16, F16, 4096), (32, SIGNS, 4096), (64, SIGNS, 2048),
                                       (96, SIGNS, 0), (256, SIGNS, 0)])
def test_direct_sums_where_there_are_more_than_a_few_chunks(rules, s, val, few):
    assert not rules("direct", s, 3, few, 1, val) or few == 0
    assert rules("direct", s, 3, few + 1, 1, val)
    assert rules("direct", s, s, 1, 1, val)                 # (every entry kept: long sums)
    assert not rules("direct", s, 3, 1 << 20, 1, val, STRIDE, True)
    assert bool(rules("direct", s, 3, 1 << 20, 1, F16)) == (s == 16)


def test_workgroups_per_cu_of_large_launches(rules):
    for s, scheme, want in ((32, TOPK, 10), (32, RANDOM, 10), (16, TOPK, 10), (64, TOPK, 0)):
        assert rules("compress_wgs", s, 4, 10241, 1, F32, scheme, True) == want
        assert rules("compress_wgs", s, 4, 10240, 1, F32, scheme, True) == 0
    m26, m25 = 1 << 26, 1 << 25
    for s, k, R, scheme, n, want in ((64, 32, 2, TOPK, m25, 4), (64, 32, 4, TOPK, m25, 3), (64, 16, 2, TOPK, m26, 0),
                                     (64, 32, 16, TOPK, m26, 0), (32, 16, 2, TOPK, m26, 5), (32, 16, 4, TOPK, m25, 4),
                                     (64, 32, 4, RANDOM, m26, 5), (64, 32, 2, RANDOM, m26, 0),
                                     (32, 16, 4, RANDOM, m26, 6), (32, 16, 8, RANDOM, m26, 4)):
        assert rules("decompress_wgs", s, k, n + 1, R, F32, scheme) == want
        assert rules("decompress_wgs", s, k, n, R, F32, scheme) == 0
        assert rules("decompress_wgs", s, k, n + 1, R, F16, scheme) == 0
    # that many fit 160 KB, one more does not; within the 64 KB of a launch
    for wgs in (3, 4, 5, 6, 8, 10):
        for static in (9216, 10240, 17408):
            total = rules("spare", static, 1, wgs) + static
            assert total <= 65536 and (wgs + 1) * total > 163840
            assert wgs * total <= 163840 or total == static
    assert rules("spare", 9216, 1, 0) == 0


# (s, k, R, scheme, workgroups with bf16 and with fp32 parameters)
@pytest.mark.parametrize("s,k,R,scheme,bf16,f32", [
    # entries one by one, or few lanes of them: as many workgroups as fit
    (64, 2, 64, TOPK, 0, 0), (64, 2, 32, TOPK, 0, 0), (64, 1, 64, TOPK, 0, 0), (64, 30, 4, TOPK, 0, 0),
    (64, 18, 8, TOPK, 0, 0), (32, 1, 64, TOPK, 0, 0), (32, 2, 32, TOPK, 0, 0), (32, 15, 4, TOPK, 0, 0),
    (32, 2, 64, RANDOM, 0, 0), (32, 1, 64, RANDOM, 0, 0), (64, 2, 64, RANDOM, 0, 0), (64, 32, 8, RANDOM, 0, 0),
    # few entries a replica: more workgroups, or all
    (64, 4, 32, TOPK, 6, 6), (64, 4, 16, TOPK, 0, 6), (64, 8, 16, TOPK, 4, 4), (64, 12, 16, TOPK, 0, 4),
    (32, 4, 16, TOPK, 8, 6), (32, 8, 4, TOPK, 0, 5), (32, 12, 4, TOPK, 8, 5), (32, 8, 8, TOPK, 5, 4),
    (32, 12, 8, TOPK, 5, 4),
    # the other lines
    (64, 16, 16, TOPK, 3, 3), (64, 20, 4, TOPK, 4, 4), (32, 16, 2, TOPK, 5, 6), (32, 16, 3, TOPK, 5, 5),
    (32, 20, 2, TOPK, 6, 5), (32, 24, 2, TOPK, 5, 5), (32, 24, 4, TOPK, 4, 4), (64, 4, 32, RANDOM, 0, 0), (64, 4, 32, RAW, 5, 0), (64, 16, 16, RANDOM, 5, 5),
    (32, 4, 16, RANDOM, 6, 0), (32, 4, 32, RANDOM, 5, 0),
    # chunk 96 and 128 by classes; twelve entries on two classes
    (128, 16, 4, TOPK, 0, 3), (128, 32, 4, TOPK, 3, 0), (128, 24, 4, TOPK, 0, 3), (128, 8, 8, TOPK, 0, 0),
    (128, 16, 2, TOPK, 0, 0), (96, 12, 4, TOPK, 0, 4), (96, 24, 4, TOPK, 0, 4), (96, 12, 2, TOPK, 0, 0),
    (32, 12, 2, TOPK, 8, 0), (32, 8, 3, TOPK, 0, 0), (32, 12, 1, TOPK, 0, 0)])
def test_workgroups_by_entries_and_parameters(rules, s, k, R, scheme, bf16, f32):
    scheme, dct = scheme if scheme == RAW else (scheme, True)
    for n in ((1 << 26) + 1, 147095552):
        assert rules("decompress_wgs", s, k, n, R, F32, scheme, dct) == bf16
        assert rules("decompress_wgs_f32", s, k, n, R, F32, scheme, dct) == f32
        if scheme == TOPK and rules("classes", s, k, n, R, F32, TOPK, True, 0, 1) == 0:
            assert bf16 == 0                                  # (one wavefront a workgroup)


# (s, k, R, values, scheme, elements from which on, workgroups with bf16 and with fp32 parameters)
@pytest.mark.parametrize("s,k,R,val,scheme,line,bf16,f32", [
    (64, 16, 4, SIGNS, TOPK, 23, 4, 0), (64, 32, 2, F16, TOPK, 23, 4, 3), (64, 32, 8, SIGNS, TOPK, 23, 0, 0),
    (64, 16, 4, F32, TOPK, 24, 3, 3), (64, 5, 4, SIGNS, TOPK, 23, 0, 0),
    (64, 16, 4, SIGNS, RANDOM, 25, 0, 0), (64, 16, 4, F32, RANDOM, 25, 4, 0),
    (96, 12, 4, F16, TOPK, 23, 4, 4), (96, 24, 4, F32, TOPK, 25, 4, 0),
    (96, 12, 4, F32, RANDOM, 25, 4, 0), (32, 8, 4, F32, RANDOM, 25, 5, 0), (32, 8, 4, F32, TOPK, 25, 0, 5),
    (32, 4, 8, SIGNS, RANDOM, 25, 0, 0), (128, 16, 4, F32, TOPK, 25, 0, 0),
    (32, 16, 4, SIGNS, TOPK, 26, 5, None), (32, 4, 2, SIGNS, TOPK, 23, None, 5), (32, 1, 4, F16, TOPK, 26, 5, None),
    (32, 4, 4, SIGNS, TOPK, 23, 0, 5), (32, 2, 8, SIGNS, TOPK, 23, 0, 0),
    (32, 8, 3, SIGNS, RANDOM, 24, 0, 6), (32, 16, 4, F16, RANDOM, 24, 0, 5)])
def test_workgroups_of_adamw(rules, s, k, R, val, scheme, line, bf16, f32):
    for n, on in ((1 << line, False), ((1 << line) + 1, True), (147095552, True)):
        for name, want in (("decompress_wgs", bf16), ("decompress_wgs_f32", f32)):
            if want is not None:                              # (None: its line is another one)
                assert rules(name, s, k, n, R, val, scheme, True, 1) == (want if on else 0)


def test_one_or_two_bf16_entries_of_16_are_limited_later(rules):
    for name, k, tiles, want in (("compress_wgs_bf16", 1, 32768, 0), ("compress_wgs_bf16", 2, 32768, 0),
                                 ("compress_wgs_bf16", 2, 32769, 8), ("compress_wgs_bf16", 4, 10241, 10),
                                 ("compress_wgs", 1, 10241, 10)):
        assert rules(name, 16, k, tiles) == want


def test_signs_of_many_replicas_are_counted(rules):
    for k, R in ((17, 16), (4, 32), (3, 48), (16, 32)):
        assert rules("counts", 64, k, 0, R, SIGNS, RANDOM, True) and not rules("counts", 64, k, 0, R - 1, SIGNS, RANDOM, True)
        assert not rules("counts", 64, k, 0, R, F16, RANDOM, True)


def tiles(s, t):
    return 64 * s * t + 1


def test_lane_kernels_are_those_that_are_built(rules):
    """The table behind the rules against the lists of the units."""
    for s, ks in ((16, (1, 2, 4, 8)), (32, (1, 2, 4, 8, 16)), (64, (1, 2, 4, 8, 16, 32)), (96, (6, 12, 24, 48)),
                  (128, (1, 4, 8, 16, 32, 64)), (192, ()), (256, ()), (48, ())):
        assert tuple(k for k in range(1, s + 1) if rules("lane", s, k, 0)) == ks
        assert not any(rules("lane", s, k, 0, adam=1) for k in range(1, s + 1))
    for val, pairs in ((F16, {(64, 32), (64, 16), (64, 8), (32, 16), (32, 8), (32, 4), (32, 2), (32, 1)}),
                       (SIGNS, {(64, 32), (64, 16), (32, 16), (32, 8), (32, 4), (32, 2), (32, 1)})):
        got = {(s, k) for s in range(1, 257) for k in range(1, s + 1) if rules("lane", s, k, 0, val=val)}
        assert got == pairs


@pytest.mark.parametrize("s,k,R,val,adam,bf16,n,want", [
    # AdamW: idle lanes with many replicas
    (32, 4, 16, SIGNS, 1, 1, tiles(32, 1025), 2), (32, 4, 16, SIGNS, 1, 1, tiles(32, 1024), 4),
    (32, 4, 8, SIGNS, 1, 1, tiles(32, 1025), 4), (64, 32, 16, F16, 1, 0, tiles(64, 1025), 4),
    (64, 21, 16, F32, 1, 1, tiles(64, 100), 4), (128, 42, 16, SIGNS, 1, 0, tiles(128, 2000), 4),
    # few tiles
    (64, 21, 2, F32, 0, 1, tiles(64, 1024), 4), (64, 5, 2, F32, 0, 1, tiles(64, 1025), 2),
    (64, 8, 2, F32, 0, 0, tiles(64, 1536), 0), (64, 8, 2, F32, 0, 0, tiles(64, 1537), 2),
    (64, 32, 2, F32, 0, 0, tiles(64, 1537), 4), (64, 2, 16, F32, 0, 0, tiles(64, 1537), 2),
    (128, 16, 2, F32, 0, 0, tiles(128, 640), 4), (128, 16, 2, F32, 0, 0, tiles(128, 641), 0),
    (128, 16, 2, F32, 0, 0, tiles(128, 1024), 0), (128, 16, 2, F32, 0, 0, tiles(128, 1025), 4),
    (96, 12, 2, F32, 0, 1, tiles(96, 100), 0), (96, 32, 16, F32, 0, 0, tiles(96, 1025), 4),
    # many entries, idle lanes
    (32, 16, 16, F32, 0, 0, tiles(32, 5000), 0), (32, 16, 15, F32, 0, 0, tiles(32, 5000), 2),
    (128, 64, 16, F32, 0, 0, tiles(128, 5000), 0), (128, 1, 16, F32, 0, 1, tiles(128, 1025), 0),
    # large shards of bf16 parameters
    (64, 32, 4, F32, 0, 1, 1 << 25, 0), (64, 32, 4, F32, 0, 1, (1 << 25) + 1, 4),
    (64, 8, 4, F32, 0, 1, (1 << 25) + 1, 2), (64, 4, 16, F32, 0, 1, (1 << 25) + 1, 2),
    (64, 8, 2, F32, 0, 1, (1 << 25) + 1, 0), (64, 32, 4, F16, 0, 1, (1 << 25) + 1, 0),
    (128, 16, 4, F32, 0, 1, 1 << 25, 4), (128, 16, 4, F32, 0, 1, (1 << 25) + 1, 0),
    (128, 16, 8, F32, 0, 1, (1 << 25) + 1, 4), (128, 5, 2, F16, 0, 1, (1 << 25) + 1, 2),
    # no class kernels; chunk 16
    (48, 6, 2, F32, 0, 1, tiles(48, 100), 0), (256, 32, 2, F32, 0, 1, tiles(256, 100), 4),
    (16, 4, 2, F32, 0, 1, tiles(16, 100), 0), (16, 4, 2, F32, 0, 0, tiles(16, 100), 2),
    (16, 3, 2, F32, 0, 1, tiles(16, 100), 2)])
def test_decompress_classes(rules, s, k, R, val, adam, bf16, n, want):
    assert rules("classes", s, k, n, R, val, TOPK, True, adam, bf16) == want


def test_lane_kernels_of_the_schemes(rules):
    for val, pairs in ((F32, {(64, k) for k in (1, 2, 4, 8, 16, 32)} | {(32, k) for k in (1, 2, 4, 8, 16)} |
                        {(16, 1), (16, 2)}),
                       (SIGNS, {(64, k) for k in (4, 8, 16, 32)} | {(32, k) for k in (1, 2, 4, 8, 16)})):
        got = {(s, k) for s in range(1, 257) for k in range(1, s + 1)
               if rules("lane_scheme", s, k, 0, val=val, scheme=RANDOM)}
        assert got == pairs


@pytest.mark.parametrize("s,k,val,adam,bf16,n,want", [
    (16, 2, F32, 0, 1, tiles(16, 10000), 0), (16, 1, F32, 0, 0, tiles(16, 6144), 0),
    (16, 1, F32, 0, 0, tiles(16, 6145), 2), (16, 2, F32, 0, 0, tiles(16, 10000), 0),
    (16, 2, F16, 0, 1, tiles(16, 10000), 2), (16, 2, F32, 1, 1, tiles(16, 10000), 2),
    (64, 8, F32, 0, 0, tiles(64, 3072), 0), (64, 8, F32, 0, 0, tiles(64, 3073), 2),
    (64, 8, F32, 0, 1, 1 << 28, 0), (64, 16, F32, 0, 0, tiles(64, 10000), 0),
    (64, 32, F32, 0, 1, 1 << 28, 0), (32, 4, F32, 0, 0, tiles(32, 3073), 2),
    (32, 4, SIGNS, 0, 0, tiles(32, 10000), 0), (32, 2, SIGNS, 0, 0, tiles(32, 10000), 2),
    (64, 32, SIGNS, 1, 1, tiles(64, 10000), 4), (32, 4, SIGNS, 1, 0, tiles(32, 100), 4),
    (64, 2, SIGNS, 0, 1, tiles(64, 1000), 4), (64, 2, SIGNS, 0, 1, tiles(64, 2000), 2),
    (128, 16, F32, 0, 1, tiles(128, 100), 4), (48, 4, F32, 0, 1, tiles(48, 100), 0)])
def test_scheme_classes(rules, s, k, val, adam, bf16, n, want):
    for dct in (False, True):
        assert rules("scheme_classes", s, k, n, 4, val, RANDOM, dct, adam, bf16) == want
