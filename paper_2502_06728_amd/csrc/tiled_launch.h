// Host-side launchers of the tiled kernels.  Each translation unit tiled_*.hip instantiates
// one family of kernels and defines its launcher, so the families compile in parallel.
// A launcher returns true if it has a kernel for (p.s, p.k) and has enqueued it.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

#include "deto_device.hip.h"

namespace deto {

constexpr int64_t kLargeShard = int64_t{1} << 25;   // elements from which on memory decides, not latency

struct CompressLaunch {
    KParams p;
    int64_t tiles;          // full 64-chunk tiles, one workgroup each
    int64_t n;              // shard length
    int64_t n_chunks;       // ceil(n / s): the chunks past the last full tile ride along
    const void* grad;
    bool grad_bf16;
    float* mom;
    void* idx;              // may be null for Striding/Random; dtype per p.idx_u8
    void* val;              // dtype per p.val_dtype
    float* coeff_dbg;
    uint32_t stride_mask[4];  // Striding: kept positions of every chunk (bit i%32 of word i/32)
    hipStream_t stream;
};

struct DecompressLaunch {
    KParams p;
    int64_t tiles;
    int64_t n;
    int64_t n_chunks;
    const void* idx;        // null: indices regenerated from the scheme
    int64_t idx_stride;     // replica strides in elements
    const void* val;
    int64_t val_stride;
    void* params;
    bool param_bf16;
    float* presign_dbg;
    uint32_t stride_mask[4];
    hipStream_t stream;
    AdamPtrs adam;          // moment arrays when p.adam
};

// A shard of at most this many 64-chunk tiles counts as small: the launch is a few occupancy
// rounds long, so what a tile takes from its first load to its last store decides the duration,
// not the instructions per element.  The compress half then spreads a tile over more wavefronts
// (chunk 64: two coefficient classes instead of a lane per chunk, and four up to 512 tiles; chunk 128:
// four instead of two).  Measured on MI355X: 4 - 13 % shorter launches at 1,300 - 8,000 tiles, 4 - 5 % longer
// ones at 36,000.  The environment variable DETO_SMALL_SHARD_TILES overrides the limit (0: never).
inline int64_t small_shard_tiles() {
    const char* e = getenv("DETO_SMALL_SHARD_TILES");
    if (e && *e) {
        char* end = nullptr;
        const long long v = strtoll(e, &end, 10);
        if (end != e && v >= 0) return static_cast<int64_t>(v);
    }
    return 8192;
}

// grid of a launch: one workgroup per tile plus one per tail chunk
inline unsigned tiled_grid(int64_t tiles, int64_t n_chunks) {
    return static_cast<unsigned>(tiles + (n_chunks - tiles * kWave));
}

// What the lane-per-chunk kernels are instantiated for: the k values of each chunk size with fp32
// values and int32 indices, and the (chunk, k) pairs with byte indices and 16-bit values or two-bit
// signs; for Striding and Random the (chunk, k) pairs with fp32 and with narrow values.
#ifdef DETO_TILED_ONLY_64_32   // development builds: one instantiation, seconds to compile
#define DETO_LANE_TOPK_16(X)
#define DETO_LANE_TOPK_32(X)
#define DETO_LANE_TOPK_64(X) X(32)
#define DETO_LANE_TOPK_96(X)
#define DETO_LANE_TOPK_128(X)
#define DETO_LANE_16BIT_32(X)
#define DETO_LANE_16BIT_64(X) X(64, 32)
#define DETO_LANE_SIGNS(X) X(64, 32)
#define DETO_LANE_SCHEME(X) X(64, 32)
#define DETO_LANE_SCHEME_SMALL(X)
#define DETO_LANE_SCHEME_NARROW_32(X)
#define DETO_LANE_SCHEME_NARROW_64(X) X(64, 32)
#else
#define DETO_LANE_TOPK_16(X) X(1) X(2) X(4) X(8)
#define DETO_LANE_TOPK_32(X) X(1) X(2) X(4) X(8) X(16)
#define DETO_LANE_TOPK_64(X) X(1) X(2) X(4) X(8) X(16) X(32)
#define DETO_LANE_TOPK_96(X) X(6) X(12) X(24) X(48)                 // decompress only
#define DETO_LANE_TOPK_128(X) X(1) X(4) X(8) X(16) X(32) X(64)      // decompress only
#define DETO_LANE_16BIT_32(X) X(32, 16) X(32, 8) X(32, 4) X(32, 2) X(32, 1)
#define DETO_LANE_16BIT_64(X) X(64, 32) X(64, 16) X(64, 8)
#define DETO_LANE_SIGNS(X) X(64, 32) X(64, 16) X(32, 16) X(32, 8) X(32, 4) X(32, 2) X(32, 1)
#define DETO_LANE_SCHEME(X) X(64, 32) X(64, 16) X(64, 8) X(32, 16) X(32, 8)
#define DETO_LANE_SCHEME_SMALL(X) X(32, 4) X(32, 2) X(32, 1) X(64, 4) X(64, 2) X(64, 1) X(16, 2) X(16, 1)
#define DETO_LANE_SCHEME_NARROW_32(X) X(32, 16) X(32, 8) X(32, 4) X(32, 2) X(32, 1)
#define DETO_LANE_SCHEME_NARROW_64(X) X(64, 32) X(64, 16) X(64, 8) X(64, 4)
#endif

bool launch_compress_topk_s64(const CompressLaunch& a);
bool launch_compress_topk_s32(const CompressLaunch& a);
bool launch_compress_topk_s16(const CompressLaunch& a);
bool launch_decompress_idx_s64(const DecompressLaunch& a);
bool launch_decompress_idx_s32(const DecompressLaunch& a);
bool launch_decompress_idx_s16(const DecompressLaunch& a);
bool launch_decompress_idx_s96(const DecompressLaunch& a);
bool launch_decompress_idx_s128(const DecompressLaunch& a);
bool launch_compress_topk_packed(const CompressLaunch& a);     // byte indices + 16-bit values
bool launch_decompress_idx_packed(const DecompressLaunch& a);
bool launch_compress_topk_packed_s32(const CompressLaunch& a);
bool launch_decompress_idx_packed_s32(const DecompressLaunch& a);
bool launch_compress_topk_ternary(const CompressLaunch& a);    // byte indices + two-bit signs
bool launch_decompress_idx_ternary(const DecompressLaunch& a);
bool launch_compress_scheme_narrow_s32(const CompressLaunch& a);   // Striding / Random, narrow payload
bool launch_decompress_scheme_narrow_s32(const DecompressLaunch& a);
bool launch_compress_scheme_narrow_s64(const CompressLaunch& a);
bool launch_decompress_scheme_narrow_s64(const DecompressLaunch& a);
bool launch_compress_scheme(const CompressLaunch& a);
bool launch_decompress_scheme(const DecompressLaunch& a);
bool launch_compress_scheme_small(const CompressLaunch& a);    // low compression rates
bool launch_decompress_scheme_small(const DecompressLaunch& a);

// Matrix-core kernels: tiles of 32 complete chunks, persistent single-wavefront workgroups.
// A launcher returns the number of leading chunks it has taken (0: no kernel for this request).
// NB = chunk size / 32.  What nothing else takes: both halves at 160 and 224; compress at 32 and 64
// with k > s/2, and with 16-bit values or byte indices (at 32 also fp32 + int32) at a k without a
// lane-per-chunk kernel.
#ifdef DETO_TILED_ONLY_64_32
#define DETO_MFMA_COMPRESS_LIST(X) X(2)
#define DETO_MFMA_DECOMPRESS_LIST(X) X(5)
#else
#define DETO_MFMA_COMPRESS_LIST(X) X(1) X(2) X(5) X(7)
#define DETO_MFMA_DECOMPRESS_LIST(X) X(5) X(7)
#endif

inline unsigned mfma_grid(int64_t tiles, size_t smem_bytes) {
    const int64_t per_cu = static_cast<int64_t>((160u * 1024u) / smem_bytes);   // LDS-limited
    const int64_t cap = 256 * (per_cu < 8 ? per_cu : 8);
    return static_cast<unsigned>(tiles < cap ? tiles : cap);
}

int64_t launch_compress_mfma(const CompressLaunch& a);
int64_t launch_decompress_mfma(const DecompressLaunch& a);

// Two-lanes-per-chunk kernels (register-resident fast DCT split between lanes t and t+32): the
// chunk sizes that do not fit one lane.  Same tiles and return convention.
int64_t launch_compress_pair_96(const CompressLaunch& a);    // one translation unit each:
int64_t launch_compress_pair_128(const CompressLaunch& a);   // the longest compiles
int64_t launch_compress_pair_192(const CompressLaunch& a);
int64_t launch_compress_pair_256(const CompressLaunch& a);
inline int64_t launch_compress_pair(const CompressLaunch& a) {
    int64_t c = launch_compress_pair_96(a);
    if (!c) c = launch_compress_pair_128(a);
    if (!c) c = launch_compress_pair_192(a);
    return c ? c : launch_compress_pair_256(a);
}

// Lane per chunk, wavefront per coefficient class (split_kernels.hip.h): tiles of 64 chunks,
// k <= s/2 in the compress half.  Same return convention.
int64_t launch_decompress_split(const DecompressLaunch& a, int classes);        // fp32 + int32
int64_t launch_decompress_split_narrow(const DecompressLaunch& a, int classes); // other formats
int64_t launch_compress_split_scheme(const CompressLaunch& a);                   // Striding / Random
int64_t launch_decompress_split_scheme(const DecompressLaunch& a, int classes);  // ... no indices
int64_t launch_decompress_split_amsgrad(const DecompressLaunch& a, int classes); // the same three,
int64_t launch_decompress_split_narrow_amsgrad(const DecompressLaunch& a, int classes);   // AdamW
int64_t launch_decompress_split_scheme_amsgrad(const DecompressLaunch& a, int classes);   // with amsgrad
int64_t launch_decompress_split_scheme_counts(const DecompressLaunch& a, int classes);   // count_signs
int64_t launch_decompress_split_scheme_counts_amsgrad(const DecompressLaunch& a, int classes);
// Striding / Random on the momentum itself (raw_kernels.hip.h): (chunk size, pieces of four elements a
// thread)
#define DETO_RAW_COMPRESS_LIST(X) X(16, 2) X(32, 2) X(64, 2) X(96, 3) X(128, 2) X(128, 4) X(192, 3) X(256, 4)
#define DETO_RAW_DECOMPRESS_LIST(X) \
    X(16, 2) X(16, 4) X(32, 2) X(32, 4) X(64, 2) X(64, 4) X(96, 3) X(96, 6) X(128, 2) X(128, 4) X(192, 3) \
    X(192, 6) X(256, 4)
#define DETO_RAW_DECOMPRESS_PLAIN_LIST(X) X(32, 8) X(64, 8) X(128, 8) X(256, 8)      // (not AdamW)
int64_t launch_compress_raw(const CompressLaunch& a);
int64_t launch_decompress_raw_values(const DecompressLaunch& a);             // plain update
int64_t launch_decompress_raw_signs(const DecompressLaunch& a);
int64_t launch_decompress_raw_adamw(const DecompressLaunch& a);
int64_t launch_decompress_raw_signs_adamw(const DecompressLaunch& a);
int64_t launch_decompress_raw_amsgrad(const DecompressLaunch& a);
int64_t launch_decompress_raw_signs_amsgrad(const DecompressLaunch& a);
// ... tiles in gangs (decompress_gangs says which):
int64_t launch_decompress_split_gang(const DecompressLaunch& a, int classes);
int64_t launch_decompress_split_narrow_gang(const DecompressLaunch& a, int classes);
// 16-bit values, or byte indices:
int64_t launch_compress_split_narrow_96(const CompressLaunch& a);
int64_t launch_compress_split_narrow_128(const CompressLaunch& a);
int64_t launch_compress_split_narrow_192(const CompressLaunch& a);
int64_t launch_compress_split_narrow_256(const CompressLaunch& a);
// chunk 64 on a small shard only (see small_shard_tiles); tried before the lane-per-chunk kernel
int64_t launch_compress_split_64(const CompressLaunch& a);
int64_t launch_compress_split_96(const CompressLaunch& a);
int64_t launch_compress_split_128(const CompressLaunch& a);
int64_t launch_compress_split_192(const CompressLaunch& a);
int64_t launch_compress_split_256(const CompressLaunch& a);      // k > 32
int64_t launch_compress_halves_256(const CompressLaunch& a);     // k <= 32, any format but signs

// Direct sums on the matrix cores (direct_kernels.hip.h): what compress_generic would serve, bit for
// bit, at the chunk sizes of the list.  Takes all chunks or none.
#ifdef DETO_TILED_ONLY_64_32
#define DETO_DIRECT_COMPRESS_LIST(X) X(64)
#else
#define DETO_DIRECT_COMPRESS_LIST(X) X(16) X(32) X(64) X(96) X(128) X(160) X(192) X(224) X(256)
#endif
int64_t launch_compress_direct(const CompressLaunch& a);
inline bool direct_compress(const KParams& p) {
    if (p.scheme != 0 || (p.s != 16 && p.val_dtype != 3)) return false;
#define X(S) if (p.s == S) return true;
    DETO_DIRECT_COMPRESS_LIST(X)
#undef X
    return false;
}

// Few chunks stay on the general kernel, a wavefront each, up to about the round that fits the chip,
// at the chunk sizes where its direct sums are short.  us, general / matrix cores, signs: 16/3 1,000
// chunks 8.8 / 10.0, 4,000 9.4 / 9.9, 75,000 72 / 12; 64/8 1,000 9.8 / 11.5, 2,500 11.7 / 11.9, 4,000
// 13.9 / 11.8; 96/12 1,000 17.0 / 12.9; 256/64 7 chunks 70 / 27.
inline bool few_direct(const KParams& p, int64_t chunks) {
    return p.k < p.s && chunks <= (p.s <= 32 ? 4096 : p.s == 64 ? 2048 : 0);
}

// A lane-per-chunk decompress kernel for this request with transmitted indices (plain SGD update)?
inline bool lane_decompress(const KParams& p) {
    if (p.adam) return false;
    if (p.val_dtype == 0 && !p.idx_u8) {
#define X(K) if (p.k == K) return true;
        if (p.s == 16) { DETO_LANE_TOPK_16(X) }
        else if (p.s == 32) { DETO_LANE_TOPK_32(X) }
        else if (p.s == 64) { DETO_LANE_TOPK_64(X) }
        else if (p.s == 96) { DETO_LANE_TOPK_96(X) }
        else if (p.s == 128) { DETO_LANE_TOPK_128(X) }
#undef X
        return false;
    }
    if (!p.idx_u8 || p.val_dtype == 0) return false;
#define X(S, K) if (p.s == S && p.k == K) return true;
    if (p.val_dtype == 3) { DETO_LANE_SIGNS(X) }
    else { DETO_LANE_16BIT_32(X) DETO_LANE_16BIT_64(X) }
#undef X
    return false;
}

// Which decompress kernel serves transmitted indices: the number of coefficient classes
// (wavefronts per tile) of the wavefront-per-class kernels, or 0 for a lane per chunk (only if
// `lane`: there is one).
//
// A lane per chunk needs the fewest instructions but holds a whole chunk in registers: two
// wavefronts per SIMD up to chunk 64, one at 96 and 128, each with little in flight.  Two classes
// cost about a third more instructions at twice the wavefronts, four classes half more again
// at up to seven per SIMD.  So what decides is whether a shape is bound by memory latency (many
// bytes per element: AdamW's moments, fp32 parameters, fp32 + int32 payloads) or by
// instructions (few bytes, or many entries per byte: two-bit signs), and how many rounds of
// workgroups the launch is: one round of a lane per chunk is 1,024 tiles at one wavefront per SIMD
// and 2,048 at two.
//
// The lines were drawn through 7,290 timed shapes (chunk 32 ... 128, seven k each, three payload
// formats, both parameter types and optimizers, R = 2, 4, 16, 0.3 ... 147 M parameters, each call on
// other buffers): the choice costs 1.6 % over the best of the three on average, and 35 shapes run
// more than 5 % longer than on the kernels that served them before there were classes, none of
// them by more than 13 %.  us, a lane per chunk / two / four classes:
//   AdamW: four classes, except where a wavefront's share of a replica's payload (16 rows of k
//   entries) leaves its lanes idle and there are many replicas' to scatter.
//     64/16, signs, R = 4, 147 M bf16     - /523/509   32/4, signs, R = 16, 30 M bf16  - /136/158
//     64/32, fp16, R = 16, 1 M bf16       - / 32/ 21   32/4, fp16, R = 16, 4 M fp32    - / 29/ 32
//   Few tiles: four classes where there is no lane per chunk; a lane per chunk where its launch is
//   about one round or less.
//     64/21, fp32, R = 2, 1 M bf16        - / 12/  8   64/8, fp32, R = 2, 3 M fp32   7.9/9.5/9.1
//     128/16, fp32, R = 2, 8 M fp32    19.8/19.7/21.9  64/8, fp32, R = 2, 12 M fp32   26/ 24/ 24
//   Eight or more entries per element, R*k >= 8 s: the instructions of the scatter are what is left.
//     32/16, fp32, R = 16, 8 M fp32    101/106/105   30 M 380/399/388
//   Idle lanes without AdamW: 128/1, fp32, R = 16, 30 M bf16 51/51/58, 64/2, fp32, R = 16, 8 M fp32
//   23/21/26.
//   Large shards of bf16 parameters: from 2^25 elements on (with the line at 2^26 or 10^8 the
//   average loss of the shapes above 40 M goes from 0.5 % to 1.4 or 2.5 %).
//     64/32, fp32, 147 M, R = 4         512/510/504    30 M, R = 2  65/ 69/ 66
//     64/16, fp32, 147 M, R = 4         302/305/289    30 M, R = 2  44/ 50/ 49
inline int decompress_classes(const KParams& p, int64_t n, bool param_bf16, bool lane) {
    const int64_t rk = static_cast<int64_t>(p.R) * p.k;    // entries per chunk to scatter
    const int64_t tiles = n / (kWave * p.s);
    const bool plain = p.val_dtype == 0 && !p.idx_u8, quads = p.k % 4 == 0;
    const bool large = n > kLargeShard, few = tiles <= 1024;
    if (p.s == 192 || p.s == 256) return 4;
    if (p.s != 16 && p.s != 32 && p.s != 64 && p.s != 96 && p.s != 128) return 0;
    if (p.s == 16) return (lane && param_bf16) ? 0 : 2;
    if (p.adam) return (few || p.k >= 16 || (quads ? plain || rk <= p.s : 4 * rk <= p.s)) ? 4 : 2;
    if (lane && rk >= 8 * p.s) return 0;
    if (p.s >= 96) {
        if (lane && few && tiles > 640) return 0;
        if (!param_bf16) return 4;
        if (lane && p.s == 128 && p.k < 4 && !few) return 0;
        if (p.s == 128 && (rk >= p.s || !large)) return 4;
        return lane ? 0 : (large ? 2 : 4);
    }
    const bool wide = plain && p.k >= 8;    // (four classes, for SGD)
    if (!lane) return (few || p.k >= 16 || (wide && !param_bf16 && p.s == 64 && 2 * rk >= p.s)) ? 4 : 2;
    if (tiles <= 1536) return 0;
    if (!param_bf16) {
        const bool split = plain || rk <= (quads ? 16 : 8);
        return !split ? 0 : (wide && p.s == 64 && 2 * rk >= p.s) ? 4 : 2;
    }
    if (!large || !plain || !quads || p.R < 2) return 0;
    return rk >= p.s ? (wide ? 4 : 2) : (p.s == 64 && 2 * rk >= p.s) ? 2 : 0;
}

// The same for Striding and Random without transmitted indices.
inline bool lane_scheme(const KParams& p) {
    if (p.adam) return false;
#define X(S, K) if (p.s == S && p.k == K) return true;
    if (p.val_dtype == 0) { DETO_LANE_SCHEME(X) DETO_LANE_SCHEME_SMALL(X) }
    else { DETO_LANE_SCHEME_NARROW_32(X) DETO_LANE_SCHEME_NARROW_64(X) }
#undef X
    return false;
}

// The sums over the replicas are formed in registers, so large groups cost little; a shuffle costs
// one of the wavefronts k steps, which is what the high rates lose.  AdamW: four classes at every
// size (2,870 timed shapes of chunk 32 and 64, both domains, fp32 values and signs, else as above:
// 0.4 % over the better of two and four on average, 2 % and 7 % for the former rule and for two).
// Plain SGD: a lane per chunk where there is one, except for fp32 parameters at low rates on launches
// of more than a round and a half of it, 3,072 tiles (none of 2,870 shapes runs more than 5 % longer
// than on the kernels before there were classes; 8 with the line at 2,048, 39 at 1,024); twice that
// at chunk 16 (16/1, fp32, Random on coefficients: 4 M 8.1/9.7, 8 M 15.5/15.5).  us:
//   64/8, fp32, AdamW, two / four classes           147 M bf16, R = 4 532/523   30 M fp32, R = 2 145/134
//   64/8, fp32, R = 2, Random, a lane / two classes 1 M fp32 6.2/7.5   8 M 16.1/17.1   30 M 55/51
//   32/2, signs, R = 2, Random on coefficients      6 M fp32 10.8/13.7
//   64/32, fp32, R = 4, Random                      100 M bf16 210/207   147 M 305/307
//   16/2, fp32, R = 2, Random                       30 M bf16 29/45   fp32 51/49   16/1 50/44
inline int scheme_classes(const KParams& p, int64_t n, bool param_bf16, bool lane) {
    if (!lane) {
        const int c = decompress_classes(p, n, param_bf16, false);
        return (c && p.s != 16 && (p.adam || p.s >= 96)) ? 4 : c;
    }
    const bool low = 16 * p.k <= p.s ||
                     (8 * p.k <= p.s && (p.s == 64 || (p.s == 32 && p.val_dtype == 0)));
    return (!param_bf16 && low && n / (kWave * p.s) > (p.s == 16 ? 6144 : 3072)) ? 2 : 0;
}

// How many workgroups of a large launch share a CU (0: as many as fit).  Every tile in flight is a
// window of its own in every array, and from some 150 KB in flight per CU on more windows no longer
// hide latency but cost the memory its locality.  Where tiles are heavy and the kernel does not need
// the wavefronts for its arithmetic or its latencies, fewer are faster.  The lines come from timed
// shapes on rotating buffers (11 ... 147 M parameters compress, 36 ... 147 M decompress; both element
// types); in brackets the time at the chosen number over the time without a limit.
//   compress, a lane per chunk: chunk 32, top-k (k 1, 8, 16, fp32, fp16, signs) and coefficients 10
//   (0.95 - 0.99; fewer lose where signs leave the transform as the bound: 32/16 30 M bf16 8 1.03); chunk 16
//   10 (0.95 - 1.01; with one or two entries of bf16 gradients 11 M 1.01, 30 M 1.01 - 1.02, 45 M 0.99,
//   hence the second line).
constexpr int64_t kLimitedTiles = 10240;      // (40 tiles per CU)
inline int compress_workgroups(const KParams& p, int64_t tiles, bool grad_bf16) {
    if (tiles <= kLimitedTiles) return 0;
    if (p.s == 16 && p.k <= 2 && grad_bf16) return 0;     // (up to 2^25 elements: above, compress_gang_workgroups)
    // (signs, top-k, chunk 32, 7: 32/16 147 M bf16 277, 273; 32/4 28 M fp32 65.0, 64.0; fp32 gradients from 2^25
    // elements on 5: 32/16 333, 321, 32/4 60 M 134, 128)
    if (p.s == 32 && p.scheme == 0 && p.val_dtype == 3)
        return !grad_bf16 && tiles * (kWave * p.s) > kLargeShard ? 5 : 7;
    return p.s <= 32 ? 10 : 0;
}
// Tiles in gangs (run_log2), compress: from 2^20 elements on.  In gangs over in a row, geometric mean over random
// shapes on rotating buffers (largest): chunk 16 1 - 4 M 0.96 (1.01), from 8 M on 0.97; chunk 32 fp32 values 1 - 4 M
// 0.94 (1.00), from 8 M on 0.96; chunk 64 2 - 8 M 0.97 (1.02), from 8 M on 0.95; but below 1 M chunk 32 1.00 (1.02), chunk
// 64 with 16-bit values 1.02 (1.04).  Chunk 32 with 16-bit values 0.98, signs the same either way.
// (DETO_SMALL_SHARD_TILES = 0: no shard is small.)
constexpr int64_t kCompressGangs = int64_t{1} << 20;
inline int compress_run_log2(const KParams& p, int64_t n) {
    if (n <= kCompressGangs && small_shard_tiles() != 0) return 6;
    return run_log2(p.s, p.k, p.val_dtype, p.scheme != 0 ? 0 : p.idx_u8 ? 1 : 4, kRunBytes);
}
// Fewer of them are in flight at no loss.  us without a limit, or at the one above, and at the chosen one (147 M;
// 60 M):
//   chunk 32, from 2^25 elements on: fp32 values, bf16 gradients, k >= 8 5 (349, 327; 147, 139), fewer
//     entries 6 (279, 262; 118, 112), fp32 gradients 5 (399, 386; 166, 159); 16-bit values 7 and 5
//   chunk 16, from 2^25 on, 8 (291, 284; 121, 118)
//   chunk 64, top-k, from 2^26 on: fp32 gradients 5 (428, 416; 100 M 286, 279); bf16 with 32 fp32 entries 5
//     (358, 349; at 60 M 150, 154), 16-bit values 7 (301, 296), others none (64/16 60 M at 5 128, 136); Striding
//     and Random on coefficients, bf16, from 2^27 on, 6 (308, 303; 861 M 1,763, 1,719; 80 M 168, 169)
inline int compress_gang_workgroups(const KParams& p, int64_t tiles, bool grad_bf16) {
    const int64_t n = tiles * (kWave * p.s);
    if (p.s == 64) {
        if (n <= (int64_t{1} << 26)) return 0;
        if (p.scheme != 0) return grad_bf16 && n > (int64_t{1} << 27) ? 6 : 0;
        if (!grad_bf16) return 5;
        return p.k < 32 ? 0 : p.val_dtype == 0 ? 5 : 7;
    }
    if (n <= kLargeShard) return compress_workgroups(p, tiles, grad_bf16);
    if (p.s == 16) return 8;
    if (!grad_bf16) return 5;
    return p.val_dtype != 0 ? 7 : p.k >= 8 ? 5 : 6;
}
//   decompress (classes: wavefronts a workgroup; 0: a lane per chunk, one wavefront), fp32 values and
//   plain update, from 2^26 elements on but where a line says otherwise (narrow payloads are bound by
//   the scatter).  With indices what has to be in flight is k entries a replica and chunk, in groups of
//   four: the fewer there are the more workgroups it takes, and entries one by one take all there are
//   (147 M, bf16, at 3 or 4 a CU: 64/2 R = 64 2.08, 64/4 R = 32 1.59, 64/8 R = 16 1.12, 64/30 R = 4 1.22,
//   32/4 R = 16 1.40, 32/15 R = 4 1.62).
//     chunk 128, k >= 16, R*k >= s/2 with fp32 parameters, s with bf16: 3 (0.92 - 0.98; 36 M 1.01 - 1.05;
//       R*k = s/4 1.03)
//     chunk 96, fp32 parameters, R*k >= s/2: 4, from 2^25 on (0.97 - 1.00)
//     chunk 64, R*k >= s: k >= 16 4 (0.98 - 1.01), from 2s on 3 (0.94 - 1.01); 8 and 12 on four classes 4
//       (0.96 - 1.01); 4 6 (fp32 0.96 - 0.98, bf16 from 2s on 0.97 - 0.99)
//     chunk 32, R*k >= s: k >= 16 5 (0.93 - 0.99), but 16 fp32 R = 2 and 20 bf16 R = 2 6 (0.95 - 1.00; at 5
//       1.00 and 1.08), from 2s on 4, also from 2^25 on (0.92 - 0.99); 8 and 12 5 (fp32 0.94 - 1.01, from
//       2s on 4; bf16 0.95 - 0.97 from 2s on, 1.03 - 1.08 below); 4, fp32, 6, from 2^25 on (0.92 - 1.00)
//     chunk 32, bf16 parameters, two classes (4 and 12 entries), R*k >= 3s/4, 12 below 2s: 8 (0.95 - 0.97)
//   Without indices (a lane per chunk), R*k >= 2s and k >= 4 (at these numbers 32/2 R = 64 1.24, 32/1
//   R = 64 1.34, 64/2 R = 64 1.13):
//     chunk 64 5 (0.94 - 1.02), not 32 from 4s on (1.02 at 70 M) nor 4 with the transform (1.02)
//     chunk 32 6, from 4s on 4, k = 4 5 (0.91 - 1.00)
//   AdamW, four classes, R*k <= s: the batches of parameters and moments are in flight.
//     chunk 96: narrow or raw 4 from 2^23 on (0.98 - 1.00), the rest with bf16 parameters from 2^25 on
//       (0.98 - 0.99; 20 M 1.04)
//     chunk 64, bf16 parameters: narrow payloads, with indices or raw, 4 from 2^23 on (0.96 - 0.99), fp32
//       values of the transform domain from 2^25 on (0.97 - 0.99); the others, and R*k = 4s, lose up to 1.07
//     Random and Striding at chunk 32, fp32 values, bf16 parameters: 5 from 2^25 on (0.96 - 0.99)
//     chunk 32, narrow payloads of at most four replicas (more of them up to 1.30): with indices 5, fp32
//       parameters from 2^23 on (0.96 - 1.01), bf16 from 2^26 on (0.96 - 1.00), but not 4 and 8 entries of four
//       replicas (1.00 - 1.03); Random and Striding with fp32 parameters from 2^24 on 5 (0.95 - 1.00), signs
//       of the transform domain 6 (0.96 - 1.00; at 5 1.06)
inline int adamw_workgroups(const KParams& p, int64_t n, bool idx, bool param_bf16, int classes) {
    const int64_t rk = static_cast<int64_t>(p.R) * p.k;
    const bool plain = p.val_dtype == 0 && !(idx && p.idx_u8);
    // (amsgrad's kernels, with larger batches, gain nothing)
    if (p.amsgrad || classes != 4 || n <= (int64_t{1} << 23)) return 0;
    const bool large = n > kLargeShard;
    if (p.s == 32 && p.R <= 4 && !plain) {
        if (idx && !param_bf16) return 5;
        if (idx) return n > (int64_t{1} << 26) && (p.R < 4 || p.k >= 16 || p.k % 4 != 0) ? 5 : 0;
        if (!param_bf16) return n > (int64_t{1} << 24) ? (p.val_dtype == 3 ? 6 : 5) : 0;
    }
    if (rk > p.s) return 0;
    if (p.s == 96) return (idx && !plain) || (large && param_bf16) ? 4 : 0;
    if (!param_bf16) return 0;
    if (p.s == 64) return (plain ? !idx && large : idx) ? 4 : 0;
    return p.s == 32 && !idx && plain && large ? 5 : 0;
}
inline int decompress_workgroups(const KParams& p, int64_t n, bool idx, bool param_bf16, int classes) {
    if (p.adam) return adamw_workgroups(p, n, idx, param_bf16, classes);
    const int64_t rk = static_cast<int64_t>(p.R) * p.k;
    const bool large = n > (int64_t{1} << 26);
    if (p.val_dtype != 0 || p.idx_u8 || rk >= 8 * p.s || idx != (classes != 0)) return 0;
    if (idx && p.k % 4 == 0) {
        if (p.s == 128)
            return large && classes == 4 && p.k >= 16 && (param_bf16 ? rk : 2 * rk) >= p.s ? 3 : 0;
        if (p.s == 96) return n > kLargeShard && !param_bf16 && 2 * rk >= p.s ? 4 : 0;
        if (p.s == 32 && param_bf16 && classes == 2 && 4 * rk >= 3 * p.s && (p.k < 8 || rk < 2 * p.s))
            return large ? 8 : 0;
    }
    if ((p.s != 32 && p.s != 64) || rk < p.s) return 0;
    const bool twice = rk >= 2 * p.s;
    if (idx) {
        if (p.k % 4 != 0) return 0;
        if (p.s == 32 && p.k >= 16 && twice) return n > kLargeShard ? 4 : 0;
        if (p.s == 32 && p.k == 4) return n > kLargeShard ? 6 : 0;
        if (!large) return 0;
        if (p.s == 64) {
            if (p.k >= 8) return classes == 4 ? 4 : 0;
            return (twice || !param_bf16) ? 6 : 0;
        }
        if (p.k >= 16) return (p.k == 16) == param_bf16 || 2 * rk >= 3 * p.s ? 5 : 6;
        return !param_bf16 ? (twice ? 4 : 5) : (twice ? 5 : 0);
    }
    if (!large || !twice || p.k < 4) return 0;
    if (p.s == 64) return (p.k == 32 && rk >= 4 * p.s) || (p.k == 4 && p.use_dct) ? 0 : 5;
    return rk < 4 * p.s ? 6 : p.k == 4 ? 5 : 4;
}
// Tiles in gangs (run_log2), transmitted indices, k a multiple of four: where windows that move side by side pay for
// the addresses and for shorter runs of the payload.  In gangs over in a row, geometric mean (largest) over some 1,300
// random shapes on rotating buffers, 8 - 160 M parameters:
//   AdamW, fp32 values, a quarter of the chunk kept or more 0.97 (1.03), or up to two replicas 0.96 (1.00); less of more
//     replicas 1.05 (1.16)
//   AdamW, 16-bit values or byte indices, chunk 64 and 128, the same and R*k <= s 0.97 (1.02); R*k > s 1.00 (1.08), chunk
//     32 1.00, signs 1.00
//   plain update, fp32 values, a quarter or more: fp32 parameters and R*k <= s/4 0.98 (1.01); chunk 32 R*k > 2s 0.97
//     (1.01), below 1.02 (1.21); chunk 64 R*k >= s 0.97 (1.04), below 1.01 (1.06) but for fp32 parameters and one replica
//     0.97 (1.01) or R*k <= s/2 up to 2^24 0.97 (1.02; above 1.03); chunk 128 from 2^25 elements on, fp32
//     parameters 0.98 (1.02), bf16 R*k > s 0.98 (1.02), below 1.00 (1.05)
constexpr int64_t kGangShard = int64_t{1} << 23;
inline bool decompress_gangs(const KParams& p, int64_t n, bool param_bf16, int classes) {
    if (p.run_lg >= 6 || classes == 0 || p.k % 4 != 0 || (p.s != 32 && p.s != 64 && p.s != 128)) return false;
    const int64_t rk = static_cast<int64_t>(p.R) * p.k;
    const bool plain = p.val_dtype == 0 && !p.idx_u8, quarter = 4 * p.k >= p.s;
    if (p.adam) {
        if (p.amsgrad || !(quarter || p.R <= 2)) return false;
        return plain || (p.s != 32 && p.val_dtype != 3 && rk <= p.s);
    }
    if (!plain || !quarter) return false;
    if (p.s == 128 && (n <= kLargeShard || (param_bf16 && rk <= p.s))) return false;
    if (!param_bf16 && (4 * rk <= p.s || (p.s == 64 && (p.R == 1 || (2 * rk <= p.s && n <= (int64_t{1} << 24))))))
        return true;
    return p.s == 128 || rk > (p.s == 32 ? 2 * p.s : p.s - 1);
}
// this call's run_log2; without indices (Striding and Random on coefficients, a lane per chunk, bf16 parameters; the
// same 900 M down to 12 M): half the chunk kept 0.96 (1.03), a quarter R*k >= 4s 0.97 (1.01), below 1.00 (1.06)
inline int decompress_run_log2(const KParams& p, int64_t n, bool idx, bool param_bf16) {
    if (n <= kGangShard) return 6;
    if (idx)
        return run_log2(p.s, p.k, p.val_dtype, p.idx_u8 ? 1 : 4, decompress_run_bytes(p.s, p.k, p.R, p.adam));
    if (!scheme_gangs(p.s, p.k) || p.val_dtype != 0 || !param_bf16 || n <= (int64_t{1} << 24)) return 6;
    if (2 * p.k != p.s && p.R * p.k < 4 * p.s) return 6;
    return run_log2(p.s, p.k, 0, 0, kSchemeRunBytes);
}
// Workgroups per CU of those, us without a limit and at the chosen one (147 M; 60 M):
//   plain update, from 2^25 elements on: chunk 128, R*k > s 3 (bf16 488, 480; 205, 203); chunk 64, R*k >= 2s 3 (471, 449;
//     198, 190; fp32 565, 538), from s on 4 (276, 271; 117, 112); chunk 32 4 (fp32 and bf16, random shapes 0.96)
//   AdamW: chunk 64, fp32 values, from 2^24 on 3 (bf16 859, 838; 350, 341; fp32 969, 936), narrow ones 4
//     bf16, 3 fp32 (643, 628); from 2^25 on chunk 128, R*k <= s, 3 (586, 577), chunk 32, fp32 parameters, 5 (653, 645)
inline int decompress_gang_workgroups(const KParams& p, int64_t n, bool param_bf16) {
    const int64_t rk = static_cast<int64_t>(p.R) * p.k;
    if (p.adam && p.s == 64) {
        if (p.val_dtype != 0 || p.idx_u8) return param_bf16 ? 4 : 3;
        return n > (int64_t{1} << 24) ? 3 : 0;
    }
    if (n <= kLargeShard) return 0;
    if (p.adam) {
        if (p.s == 128) return rk <= p.s ? 3 : 0;
        return param_bf16 ? 0 : 5;
    }
    if (p.s == 128) return rk > p.s ? 3 : 0;
    if (p.s == 64) return rk >= 2 * p.s ? 3 : rk >= p.s ? 4 : 0;
    return rk > 2 * p.s ? 4 : 0;
}
// Dynamic LDS for that: half way between what lets one workgroup more and one less onto a CU.
// static_bytes: a tile's rows, (s + 4) floats a chunk (and, where the classes list the places
// themselves, those; or, compress at small chunks, the working set of the general code for the tail,
// 10 KB).
inline unsigned spare_lds(int workgroups, int static_bytes) {
    if (workgroups == 0) return 0;
    const int total = 2 * 160 * 1024 / (2 * workgroups + 1);
    return total > static_bytes ? static_cast<unsigned>(total - static_bytes) : 0u;
}
inline int launch_workgroups(const CompressLaunch& a) {
    return a.p.run_lg < 6 ? compress_gang_workgroups(a.p, a.tiles, a.grad_bf16)
                          : compress_workgroups(a.p, a.tiles, a.grad_bf16);
}
inline int launch_workgroups(const DecompressLaunch& a, int classes) {
    return a.idx && decompress_gangs(a.p, a.n, a.param_bf16, classes)
               ? decompress_gang_workgroups(a.p, a.n, a.param_bf16)
               : decompress_workgroups(a.p, a.n, a.idx != nullptr, a.param_bf16, classes);
}
inline unsigned spare_lds(const CompressLaunch& a) {
    const int rows = 4 * kWave * (a.p.s + 4);
    return spare_lds(launch_workgroups(a), rows > 10240 ? rows : 10240);
}
inline unsigned spare_lds(const DecompressLaunch& a, int classes = 0) {
    const int s = a.p.s;
    const int places = (!a.idx && classes) ? kWave * s / 2 + 8 * (s < 32 ? 32 : s) : 0;
    return spare_lds(launch_workgroups(a, classes), 4 * kWave * (s + 4) + places);
}

// Few chunks: a launch of the wavefront-per-class kernels is then a handful of workgroups whose own
// duration counts, while the general kernels spread the same chunks over the whole chip, a wavefront
// each.  Those are 8 - 10 KB of LDS a workgroup, 16 - 20 per CU: some 5,000 chunks are one occupancy
// round.  So they serve less than a tile (20 chunks of 64, k 21, R = 16, signs: 10 against 28 us;
// 20 of 256, Random, k 128, R = 2: 16 against 30), and up to about half a round two-bit signs of
// many replicas under top-k, whose scatter the few wavefronts would do one step after the other.  us, general /
// wavefront per class, 0.3 M parameters, R = 16: 128/42 30 / 53, 256/85 50 / 102, 96/32 28 / 25; 1 M 128/42 77 / 59.
inline bool few_chunks(int64_t chunks) { return chunks < kWave; }     // compress (Striding, Random)
inline bool few_chunks_decompress(const KParams& p, int64_t chunks, bool idx) {
    return chunks < kWave ||
           (idx && p.val_dtype == 3 && chunks <= 2560 && static_cast<int64_t>(p.R) * p.k >= 4 * p.s);
}

// Two-bit signs on coefficients without indices: counted a word at a time (SignCounts), or decoded and added one by
// one?  Counting costs the same for 16 and for 33 replicas and for every k up to 16, and where a wavefront has 16
// chunks' words, most of its lanes idle.  Decompress, us, one by one / counted: 60 M bf16 32/16 R = 64 311 / 153, 64/21
// R = 20 260 / 167, 64/5 R = 33 150 / 87, fp32 64/32 R = 64 AdamW 417 / 322; but 5 M bf16 128/16 R = 20 16.0 / 18.4,
// 0.6 M fp32 64/2 R = 16 6.3 / 7.1, and few entries of 32 replicas 2.1 M fp32 16/1 11.6 / 12.4, bf16 96/3 14.6 / 15.5.
// Over 300 random shapes 0.76 of the time of one by one.
inline bool count_signs(const KParams& p) {
    return p.val_dtype == 3 && (p.k > 16 ? p.R >= 16 : p.R >= (p.k >= 4 ? 32 : 48));
}

// ---- Striding and Random on the momentum itself (raw_kernels.hip.h).  Against the kernels before them (general
// ones, a lane per chunk, classes, the stream), geometric mean over 500 random shapes each of 0.07 - 40 M elements, chunk
// 16 ... 256, formats, optimizers and 1 - 64 replicas: compress 0.73 of their time, decompress of values 0.60, of signs
// 0.61.
// Pieces of four elements a thread: few while a launch's own latency counts (1.5 M, 128/4 compress, 2 / 4 / 8
// pieces 5.0 / 5.8 / 6.7 us; AdamW 64/8 2.6 M 9.4 / 11.4 / 14.9), more where a replica's entries of a workgroup
// would be a short run (128/16, 49 replicas, signs, 18 M 43.5 / 36.1 / 36.4; 256/64 bf16 60 M, 4 replicas 174 /
// 106 / 81; signs of few replicas 128/8 R = 2 bf16 74 M 51 us in the class kernels, 59 / 54) and for compress where the
// shuffle is long (128/32 7 M 19.6 / 18.9; 256/64 60 M 144 / 127 / 129).
// Workgroups per CU of large launches, without a limit / with it (147 M): compress 128/16 fp32 328 / 4 313, bf16
// 278 / 5 263, 32/1 signs bf16 265 / 252; decompress, fp32 parameters, 128/16 206 / 5 204; AdamW, 2 pieces, 60 M
// 64/8 bf16 205 / 3 198, fp32 258 / 251.
constexpr int64_t kRawLimited = int64_t{1} << 24;
inline int raw_compress_quads(const KParams& p) {
    if (p.s == 96 || p.s == 192) return 3;
    return p.s == 256 || (p.s == 128 && p.k >= 32 && p.scheme == 2) ? 4 : 2;
}
// Everything but Random's long shuffles on a few chunks, a chain per chunk here and a wavefront per chunk in the general
// kernels (more than a quarter of 96 and more: 128/64 fp16 0.05 M 9.3 us there, 10.5 here, geometric mean up to 2^16
// elements 1.07, above 0.9).
inline bool raw_compress(const KParams& p, int64_t n) {
    return !(p.scheme == 2 && p.s >= 96 && 4 * p.k > p.s && n <= (int64_t{1} << 16));
}
// Workgroups per CU of large launches.  A workgroup whose shuffle is long for the elements it moves spends its time there,
// and memory idles below a round of them: as many as fit up to 52 elements a step (us with the limit / without: 192/96
// fp16 fp32 46 M 180 / 115, bf16 57 M 188 / 139; 256/128 bf16 78 M 254 / 186; 192/64 66 M 174 / 131), up to 80 for the
// signs of bf16 gradients (64/32 37 M 90 / 72, 128/64 58 M 132 / 107) and 6 of fp32 ones (64/32 28 M 80 / 66), and one
// more for values but where much is in flight already (16-bit ones 64/32 bf16 66 M 138 / 126, fp32 31 M 81 / 73; but
// 128/64 bf16 71 M 145 / 152, 96/48 fp32 values 40 M 100 / 107).
inline int raw_compress_workgroups(const KParams& p, int64_t n, bool grad_bf16) {
    if (n <= kRawLimited) return 0;
    const int elements = 1024 * raw_compress_quads(p);
    if (p.scheme == 2 && elements <= 52 * p.k) return 0;
    if (p.scheme == 2 && elements <= 80 * p.k) {
        if (p.val_dtype == 3) return grad_bf16 ? 0 : 6;
        if (p.s <= 64 || p.s >= 192) return grad_bf16 ? (p.val_dtype != 0 ? 6 : 5) : 5;
    }
    return grad_bf16 ? 5 : 4;
}
// (AdamW: more also where the shuffle is long, 128/64 R = 4 65 M bf16 389 / 296, and where 16 replicas and more would
// be runs of 256 bytes or less: 64/4 R = 46 signs 32 M 167 / 154, 32/2 R = 58 59 M 346 / 323)
inline int raw_decompress_quads(const KParams& p, int64_t n) {
    const bool few = p.adam ? n <= (int64_t{1} << 26) : n <= (int64_t{1} << (p.R < 16 ? 22 : 20));
    const bool many = !p.adam && n > (int64_t{1} << 23) && (p.R * p.k >= p.s || (p.val_dtype == 3 && p.s <= 128));
    if (p.s == 96) return few ? 3 : 6;
    if (p.s == 192) return few && n <= (int64_t{1} << 23) ? 3 : 6;
    if (p.s == 256) return p.adam || few || p.R * p.k < p.s ? 4 : 8;
    if (p.adam && n > (int64_t{1} << 23)) {
        const int run = 2048 / p.s * (p.val_dtype == 3 ? 4 * ((p.k + 15) / 16) : p.k * (p.val_dtype == 0 ? 4 : 2));
        if ((p.s == 128 && p.k >= 32 && p.scheme == 2) || (p.R >= 16 && run <= 256)) return 4;
    }
    return few ? 2 : many && p.s != 16 ? 8 : 4;
}
// Nearly everything.  A lane per chunk does for bf16 parameters under the plain update what is left to do, on
// launches of a few wavefronts and on large ones (narrow values 32/1 139 M 93 us, 127 here; 32/16 17 M 23.7, 26.0;
// 64/32, 4 replicas, 147 M 287, 294, but 64/8 30 M 35, 32; 0.06 M 3.2, 3.7), but for two-bit signs of more entries
// than the chunk has (147 M 32/16 R = 16 252 / 194; 64/32 R = 64 1,040 / 315; 32/2 R = 64 339 / 303; 32/1 R = 40
// 245 / 220, R = 16 154 / 162) or, up to 2^23, more than a quarter of that (32/4 R = 1 fp32 2.9 M 5.7 / 7.5, 32/2 R
// = 3 5 M 9.2 / 11.1; in the mean over random shapes 0.6 above that line, 1.0 below).  Half of a chunk of 32 is one
// full word a lane: large launches from three times the chunk on (R = 4 25 M 23.4 / 27.9, Random 85 M 81 / 100, R =
// 8 48 M 51 / 47).  The class kernels that served the rest of the large launches, over 700 random shapes of 8 - 100
// M parameters: 0.72 of their time here; entries one by one 0.33 - 0.98 (16/6 R = 6 fp16 18 M 66 / 49, 96/13 R = 12
// fp32 8.5 M 70 / 26), two-bit signs 0.2 - 1.0.
inline bool raw_decompress(const KParams& p, int64_t n, bool param_bf16) {
    const bool lane = lane_scheme(p);
    if (n <= (int64_t{1} << 17)) return !lane;
    if (lane && p.val_dtype == 3 && n <= (int64_t{1} << 23)) return 4 * p.R * p.k > p.s;
    if (n <= (int64_t{1} << 23) || !(lane && param_bf16)) return true;
    if (p.val_dtype == 3) return p.R * p.k > (p.s == 32 && p.k == 16 ? 3 * p.s : p.s);
    return p.val_dtype == 0 && p.s > 32 && n <= (int64_t{1} << 26);
}
// AdamW, 3 up to 2^26: fp32 values, and with fp32 parameters every format (signs 32/16 R = 4 65 M 270 / 253, 64/32 R = 2
// 39 M 165 / 156); but not where the shuffle is long for the workgroup's elements (signs 256/128 R = 4 34 M 162 / 201 with
// the limit; fp32 values and bf16 parameters 256/128 60 M 278 / 355, 64/21 53 M 179 / 190, 96/48 42 M 153 / 165; but chunk
// 128, 64 entries, R = 4 58 M 283 / 272).
inline int raw_decompress_workgroups(const KParams& p, int64_t n, bool param_bf16) {
    if (n <= kLargeShard) return 0;
    if (!p.adam) return param_bf16 ? 0 : 5;
    if (n > (int64_t{1} << 26) || (p.val_dtype != 0 && param_bf16)) return 0;
    const int elements = 1024 * raw_decompress_quads(p, n);
    return p.scheme == 2 && p.s != 128 && elements <= (param_bf16 ? 100 : 52) * p.k ? 0 : 3;
}
// dynamic LDS of a launch that takes `bytes` and is to have that many workgroups per CU
inline unsigned raw_lds(int bytes, int workgroups) {
    const int want = workgroups == 0 ? 0 : 2 * 160 * 1024 / (2 * workgroups + 1);
    return static_cast<unsigned>(want > bytes ? want : bytes);
}

inline int64_t launch_decompress_raw(const DecompressLaunch& a) {
    const KParams& p = a.p;
    if (a.idx || p.scheme == 0 || p.use_dct || 2 * p.k > p.s || !raw_decompress(p, a.n, a.param_bf16)) return 0;
    const bool signs = p.val_dtype == 3;
    if (!p.adam) return signs ? launch_decompress_raw_signs(a) : launch_decompress_raw_values(a);
    if (!p.amsgrad) return signs ? launch_decompress_raw_signs_adamw(a) : launch_decompress_raw_adamw(a);
    return signs ? launch_decompress_raw_signs_amsgrad(a) : launch_decompress_raw_amsgrad(a);
}

inline int64_t launch_compress_split(const CompressLaunch& a) {
    int64_t c = launch_compress_halves_256(a);
    if (!c) c = launch_compress_split_96(a);
    if (!c) c = launch_compress_split_128(a);
    if (!c) c = launch_compress_split_192(a);
    if (!c) c = launch_compress_split_256(a);
    if (!c) c = launch_compress_split_narrow_96(a);
    if (!c) c = launch_compress_split_narrow_128(a);
    if (!c) c = launch_compress_split_narrow_192(a);
    return c ? c : launch_compress_split_narrow_256(a);
}

}  // namespace deto
