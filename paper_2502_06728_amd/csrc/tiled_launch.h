// Host-side launchers of the tiled kernels.  Each translation unit tiled_*.hip instantiates
// one family of kernels and defines its launcher, so the families compile in parallel.
// A launcher returns true if it has a kernel for (p.s, p.k) and has enqueued it.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

#include "deto_device.hip.h"

namespace deto {

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
// (chunk 64: two coefficient classes instead of a lane per chunk; chunk 128: four instead of
// two).  Measured on MI355X: 4 - 13 % shorter launches at 1,300 - 8,000 tiles, 4 - 5 % longer
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
// NB = chunk size / 32.  What nothing else takes: compress at 160, 224, and at 32, 64 with
// k > s/2; decompress at 160, 224.
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
int64_t launch_compress_split_256(const CompressLaunch& a);

// Which decompress kernel serves transmitted indices: the number of coefficient classes
// (wavefronts per tile) of the wavefront-per-class kernels, or 0 for a lane per chunk; `lane`:
// the latter may be chosen (it is instantiated for some (s, k, format) only, without AdamW).
//
// A lane per chunk needs the fewest instructions but holds a whole chunk in registers: two
// wavefronts per SIMD at chunk 64, one at 96 and 128, each with little in flight.  Two classes
// cost about a third more instructions at twice the wavefronts, four classes half more again
// at up to seven per SIMD.  So what decides is whether a shape is bound by memory latency (many
// bytes per element: AdamW's moments, fp32 parameters, fp32 + int32 payloads) or by
// instructions (few bytes, or many entries per byte: two-bit signs).  Measured on MI355X, us,
// buffers rotating, a lane per chunk / two / four classes; A: 147 M bf16 parameters, R = 4;
// B: 28 M and C: 11 M fp32 parameters, R = 2; D: 28 M bf16 parameters, R = 2:
//   chunk 64, k 32, fp32 + int32, SGD   A 521/513/510  B  79/ 75/ 73  C 34/33/32  D 59/64/58
//             k 16                      A 300/296/282  B  60/ 57/ 56  C 26/26/25  D 40/46/43
//             k 8                       A 194/187/223  B  52/ 49/ 49  C 23/23/23  D 30/35/41
//             k 4                       A 141/159/208  B  49/ 46/ 47  C 22/22/22  D 26/34/40
//             k 16, fp16 + byte         A 169/200/224  B  52/ 49/ 50  C 22/24/24  D 29/41/42
//             k 16, signs, AdamW        A 601/552/515  B 145/129/123  C 61/54/51  D  - /108/100
//   chunk 32, k 16, fp32 + int32, SGD   A 508/498/494  B  75/ 72/ 73  C 33/31/30  D 57/57/56
//             k 4, signs, SGD           A 113/194/259  B  47/ 43/ 51  C 21/20/24
//             k 16, signs, AdamW        A 625/544/535  B 141/122/120  C 60/52/50  D  - /102/ 99
//   chunk 128, k 16, fp32 + int32, SGD  A 205/209/214  B  57/ 55/ 52  C 29/30/26  D 44/44/42
//             k 64, fp16 + byte         A  - /373/328  B  - / 79/ 69  C  - /42/33  D  - /67/60
// Two classes also stay ahead of four where there are many entries per chunk to scatter with
// little else to move (AdamW, chunk 32, k 4, signs, R = 16: 142 against 152 us).
constexpr int64_t kLargeShard = int64_t{1} << 25;   // elements: D's order turns between D and A
inline int decompress_classes(const KParams& p, int64_t n, bool param_bf16, bool lane) {
    const int64_t rk = static_cast<int64_t>(p.R) * p.k;    // entries per chunk to scatter
    const bool plain = p.val_dtype == 0 && !p.idx_u8, quads = p.k % 4 == 0;
    const bool large = n > kLargeShard;
    if (p.s == 192 || p.s == 256) return 4;
    if (p.s != 16 && p.s != 32 && p.s != 64 && p.s != 96 && p.s != 128) return 0;
    if (p.s == 16) return (lane && !p.adam && param_bf16) ? 0 : 2;
    if (p.adam) return (quads ? (plain || rk <= p.s) : 4 * rk <= p.s) ? 4 : 2;
    if (p.s >= 96) {
        // (many entries per chunk to scatter: chunk 96, k 24, R = 22: 51 against 53 us a step)
        if (lane && plain && rk >= 4 * p.s) return 0;
        if (!param_bf16) return 4;
        if (p.s == 128 && (rk >= p.s || !large)) return 4;
        return lane ? 0 : (large ? 2 : 4);
    }
    bool split = false, wide = false;
    if (!param_bf16) {
        split = plain ? !(p.k == 1 && 2 * rk >= p.s) : rk <= (quads ? 16 : 8);
        wide = p.s == 64 && plain && 2 * rk >= p.s;
    } else if (large && plain && quads && p.R >= 2) {
        wide = rk >= p.s;
        split = wide || (p.s == 64 && 2 * rk >= p.s);
    }
    if (split) return wide ? 4 : 2;
    return lane ? 0 : 2;
}

// The same for Striding and Random without transmitted indices (0: a lane per chunk).  The sums
// over the replicas are formed in registers, so large groups cost little; a shuffle costs one of
// the wavefronts k steps, which is what the high rates lose.  us, a lane per chunk / two / four
// classes, the shards A, B, D of decompress_classes:
//   chunk 64, k 32, signs, AdamW, Random   A 597/525/540  B 147/132/121  D 123/111/113
//             k 8, fp32, AdamW             A 628/579/557  B 147/130/122  D 121/110/104
//             k 8, fp32, SGD               A 143/138/201  B  51/ 47/ 47  D  29/ 30/ 41
//             k 32, fp32, SGD              A 307/288/364  B  64/ 66/ 78  D  43/ 54/ 71
//   chunk 32, k 4, signs, coefficients     A 114/209/290  B  46/ 48/ 62  D  26/ 43/ 59
//             k 1, signs                   A  99/135/168  B  45/ 40/ 42  D  23/ 30/ 35
inline int scheme_classes(const KParams& p, int64_t n, bool param_bf16, bool lane) {
    const bool plain = p.val_dtype == 0;
    const int64_t rk = static_cast<int64_t>(p.R) * p.k;
    if (p.adam || !lane || (p.s != 32 && p.s != 64)) {
        const int c = decompress_classes(p, n, param_bf16, false);
        return (p.s >= 96 && c) ? 4 : c;
    }
    if (!param_bf16) return (16 * p.k <= p.s || (8 * p.k <= p.s && (p.s == 64 || plain))) ? 2 : 0;
    // (Random on coefficients stays with a lane per chunk: 861 M, chunk 64: 3,666 against 3,709 us
    // a step)
    const bool large = n > kLargeShard && !(p.use_dct && p.scheme == 2);
    return (large && plain && rk >= 2 * p.s) ? 2 : 0;
}

// Striding in the raw domain, fp32 values, no transmitted indices: the streaming kernel before the
// wavefront-per-class kernels?  Not for AdamW at chunk sizes up to 64: those have the sums over the
// replicas in registers, four values a load, where the stream gathers them element by element.
// us, stream / wavefront per class: 64/8, bf16 parameters, R = 2 1 M 14.6 / 7.8, 30 M 144 / 110,
// R = 16 361 / 142; fp32 R = 2 30 M 137 / 133.  At larger chunks the stream is ahead with fp32
// parameters and few replicas: 128/4 R = 2 30 M 130 / 141, 256/32 1 M 12.8 / 15.5.
inline bool stream_before_classes(const KParams& p) { return !(p.adam && p.s <= 64); }

// Few chunks: a launch of the wavefront-per-class kernels is then a handful of workgroups whose own
// duration counts, while the general kernels spread the same chunks over the whole chip, a wavefront
// each.  Those are 8 - 10 KB of LDS a workgroup, 16 - 20 per CU: some 5,000 chunks are one occupancy
// round.  So they serve less than a tile (20 chunks of 64, k 21, R = 16, signs: 10 against 28 us;
// 20 of 256, Random, k 128, R = 2: 16 against 30), and up to about a round what gives them little
// to do per chunk: no transform (Striding and Random on the momentum itself), and two-bit signs of
// many replicas, whose scatter the few wavefronts would do one step after the other.  us, general / wavefront per class, 0.3 M parameters (1,172 chunks of 256 ... 4,688 of 64),
// signs: compress Striding 64/2 7 / 8, 96/48 6 / 10, 128/64 6 / 12, 256/128 7 / 18, Random 128/16
// 8 / 10, 128/64 15 / 15, 256/128 22 / 26; decompress Random 128/16 R = 2 9 / 10, 256/128 23 / 32,
// 256/8 R = 16 14 / 11; AdamW 128/64 R = 2 18 / 21, R = 16 33 / 24; top-k R = 16 128/42 30 / 53,
// 256/85 50 / 102, 96/32 28 / 25.  1 M: compress 128/16 12 / 10, 256/32 10 / 14; AdamW 128/16
// 17 / 11, 256/32 R = 2 14 / 16; top-k R = 16 128/42 77 / 59.
inline bool few_chunks(const KParams& p, int64_t chunks) {   // compress (Striding, Random)
    if (chunks < kWave) return true;
    // (a shuffle of more than a quarter of the chunk is a long serial chain in the general kernel)
    return !p.use_dct && chunks <= ((p.scheme == 2 && 4 * p.k > p.s) ? 2048 : 5120);
}
inline bool few_chunks_decompress(const KParams& p, int64_t chunks, bool idx) {
    if (chunks < kWave) return true;
    if (idx)
        return p.val_dtype == 3 && chunks <= 2560 && static_cast<int64_t>(p.R) * p.k >= 4 * p.s;
    return !p.use_dct && p.s >= 96 && p.R < 8 && chunks <= (p.adam ? 4096 : 2560);
}

inline int64_t launch_compress_split(const CompressLaunch& a) {
    int64_t c = launch_compress_split_96(a);
    if (!c) c = launch_compress_split_128(a);
    if (!c) c = launch_compress_split_192(a);
    if (!c) c = launch_compress_split_256(a);
    if (!c) c = launch_compress_split_narrow_96(a);
    if (!c) c = launch_compress_split_narrow_128(a);
    if (!c) c = launch_compress_split_narrow_192(a);
    return c ? c : launch_compress_split_narrow_256(a);
}

}  // namespace deto
