// Striding and Random on the momentum itself (no transform), without transmitted indices: kernels that
// stream.
//
// Nothing here needs a whole chunk in one lane: a kept element's place in the payload is the number of
// kept elements before it, so a thread that holds four consecutive elements needs its chunk's kept
// set as a bit mask and the count of bits before its word, and nothing else.  So a workgroup of four
// wavefronts holds a run of whole chunks in registers, 16 bytes a thread and access, coalesced, and
// only the k kept entries of a chunk pass through LDS.
//
// What bounds it: memory.  Random's shuffle is a serial chain per chunk, k steps of an LDS round trip
// each, one lane a chunk; it runs while the workgroup's loads are in flight.
#pragma once

#include "deto_device.hip.h"
#include "generic_kernels.hip.h"
#include "split_kernels.hip.h"

namespace deto {

constexpr int kRawThreads = 256;
constexpr int64_t kRawSmall = int64_t{1} << 23;     // elements of a shard whose launch is mostly latency

// QUADS: pieces of four elements a thread holds
template <int S, int QUADS>
struct RawGeom {
    static constexpr int kElems = 4 * kRawThreads * QUADS;
    static_assert(kElems % S == 0, "whole chunks");
    static constexpr int kChunks = kElems / S;
    static_assert(kChunks <= kRawThreads && kChunks % 4 == 0, "a lane per chunk shuffles");
    static constexpr int kWords = (S + 31) / 32;        // of a chunk's mask
    static constexpr int kPlaces = S + 4;               // bytes of a chunk's shuffle (odd word stride)
    static constexpr int kShuffleBytes = kChunks * kPlaces;
    static constexpr int kMaskBytes = kChunks * kWords * 4;
    static constexpr int kBeforeBytes = kChunks * kWords;
    // entries of the workgroup's chunks as floats; four more that a thread may read and drop
    __host__ __device__ static constexpr int entry_bytes(int k) { return 4 * kChunks * k + 16; }
    // compress: the staged entries take the place of the shuffle; indices, where asked for
    __host__ __device__ static constexpr int shared_bytes(int k) {
        return entry_bytes(k) > kShuffleBytes ? entry_bytes(k) : kShuffleBytes;
    }
    static int compress_lds(int k, bool indices) {
        return kMaskBytes + kBeforeBytes + shared_bytes(k) + (indices ? kChunks * k : 0);
    }
    static int decompress_lds(int k, bool random) {
        return kMaskBytes + kBeforeBytes + entry_bytes(k) + (random ? kShuffleBytes : 0);
    }
};

// A workgroup barrier that orders LDS only: global loads stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The chunks' kept sets: mask[row * kWords + i] = elements 32i .. 32i+31, before[...] = kept elements
// before them.  Random: thread t < kChunks shuffles chunk0 + t, a row per chunk.  Striding: row 0.
template <int S, int QUADS>
__device__ __forceinline__ void raw_kept_sets(const KParams& p, int tid, int64_t chunk0,
                                              uint32_t* mask, uint8_t* before, uint8_t* places) {
    using G = RawGeom<S, QUADS>;
    if (tid >= (p.scheme == 2 ? G::kChunks : kWave)) return;
    const int row = p.scheme == 2 ? tid : 0;
    uint32_t* bits = mask + row * G::kWords;
#pragma unroll
    for (int i = 0; i < G::kWords; ++i) bits[i] = 0u;
    auto take = [&](uint32_t at) { atomicOr(&bits[at / 32], 1u << (at % 32)); };
    if (p.scheme == 2) {
        shuffle_places<S>(p.seed, p.step, static_cast<uint64_t>(chunk0 + row), p.k,
                          places + row * G::kPlaces, take);
    } else {
        const int stride = S / p.k;
        const int off = static_cast<int>(p.step % static_cast<uint64_t>(stride));
        wave_lds_sync();                       // (one wavefront: its LDS operations are in order)
        for (int j = tid; j < p.k; j += kWave) take(static_cast<uint32_t>(off + j * stride));
        wave_lds_sync();
        if (tid != 0) return;
    }
    uint32_t sum = 0u;
#pragma unroll
    for (int i = 0; i < G::kWords; ++i) {
        before[row * G::kWords + i] = static_cast<uint8_t>(sum);   // (at most k <= 128)
        sum += __popc(bits[i]);
    }
}

// The four elements from column col on of row r: which are kept, and the entry of the first kept one
template <int S, int QUADS>
__device__ __forceinline__ void raw_quad(const KParams& p, int r, int col, const uint32_t* mask,
                                         const uint8_t* before, uint32_t& bits, uint32_t& entry) {
    using G = RawGeom<S, QUADS>;
    const int at = (p.scheme == 2 ? r * G::kWords : 0) + col / 32;
    const uint32_t word = mask[at];
    bits = word >> (col % 32);
    entry = __umul24(static_cast<uint32_t>(r), static_cast<uint32_t>(p.k)) + before[at] +
            __popc(word & ((1u << (col % 32)) - 1u));
}

template <int S, int QUADS, bool GRAD_BF16>
__global__ __launch_bounds__(kRawThreads) void compress_raw(
    KParams p, int64_t n, int64_t n_chunks, const void* __restrict__ grad, float* __restrict__ mom,
    void* __restrict__ idx_out, void* __restrict__ val_out, float* __restrict__ coeff_dbg) {
    using G = RawGeom<S, QUADS>;
    extern __shared__ __attribute__((aligned(16))) char raw_smem[];
    uint32_t* mask = reinterpret_cast<uint32_t*>(raw_smem);
    float* staged = reinterpret_cast<float*>(raw_smem + G::kMaskBytes);
    uint8_t* places = reinterpret_cast<uint8_t*>(staged);
    uint8_t* before = reinterpret_cast<uint8_t*>(staged) + G::shared_bytes(p.k);
    uint8_t* staged_at = before + G::kBeforeBytes;

    const int tid = threadIdx.x;
    const int k = p.k;
    const int64_t chunk0 = static_cast<int64_t>(blockIdx.x) * G::kChunks;
    const int64_t base = chunk0 * S;
    const int64_t left_chunks = n_chunks - chunk0;
    const int live = left_chunks < G::kChunks ? static_cast<int>(left_chunks) : G::kChunks;

    // (uniform bases and a 32-bit offset: a scalar base for every access)
    const uint32_t o = 4u * static_cast<uint32_t>(tid);
    float* mom_wg = mom + base;
    const void* grad_wg = GRAD_BF16 ? static_cast<const void*>(static_cast<const uint16_t*>(grad) + base)
                                    : static_cast<const void*>(static_cast<const float*>(grad) + base);
    float* dbg_wg = coeff_dbg ? coeff_dbg + base : nullptr;
    const int64_t room = n - base;          // elements of the shard from here on
    auto body = [&](auto guarded_tag) {
        constexpr bool kGuarded = decltype(guarded_tag)::value;
        // ---- everything is requested first
        float4 m[QUADS], g[GRAD_BF16 ? 1 : QUADS];
        uint2 h[GRAD_BF16 ? QUADS : 1];
        auto whole = [&](uint32_t i) { return !kGuarded || static_cast<int64_t>(i) + 3 < room; };
#pragma unroll
        for (int j = 0; j < QUADS; ++j) {
            const uint32_t i = o + 4u * kRawThreads * j;
            if (whole(i)) {
                m[j] = ld_f4<false>(mom_wg + i);
                if constexpr (GRAD_BF16) h[j] = ld_u2<false>(static_cast<const uint16_t*>(grad_wg) + i);
                else g[j] = ld_f4<false>(static_cast<const float*>(grad_wg) + i);
            } else {
                // the shard's end; what lies past it reads as zero
                float mv[4], gv[4];
                uint32_t hv[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool in = static_cast<int64_t>(i) + e < room;
                    mv[e] = in ? mom_wg[i + e] : 0.0f;
                    if constexpr (GRAD_BF16)
                        hv[e] = in ? static_cast<const uint16_t*>(grad_wg)[i + e] : 0u;
                    else
                        gv[e] = in ? static_cast<const float*>(grad_wg)[i + e] : 0.0f;
                }
                m[j] = make_float4(mv[0], mv[1], mv[2], mv[3]);
                if constexpr (GRAD_BF16) h[j] = make_uint2(hv[0] | (hv[1] << 16), hv[2] | (hv[3] << 16));
                else g[j] = make_float4(gv[0], gv[1], gv[2], gv[3]);
            }
        }
        raw_kept_sets<S, QUADS>(p, tid, chunk0, mask, before, places);
        lds_barrier();
        // (Random: the entries take the place of the shuffle, which is over)

        // ---- m1 = beta*m + g; kept elements go to their entry, the rest stays.  left(c): what a kept one
        // leaves behind
        auto emit = [&](auto left) {
#pragma unroll
            for (int j = 0; j < QUADS; ++j) {
                const uint32_t i = o + 4u * kRawThreads * j;
                const int r = i / S, col = i - r * S;
                uint32_t bits, entry;
                raw_quad<S, QUADS>(p, r, col, mask, before, bits, entry);
                float4 gj;
                if constexpr (GRAD_BF16)
                    gj = make_float4(__uint_as_float(h[j].x << 16),
                                     __uint_as_float(h[j].x & 0xFFFF0000u),
                                     __uint_as_float(h[j].y << 16),
                                     __uint_as_float(h[j].y & 0xFFFF0000u));
                else
                    gj = g[j];
                float c[4] = {fmaf(p.beta, m[j].x, gj.x), fmaf(p.beta, m[j].y, gj.y),
                              fmaf(p.beta, m[j].z, gj.z), fmaf(p.beta, m[j].w, gj.w)};
                if (dbg_wg && (!kGuarded || r < live))
                    st_f4<false>(dbg_wg + i, make_float4(c[0], c[1], c[2], c[3]));
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t bit = (bits >> e) & 1u;
                    if (bit) {
                        staged[entry] = c[e];
                        c[e] = left(c[e]);
                    }
                    entry += bit;
                }
                if (idx_out) {
                    uint32_t at = entry - __popc(bits & 15u);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if ((bits >> e) & 1u) staged_at[at++] = static_cast<uint8_t>(col + e);
                }
                if (whole(i)) {
                    st_f4<true>(mom_wg + i, make_float4(c[0], c[1], c[2], c[3]));
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (static_cast<int64_t>(i) + e < room) mom_wg[i + e] = c[e];
                }
            }
        };
        // (fp32 values and signs: nothing, as a constant, so that an infinity or a NaN that was sent is gone
        // from the momentum; c - c would keep it there as NaN)
        if (p.val_dtype == 1)
            emit([](float c) { return c - __uint_as_float(pack_bf16x2(c, 0.0f) << 16); });
        else if (p.val_dtype == 2)
            emit([](float c) { return c - f16_to_f32(f32_to_f16(c)); });
        else
            emit([](float) { return 0.0f; });
    };
    if (base + G::kElems <= n) body(std::false_type{});
    else body(std::true_type{});
    lds_barrier();

    // ---- the entries of the workgroup's chunks are contiguous in the payload
    const int entries = live * k;
    const int64_t e0 = chunk0 * k;
    if (p.val_dtype == 3) {
        const int nw = ternary_words_per_chunk(k);
        uint32_t* words = static_cast<uint32_t*>(val_out) + chunk0 * nw;
        for (int q = tid; q < live * nw; q += kRawThreads) {
            const int r = q / nw, j0 = 16 * (q - r * nw);
            const float* src = staged + r * k + j0;
            uint32_t word = 0u;
            const int last = min(16, k - j0) - 1;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const uint32_t code = ternary_code(src[min(j, last)]);
                word |= j <= last ? code << (2 * j) : 0u;
            }
            words[q] = word;
        }
    } else if (k % 4 == 0) {
        for (int q = tid; q < entries / 4; q += kRawThreads) {
            const float4 v = *reinterpret_cast<const float4*>(staged + 4 * q);
            if (p.val_dtype == 0) {
                st_f4<false>(static_cast<float*>(val_out) + e0 + 4 * q, v);
            } else {
                uint2 w;
                if (p.val_dtype == 1) {
                    w = make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
                } else {
                    w.x = f32_to_f16(v.x) | (static_cast<uint32_t>(f32_to_f16(v.y)) << 16);
                    w.y = f32_to_f16(v.z) | (static_cast<uint32_t>(f32_to_f16(v.w)) << 16);
                }
                st_u2<false>(static_cast<uint16_t*>(val_out) + e0 + 4 * q, w);
            }
        }
    } else {
        for (int e = tid; e < entries; e += kRawThreads)
            store_payload_value(val_out, e0 + e, p.val_dtype, staged[e]);
    }
    if (idx_out)
        for (int e = tid; e < entries; e += kRawThreads)
            store_payload_index(idx_out, e0 + e, p.idx_u8, staged_at[e]);
}

// Sums over the replicas of the entries [0, entries) behind `val`, replica 0 first, into sums[]; the
// threads [first, kRawThreads) share them, VEC consecutive entries a piece.  In flight: QN pieces of a thread, BATCH
// of their replicas.  Single 16-bit entries are loaded without a branch (the last replica's again past it): behind
// one such a load is widened, and so waited for, before the next one leaves (32/10, 32 replicas, fp16, 5.6 M 134 us
// that way, 70 in the class kernels).
template <int VEC, int VAL, int QN, int BATCH>
__device__ __forceinline__ void raw_entry_sums(const KParams& p, int tid, int first, int entries,
                                               const void* __restrict__ val, int64_t val_stride,
                                               int64_t e0, float* sums) {
    using Piece = SplitPiece<VEC, VAL, true>;
    if (tid < first) return;
    constexpr bool kAlways = VEC == 1 && VAL != 0;
    const int threads = kRawThreads - first, pieces = entries / VEC;
    for (int q0 = tid - first; q0 < pieces; q0 += QN * threads) {
        float sum[QN][VEC];
#pragma unroll
        for (int c = 0; c < QN; ++c)
#pragma unroll
            for (int e = 0; e < VEC; ++e) sum[c][e] = 0.0f;
        for (int r0 = 0; r0 < p.R; r0 += BATCH) {
            Piece b[QN][BATCH];
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
#pragma unroll
                for (int c = 0; c < QN; ++c) b[c][i].clear();
                if (!kAlways && r0 + i >= p.R) continue;
                // (a uniform base and a 32-bit offset of the lane)
                const char* replica = static_cast<const char*>(val) +
                                      (min(r0 + i, p.R - 1) * val_stride + e0) * (VAL == 0 ? 4 : 2);
#pragma unroll
                for (int c = 0; c < QN; ++c)
                    b[c][i].load_values(replica, static_cast<uint32_t>(VEC * min(q0 + c * threads, pieces - 1)), 0);
            }
#pragma unroll
            for (int i = 0; i < BATCH; ++i)
#pragma unroll
                for (int c = 0; c < QN; ++c) {
                    float x[VEC];
                    b[c][i].values(0u, x);
#pragma unroll
                    for (int e = 0; e < VEC; ++e) sum[c][e] += !kAlways || r0 + i < p.R ? x[e] : 0.0f;
                }
        }
#pragma unroll
        for (int c = 0; c < QN; ++c)
            if (q0 + c * threads < pieces)
#pragma unroll
                for (int e = 0; e < VEC; ++e) sums[VEC * (q0 + c * threads) + e] = sum[c][e];
    }
}

// The same for two-bit signs, a word of 16 entries a thread.
__device__ __forceinline__ void raw_sign_sums(const KParams& p, int tid, int first, int live,
                                              const uint32_t* __restrict__ words,
                                              int64_t val_stride, float* sums) {
    if (tid < first) return;
    const int k = p.k, nw = ternary_words_per_chunk(k);
    for (int q = tid - first; q < live * nw; q += kRawThreads - first) {
        const SignCounts counts(words, q, val_stride, p.R);
        const int r = q / nw, j0 = 16 * (q - r * nw);
        float* to = sums + r * k + j0;
        const int cnt = k - j0;
#pragma unroll
        for (int f = 0; f < 16; ++f)
            if (f < cnt) to[f] = counts.sum(f);
    }
}

// OPT: 0 plain update, 1 Decoupled AdamW, 2 with amsgrad.  SIGNS: two-bit signs, in kernels of their own: with fewer
// registers a wavefront per SIMD more than beside the sums of values (64, 2 pieces, bf16 57 against 65).  What a launch
// of 2 - 8 M parameters takes follows the workgroups per CU: 256/8 R = 2 signs 4.7 M 4 a CU 10.7 us, 5 8.1, 6 7.7.
template <int S, int QUADS, bool PARAM_BF16, int OPT, bool SIGNS>
__global__ __launch_bounds__(kRawThreads) void decompress_raw(
    KParams p, int64_t n, int64_t n_chunks, const void* __restrict__ val, int64_t val_stride,
    void* __restrict__ params, AdamPtrs ad, float* __restrict__ presign_dbg) {
    using G = RawGeom<S, QUADS>;
    extern __shared__ __attribute__((aligned(16))) char raw_smem[];
    uint32_t* mask = reinterpret_cast<uint32_t*>(raw_smem);
    float* sums = reinterpret_cast<float*>(raw_smem + G::kMaskBytes);
    uint8_t* before = reinterpret_cast<uint8_t*>(sums) + G::entry_bytes(p.k);
    uint8_t* places = before + G::kBeforeBytes;

    const int tid = threadIdx.x;
    const int k = p.k;
    const int64_t chunk0 = static_cast<int64_t>(blockIdx.x) * G::kChunks;
    const int64_t base = chunk0 * S;
    const int64_t left_chunks = n_chunks - chunk0;
    const int live = left_chunks < G::kChunks ? static_cast<int>(left_chunks) : G::kChunks;

    const uint32_t o = 4u * static_cast<uint32_t>(tid);
    void* par_wg = PARAM_BF16 ? static_cast<void*>(static_cast<uint16_t*>(params) + base)
                              : static_cast<void*>(static_cast<float*>(params) + base);
    float *m_wg = ad.m + (OPT ? base : 0), *v_wg = ad.v + (OPT ? base : 0),
          *x_wg = ad.vmax + (OPT == 2 ? base : 0);
    float* dbg_wg = presign_dbg ? presign_dbg + base : nullptr;
    const int64_t room = n - base;
    auto body = [&](auto guarded_tag) {
        constexpr bool kGuarded = decltype(guarded_tag)::value;
        // ---- parameters and moments are requested first
        float4 th[PARAM_BF16 ? 1 : QUADS], m4[OPT ? QUADS : 1], v4[OPT ? QUADS : 1],
            x4[OPT == 2 ? QUADS : 1];
        uint2 hb[PARAM_BF16 ? QUADS : 1];
        auto whole = [&](uint32_t i) { return !kGuarded || static_cast<int64_t>(i) + 3 < room; };
#pragma unroll
        for (int j = 0; j < QUADS; ++j) {
            const uint32_t i = o + 4u * kRawThreads * j;
            if (!whole(i)) continue;              // (the shard's end: element by element, below)
            if constexpr (PARAM_BF16) hb[j] = ld_u2<true>(static_cast<const uint16_t*>(par_wg) + i);
            else th[j] = ld_f4<true>(static_cast<const float*>(par_wg) + i);
            if constexpr (OPT != 0) {
                m4[j] = ld_f4<true>(m_wg + i);
                v4[j] = ld_f4<true>(v_wg + i);
                if constexpr (OPT == 2) x4[j] = ld_f4<true>(x_wg + i);
            }
        }
        // ---- the kept sets, and meanwhile, where other wavefronts are free, the sums
        raw_kept_sets<S, QUADS>(p, tid, chunk0, mask, before, places);
        const int first = (p.scheme == 2 && G::kChunks <= 2 * kWave)
                              ? (G::kChunks + kWave - 1) / kWave * kWave : 0;
        const int entries = live * k;
        const int64_t e0 = chunk0 * k;
        if constexpr (SIGNS) {
            raw_sign_sums(p, tid, first, live,
                          static_cast<const uint32_t*>(val) + chunk0 * ternary_words_per_chunk(k),
                          val_stride, sums);
        } else {
            auto entry_sums = [&](auto val_tag) {
                constexpr int VAL = decltype(val_tag)::value;
                auto sum = [&](auto vec, auto pieces, auto batch) {
                    raw_entry_sums<decltype(vec)::value, VAL, decltype(pieces)::value, decltype(batch)::value>(
                        p, tid, first, entries, val, val_stride, e0, sums);
                };
                constexpr std::integral_constant<int, 1> c1;
                constexpr std::integral_constant<int, 2> c2;
                constexpr std::integral_constant<int, 4> c4;
                constexpr std::integral_constant<int, 8> c8;
                // (one entry a thread keeps four times as many replicas in flight: where that takes no
                // second turn, and the launch's latency counts)
                if (k % 4 == 0 && (entries > kRawThreads || p.R <= 8 || n > kRawSmall)) {
                    if (p.R <= 2) sum(c4, c4, c2);
                    else if (p.R <= 4) sum(c4, c2, c4);
                    else if constexpr (VAL == 0) sum(c4, c1, c8);
                    else if (p.R <= 8) sum(c4, c2, c8);
                    else sum(c4, c1, std::integral_constant<int, 16>{});
                } else {
                    if (p.R <= 4) sum(c1, c4, c4);
                    else if (p.R <= 8) sum(c1, c2, c8);
                    else if (VAL != 0 || p.R <= 16) sum(c1, c2, std::integral_constant<int, 16>{});
                    else if constexpr (VAL == 0) sum(c1, c1, std::integral_constant<int, 32>{});
                }
            };
            if (p.val_dtype == 0) entry_sums(std::integral_constant<int, 0>{});
            else if (p.val_dtype == 1) entry_sums(std::integral_constant<int, 1>{});
            else entry_sums(std::integral_constant<int, 2>{});
        }
        lds_barrier();

        // ---- update
#pragma unroll
        for (int j = 0; j < QUADS; ++j) {
            const uint32_t i = o + 4u * kRawThreads * j;
            const int r = i / S, col = i - r * S;
            uint32_t bits, entry;
            raw_quad<S, QUADS>(p, r, col, mask, before, bits, entry);
            float y[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t bit = (bits >> e) & 1u;
                const float s = sums[entry];
                y[e] = bit ? s * p.inv_R : 0.0f;
                entry += bit;
            }
            if (!whole(i)) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (static_cast<int64_t>(i) + e >= room) break;
                    if (dbg_wg) dbg_wg[i + e] = y[e];
                    const float q = sign_or_self(y[e], p.use_sign);
                    const float old = PARAM_BF16
                        ? bf16_to_f32(static_cast<const uint16_t*>(par_wg)[i + e])
                        : static_cast<const float*>(par_wg)[i + e];
                    float nw;
                    if constexpr (OPT != 0) {
                        float vm = OPT == 2 ? x_wg[i + e] : 0.0f;
                        nw = adamw_step<OPT == 2>(p, old, q, m_wg[i + e], v_wg[i + e], vm);
                        if constexpr (OPT == 2) x_wg[i + e] = vm;
                    } else {
                        nw = fmaf(-p.lr, q, old * p.wd_scale);
                    }
                    if constexpr (PARAM_BF16) static_cast<uint16_t*>(par_wg)[i + e] = f32_to_bf16(nw);
                    else static_cast<float*>(par_wg)[i + e] = nw;
                }
                continue;
            }
            if (dbg_wg) st_f4<false>(dbg_wg + i, make_float4(y[0], y[1], y[2], y[3]));
            float4 o4;
            if constexpr (PARAM_BF16)
                o4 = make_float4(__uint_as_float(hb[j].x << 16),
                                 __uint_as_float(hb[j].x & 0xFFFF0000u),
                                 __uint_as_float(hb[j].y << 16),
                                 __uint_as_float(hb[j].y & 0xFFFF0000u));
            else
                o4 = th[j];
            const float old[4] = {o4.x, o4.y, o4.z, o4.w};
            float nw[4];
            if constexpr (OPT != 0) {
                float m[4] = {m4[j].x, m4[j].y, m4[j].z, m4[j].w};
                float v[4] = {v4[j].x, v4[j].y, v4[j].z, v4[j].w};
                float4 vm = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if constexpr (OPT == 2) vm = x4[j];
                float x[4] = {vm.x, vm.y, vm.z, vm.w};
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    nw[e] = adamw_step<OPT == 2>(p, old[e], sign_or_self(y[e], p.use_sign), m[e],
                                                 v[e], x[e]);
                st_f4<true>(m_wg + i, make_float4(m[0], m[1], m[2], m[3]));
                st_f4<true>(v_wg + i, make_float4(v[0], v[1], v[2], v[3]));
                if constexpr (OPT == 2) st_f4<true>(x_wg + i, make_float4(x[0], x[1], x[2], x[3]));
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    nw[e] = fmaf(-p.lr, sign_or_self(y[e], p.use_sign), old[e] * p.wd_scale);
            }
            if constexpr (PARAM_BF16)
                st_u2<true>(static_cast<uint16_t*>(par_wg) + i,
                            make_uint2(pack_bf16x2(nw[0], nw[1]), pack_bf16x2(nw[2], nw[3])));
            else
                st_f4<true>(static_cast<float*>(par_wg) + i,
                            make_float4(nw[0], nw[1], nw[2], nw[3]));
        }
    };
    if (base + G::kElems <= n) body(std::false_type{});
    else body(std::true_type{});
}

}  // namespace deto
