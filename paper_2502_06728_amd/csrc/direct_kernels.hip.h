// Matrix-core compress kernels that give the bits of the general kernels: top-k where the DCT has
// to be the sum over t in ascending order, one fused multiply-add per term, that
// compress_generic forms (two-bit signs without a lane-per-chunk kernel; every format at chunk 16
// but fp32 + int32 at its lane-per-chunk k).
//
// Why the bits matter: a near tie at the k-th magnitude is decided by the coefficients' rounding,
// and the new momentum carries the inverse transform's rounding into the next call's ties.
// Why the matrix cores give them: v_mfma_f32_16x16x4_f32 adds its four products in ascending order
// with one rounding each (fp32 fused multiply-adds, subnormals kept): against an fmaf chain over
// 64 terms 0 of 256,000 sums differed, also with subnormal products.  A chain of MFMAs over
// t = 0, 4, 8, ... is therefore compress_generic's loop for 16 coefficients of 16 chunks.  The
// inverse runs over all S coefficients with zeros in place of the dropped ones, which leave an
// fmaf chain as it is.
//
// What bounds it: S multiply-adds per element and direction on the fp32 matrix pipe, 256 FLOP a cycle
// and CU: 82 us for 12.6 M parameters at chunk 256, 20 at 64; the selection on the vector pipe (some
// 60 instructions an element, about 20 us there) runs beside it in other wavefronts.  Measured,
// signs, 12.6 M parameters, bf16 gradients, the general kernel before and this one, us: 16/8 777 and
// 47, 64/8 377 and 61, 96/12 640 and 82, 128/16 626 and 86, 192/24 900 and 117, 256/64 1,398 and 142.
//
// A workgroup owns NC consecutive chunks as LDS rows.
//   product    wavefront w computes the 16-coefficient blocks w, w + NW, ... for all NC chunks:
//              A = the cosines, gathered from a table of one period (2t+1 is odd: the 16 lanes of a
//              block hit 16 banks), B = the rows (row stride S + 4: 16 chunks x 4 terms hit all
//              64 banks).  A gathered cosine serves all NC / 16 column blocks.
//   selection  L = S / Q lanes share a chunk, Q coefficients each, four consecutive ones at a
//              time: bisection on the magnitudes' bits, from the chunk's largest downwards, until
//              a candidate has exactly k at or above it; L <= 16 keeps the counts within DPP rows.
//              Emission positions: one packed prefix sum over the L lanes.
#pragma once

#include "deto_device.hip.h"
#include "fast_dct.hip.h"
#include "generic_kernels.hip.h"

namespace deto {

typedef float f32x4_acc __attribute__((ext_vector_type(4)));

template <int S>
struct DirectGeom {
    static_assert(S % 16 == 0 && S <= 256, "whole blocks of 16 coefficients");
    static constexpr int NC = S == 16 ? 64 : 32;                   // chunks per workgroup
    static constexpr int NW = S <= 32 ? 1 : S == 64 ? 2 : (S == 192 || S == 256) ? 8 : 4;   // wavefronts
    static constexpr int kThreads = kWave * NW;
    static constexpr int Q = NC * S / kThreads;                    // coefficients per lane
    static constexpr int L = S / Q;                                // lanes per chunk
    static_assert(Q % 4 == 0 && Q <= 32 && L <= 16 && (L & (L - 1)) == 0, "DPP rows");
    static constexpr int JB = S / 16;
    static constexpr int BJ = (JB + NW - 1) / NW;                  // coefficient blocks per wavefront
    static constexpr int CB = NC / 16;
    static constexpr int kRow = S + 4;
    static constexpr bool kStageValues = S == 16;                  // formats other than two-bit signs
};

// cos(pi t / (2S)), t = 0 ... S, rounded once from double: compress_generic's table (built there at
// run time).  From pi/4 on as the sine of the complement, where the series converge fast.
template <int S>
struct CosQuarter {
    float v[S + 1];
    constexpr CosQuarter() : v{} {
        for (int t = 0; t < S; ++t)
            v[t] = static_cast<float>(2 * t <= S ? ct_cos(kPi * t / (2.0 * S))
                                                 : ct_sin(kPi * (S - t) / (2.0 * S)));
        v[S] = 0.0f;
    }
};
template <int S>
__device__ constexpr CosQuarter<S> kCosQuarter{};

// the value of another lane (quad permutations; groups of 8 and 16 by mirroring, which pairs lanes
// that hold equal partial results)
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_mov(uint32_t x) {
    return static_cast<uint32_t>(
        __builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, 0xf, 0xf, false));
}
// op over the L lanes of a group, in every lane of it
template <int L, class Op>
__device__ __forceinline__ uint32_t group_reduce(uint32_t x, Op op) {
    if constexpr (L >= 2) x = op(x, dpp_mov<0xB1>(x));     // quad_perm 1,0,3,2
    if constexpr (L >= 4) x = op(x, dpp_mov<0x4E>(x));     // quad_perm 2,3,0,1
    if constexpr (L >= 8) x = op(x, dpp_mov<0x141>(x));    // row_half_mirror
    if constexpr (L >= 16) x = op(x, dpp_mov<0x140>(x));   // row_mirror
    return x;
}
// sum over the lanes of the group before this one
template <int L>
__device__ __forceinline__ uint32_t group_exclusive_sum(uint32_t own, int part) {
    uint32_t x = own;
    auto step = [&](uint32_t shifted, int d) { x += part >= d ? shifted : 0u; };
    if constexpr (L >= 2) step(dpp_mov<0x111>(x), 1);      // row_shr 1, 2, 4, 8
    if constexpr (L >= 4) step(dpp_mov<0x112>(x), 2);
    if constexpr (L >= 8) step(dpp_mov<0x114>(x), 4);
    if constexpr (L >= 16) step(dpp_mov<0x118>(x), 8);
    return x - own;
}

// acc[b][cb] = the sums over u = 0 ... S-1, ascending, of cosine times row entry u, for the 16 block
// rows and the 16 chunks of column block cb.  Lane (i, h) brings in block row i's cosines and chunk
// i's entries for the terms u = h, h + 4, ...; cur[b] is the byte of the first of those cosines in
// the table and advances by inc[b] per step, modulo the period.  BJ: blocks this wavefront has.
template <int S, int BJ>
__device__ __forceinline__ void direct_product(const float* __restrict__ tab,
                                               const float* __restrict__ rows, int i, int h,
                                               uint32_t (&cur)[DirectGeom<S>::BJ],
                                               const uint32_t (&inc)[DirectGeom<S>::BJ],
                                               f32x4_acc (&acc)[DirectGeom<S>::BJ][DirectGeom<S>::CB]) {
    using G = DirectGeom<S>;
    constexpr uint32_t kPeriod = 4u * 4u * S;              // bytes
#pragma unroll
    for (int b = 0; b < BJ; ++b)
#pragma unroll
        for (int cb = 0; cb < G::CB; ++cb) acc[b][cb] = f32x4_acc{0.0f, 0.0f, 0.0f, 0.0f};
    const float* x = rows + i * G::kRow + h;
    // (sixteen terms at a time, the next sixteen requested before these are multiplied)
    constexpr int kGroups = S / 16;
    struct Terms {
        float a[4][BJ], bx[4][G::CB];
    };
    auto request = [&](int g, Terms& t) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
            for (int cb = 0; cb < G::CB; ++cb)
                t.bx[u][cb] = x[cb * 16 * G::kRow + 16 * g + 4 * u];
#pragma unroll
            for (int b = 0; b < BJ; ++b) {
                t.a[u][b] =
                    *reinterpret_cast<const float*>(reinterpret_cast<const char*>(tab) + cur[b]);
                const uint32_t nx = cur[b] + inc[b];
                cur[b] = min(nx, nx - kPeriod);            // (wraps below zero to a large number)
            }
        }
    };
    auto multiply = [&](const Terms& t) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int b = 0; b < BJ; ++b)
#pragma unroll
                for (int cb = 0; cb < G::CB; ++cb)
                    acc[b][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(t.a[u][b], t.bx[u][cb],
                                                                      acc[b][cb], 0, 0, 0);
    };
    Terms t0, t1;
    request(0, t0);
#pragma unroll 1
    for (int g = 0; g < kGroups; g += 2) {
        if (g + 1 < kGroups) request(g + 1, t1);
        multiply(t0);
        if (g + 2 < kGroups) request(g + 2, t0);
        if (g + 1 < kGroups) multiply(t1);
    }
}

// Compress half, top-k.  Workgroups [0, tiles): NC whole chunks; one more for what is left (fewer
// chunks, the last possibly ragged): its accesses are checked against the end of the shard.
template <int S, bool GRAD_BF16>
__global__ __launch_bounds__(DirectGeom<S>::kThreads) void compress_direct(
    KParams p, int64_t tiles, int64_t n, int64_t n_chunks, const void* __restrict__ grad,
    float* __restrict__ mom, void* __restrict__ idx_out, void* __restrict__ val_out,
    float* __restrict__ coeff_dbg) {
    using G = DirectGeom<S>;
    constexpr int NC = G::NC, NW = G::NW, Q = G::Q, L = G::L, BJ = G::BJ, CB = G::CB;
    constexpr int kRow = G::kRow, kThreads = G::kThreads;
    constexpr int kV = Q / 4;                              // groups of four coefficients per lane
    __shared__ __attribute__((aligned(16))) float rows[NC * kRow];
    __shared__ float tab[4 * S];
    // entry pos of chunk c at [c * S + pos]: index | code << 8 (two-bit signs); with kStageValues the
    // index alone and the value beside it
    __shared__ __attribute__((aligned(16))) uint16_t staged[NC * S];
    __shared__ __attribute__((aligned(16))) float staged_val[G::kStageValues ? NC * S : 1];

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int k = p.k;
    const int64_t tile = blockIdx.x;
    // (every other workgroup deals its blocks out from the middle: where JB is not a multiple of NW,
    // the wavefronts with one block more are then not all on the same SIMDs)
    const int w = __builtin_amdgcn_readfirstlane(((tid >> 6) + (tile & 1) * (NW / 2)) & (NW - 1));
    const bool partial = tile >= tiles;
    const int live = partial ? static_cast<int>(n_chunks - tiles * NC) : NC;
    const int64_t base = tile * static_cast<int64_t>(NC * S);
    const int64_t chunk0 = tile * NC;

    // ---- m1 = beta*m + g, coalesced, into the rows (zero past the end of the shard)
    auto fold_piece = [&](int e4) {
        const float4 m = ld_f4<false>(mom + base + e4);
        float4 g;
        if constexpr (GRAD_BF16) {
            const uint2 gb = ld_u2<false>(static_cast<const uint16_t*>(grad) + base + e4);
            g = make_float4(__uint_as_float(gb.x << 16), __uint_as_float(gb.x & 0xFFFF0000u),
                            __uint_as_float(gb.y << 16), __uint_as_float(gb.y & 0xFFFF0000u));
        } else {
            g = ld_f4<false>(static_cast<const float*>(grad) + base + e4);
        }
        const int r = e4 / S, col = e4 - r * S;
        *reinterpret_cast<float4*>(&rows[r * kRow + col]) =
            make_float4(fmaf(p.beta, m.x, g.x), fmaf(p.beta, m.y, g.y), fmaf(p.beta, m.z, g.z),
                        fmaf(p.beta, m.w, g.w));
    };
    if (!partial) {
#pragma unroll
        for (int v = 0; v < kV; ++v) fold_piece(4 * (tid + kThreads * v));
    } else {
        for (int v = 0; v < kV; ++v) {
            const int e4 = 4 * (tid + kThreads * v);
            if (base + e4 + 3 < n) {
                fold_piece(e4);
            } else {
                const int r = e4 / S, col = e4 - r * S;
                for (int j = 0; j < 4; ++j) {
                    const int64_t i = base + e4 + j;
                    float x = 0.0f;
                    if (i < n) {
                        const float g = GRAD_BF16 ? bf16_to_f32(static_cast<const uint16_t*>(grad)[i])
                                                  : static_cast<const float*>(grad)[i];
                        x = fmaf(p.beta, mom[i], g);
                    }
                    rows[r * kRow + col + j] = x;
                }
            }
        }
    }
    // the cosine table, one period from its first quarter
    for (int t = tid; t <= S; t += kThreads) {
        const float c = kCosQuarter<S>.v[t];
        tab[t] = c;
        tab[2 * S - t] = -c;
        tab[2 * S + t] = -c;
        if (t > 0) tab[4 * S - t] = c;
    }
    __syncthreads();

    // ---- coefficients: block row i of block jb is coefficient 16 jb + i
    const int i = lane & 15, h = lane >> 4;
    f32x4_acc acc[BJ][CB];
    float4 x[BJ][CB];                                      // m1 at the places this lane writes later
    auto place = [&](int b, int cb) -> float* {
        return &rows[(16 * cb + i) * kRow + 16 * (w + NW * b) + 4 * h];
    };
    auto active = [&](int b) { return G::JB % NW == 0 || b + 1 < BJ || w + NW * b < G::JB; };
    auto product = [&](uint32_t (&cur)[BJ], const uint32_t (&inc)[BJ]) {
        if (active(BJ - 1)) direct_product<S, BJ>(tab, rows, i, h, cur, inc, acc);
        else if constexpr (BJ > 1) direct_product<S, BJ - 1>(tab, rows, i, h, cur, inc, acc);
    };
    {
        uint32_t cur[BJ], inc[BJ];
#pragma unroll
        for (int b = 0; b < BJ; ++b) {
            const uint32_t j = 16 * (w + NW * b) + i;
            cur[b] = 4u * ((2 * h + 1) * j % (4 * S));     // term t = h first: (2t+1) j
            inc[b] = 4u * (8 * j % (4 * S));
        }
        product(cur, inc);
    }
#pragma unroll
    for (int b = 0; b < BJ; ++b)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
            if (active(b)) x[b][cb] = *reinterpret_cast<const float4*>(place(b, cb));
    __syncthreads();
#pragma unroll
    for (int b = 0; b < BJ; ++b) {
        const bool first = w + NW * b == 0 && h == 0;      // holds coefficient 0
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
            if (active(b))
                *reinterpret_cast<float4*>(place(b, cb)) =
                    make_float4(acc[b][cb][0] * (first ? p.alpha0 : p.alpha), acc[b][cb][1] * p.alpha,
                                acc[b][cb][2] * p.alpha, acc[b][cb][3] * p.alpha);
    }
    __syncthreads();

    // ---- selection: this lane's coefficients are 4 (L v + part) + e
    {
        const int chunk = tid / L, part = tid % L;
        float* mine = &rows[chunk * kRow + 4 * part];
        float c[Q];
        uint32_t mag[Q];
#pragma unroll
        for (int v = 0; v < kV; ++v) {
            const float4 t = *reinterpret_cast<const float4*>(mine + 4 * L * v);
            c[4 * v] = t.x; c[4 * v + 1] = t.y; c[4 * v + 2] = t.z; c[4 * v + 3] = t.w;
        }
        if (coeff_dbg && chunk < live) {
            float* dbg = coeff_dbg + (chunk0 + chunk) * S + 4 * part;
#pragma unroll
            for (int v = 0; v < kV; ++v)
                *reinterpret_cast<float4*>(dbg + 4 * L * v) =
                    make_float4(c[4 * v], c[4 * v + 1], c[4 * v + 2], c[4 * v + 3]);
        }
        uint32_t top = 0u;
#pragma unroll
        for (int m = 0; m < Q; ++m) {
            mag[m] = __float_as_uint(c[m]) & 0x7FFFFFFFu;
            top = max(top, mag[m]);
        }
        top = group_reduce<L>(top, [](uint32_t a, uint32_t b) { return max(a, b); });
        auto count_at_least = [&](uint32_t cand) -> int {
            uint32_t cnt = 0u;
#pragma unroll
            for (int m = 0; m < Q; m += 4)
                cnt = add_if_at_least(cnt, mag[m], mag[m + 1], mag[m + 2], mag[m + 3], cand);
            return static_cast<int>(
                group_reduce<L>(cnt, [](uint32_t a, uint32_t b) { return a + b; }));
        };
        // lo: at least k magnitudes reach it; hi: fewer than k do.  First downwards from the
        // largest in growing steps (one octave, four, sixteen, ...), then by halves.  A candidate is
        // always between the two, so every step narrows a running chunk's bracket: 2^23, 2^25, 2^27
        // and 2^29 downwards at most (hi - lo never exceeds 2^31), then at most 32 halves.
        uint32_t lo = 0u, hi = top + 1u, thr = 0u, step = 1u << 23;
        bool open = k < S, down = true;
        while (__any(open && hi - lo > 1u)) {
            const bool run = open && hi - lo > 1u;
            const bool stride = down && hi - lo > step;
            const uint32_t cand = stride ? hi - step : lo + ((hi - lo) >> 1);
            const int cnt = count_at_least(cand);
            if (run) {
                if (cnt >= k) {
                    lo = cand;
                    down = false;
                } else {
                    hi = cand;
                }
                if (stride) step <<= 2;
                if (cnt == k) {
                    thr = cand;
                    open = false;
                }
            }
        }
        // an open chunk has a tie at magnitude lo: everything above it, and of its equals the first
        uint32_t keep = 0u;                                // bit 4v + e
        const uint32_t thr_gt = open ? lo + 1u : thr;
#pragma unroll
        for (int m = 0; m < Q; ++m) keep |= mag[m] >= thr_gt ? 1u << m : 0u;
        // counts of the groups of four (at most 64 over the lanes of a chunk: a byte each)
        auto counts = [&](uint32_t bits, uint32_t (&packed)[2]) {
            packed[0] = packed[1] = 0u;
#pragma unroll
            for (int v = 0; v < kV; ++v)
                packed[v / 4] |= static_cast<uint32_t>(__popc((bits >> (4 * v)) & 0xFu)) << (8 * (v % 4));
        };
        // position of the first of this lane's entries of group v among all entries of the chunk
        auto positions = [&](uint32_t bits, int (&at)[kV]) {
            uint32_t own[2], before[2] = {0u, 0u}, all[2] = {0u, 0u};
            counts(bits, own);
#pragma unroll
            for (int j = 0; j < (kV + 3) / 4; ++j) {
                before[j] = group_exclusive_sum<L>(own[j], part);
                all[j] = group_reduce<L>(own[j], [](uint32_t a, uint32_t b) { return a + b; });
            }
            int lower = 0;
#pragma unroll
            for (int v = 0; v < kV; ++v) {
                at[v] = lower + ((before[v / 4] >> (8 * (v % 4))) & 0xFF);
                lower += (all[v / 4] >> (8 * (v % 4))) & 0xFF;
            }
        };
        if (__any(open)) {
            uint32_t equal = 0u;
#pragma unroll
            for (int m = 0; m < Q; ++m) equal |= mag[m] == lo ? 1u << m : 0u;
            const int need = k - static_cast<int>(group_reduce<L>(
                                     __popc(keep), [](uint32_t a, uint32_t b) { return a + b; }));
            int at[kV];
            positions(equal, at);
#pragma unroll
            for (int v = 0; v < kV; ++v)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t bit = 1u << (4 * v + e);
                    if (open && (equal & bit) && at[v]++ < need) keep |= bit;
                }
        }
        int at[kV];
        positions(keep, at);
        uint16_t* out = &staged[chunk * S];
#pragma unroll
        for (int v = 0; v < kV; ++v) {
            float left[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int m = 4 * v + e;
                const uint32_t j = 4 * (L * v + part) + e;
                left[e] = 0.0f;
                if ((keep >> m) & 1u) {
                    if constexpr (G::kStageValues) {
                        out[at[v]] = static_cast<uint16_t>(j);
                        staged_val[chunk * S + at[v]] = c[m];
                        left[e] = payload_roundtrip(p.val_dtype, c[m]);
                    } else {
                        out[at[v]] = static_cast<uint16_t>(j | (ternary_code(c[m]) << 8));
                        left[e] = c[m];
                    }
                    ++at[v];
                    left[e] *= j == 0 ? p.alpha0 : p.alpha;
                }
            }
            *reinterpret_cast<float4*>(mine + 4 * L * v) = make_float4(left[0], left[1], left[2], left[3]);
        }
    }
    __syncthreads();

    // ---- payload: the tile's entries are contiguous in both arrays
    if (k % 4 == 0) {
        for (int q = tid; q < live * k / 4; q += kThreads) {
            const int c = 4 * q / k, pos = 4 * q - c * k;
            const uint2 t = *reinterpret_cast<const uint2*>(&staged[c * S + pos]);
            const uint32_t a0 = t.x & 0xFFu, a1 = (t.x >> 16) & 0xFFu, a2 = t.y & 0xFFu,
                           a3 = (t.y >> 16) & 0xFFu;
            const int64_t e = chunk0 * k + 4 * q;
            if (p.idx_u8)
                *reinterpret_cast<uint32_t*>(static_cast<uint8_t*>(idx_out) + e) =
                    a0 | (a1 << 8) | (a2 << 16) | (a3 << 24);
            else
                *reinterpret_cast<int4*>(static_cast<int32_t*>(idx_out) + e) =
                    make_int4(static_cast<int>(a0), static_cast<int>(a1), static_cast<int>(a2),
                              static_cast<int>(a3));
        }
    } else {
        for (int q = tid; q < live * k; q += kThreads) {
            const int c = q / k, pos = q - c * k;
            store_payload_index(idx_out, chunk0 * k + q, p.idx_u8, staged[c * S + pos] & 0xFF);
        }
    }
    if (p.val_dtype == 3) {
        const int nw = ternary_words_per_chunk(k);
        for (int q = tid; q < live * nw; q += kThreads) {
            const int c = q / nw, j0 = 16 * (q - c * nw);
            const int in = min(16, k - j0);
            uint32_t word = 0u;
            if constexpr (G::kStageValues) {
                for (int e = 0; e < in; ++e)
                    word |= ternary_code(staged_val[c * S + j0 + e]) << (2 * e);
            } else {
                const uint4* s4 = reinterpret_cast<const uint4*>(&staged[c * S + j0]);
                const uint4 t0 = s4[0], t1 = s4[1];
                const uint32_t two[8] = {t0.x, t0.y, t0.z, t0.w, t1.x, t1.y, t1.z, t1.w};
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    word |= (((two[e] >> 8) & 3u) | (((two[e] >> 24) & 3u) << 2)) << (4 * e);
                // (places past the chunk's k entries hold whatever an earlier launch left)
                word &= 0xFFFFFFFFu >> (32 - 2 * in);
            }
            static_cast<uint32_t*>(val_out)[chunk0 * nw + q] = word;
        }
    } else if constexpr (G::kStageValues) {
        for (int q = tid; q < live * k; q += kThreads) {
            const int c = q / k, pos = q - c * k;
            store_payload_value(val_out, chunk0 * k + q, p.val_dtype, staged_val[c * S + pos]);
        }
    }

    // ---- m <- m1 - q: block row i of block jb is element 16 jb + i
    {
        uint32_t cur[BJ], inc[BJ];
#pragma unroll
        for (int b = 0; b < BJ; ++b) {
            const uint32_t odd = 2 * (16 * (w + NW * b) + i) + 1;
            cur[b] = 4u * (odd * h % (4 * S));             // term j = h first: (2n+1) j
            inc[b] = 4u * (4 * odd % (4 * S));
        }
        product(cur, inc);
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < BJ; ++b)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
            if (active(b))
                *reinterpret_cast<float4*>(place(b, cb)) =
                    make_float4(x[b][cb].x - acc[b][cb][0], x[b][cb].y - acc[b][cb][1],
                                x[b][cb].z - acc[b][cb][2], x[b][cb].w - acc[b][cb][3]);
    __syncthreads();
    for (int v = 0; v < kV; ++v) {
        const int e4 = 4 * (tid + kThreads * v);
        const int r = e4 / S, col = e4 - r * S;
        const float4 y = *reinterpret_cast<const float4*>(&rows[r * kRow + col]);
        if (!partial || base + e4 + 3 < n) {
            st_f4<true>(mom + base + e4, y);
        } else {
            const float ys[4] = {y.x, y.y, y.z, y.w};
            for (int j = 0; j < 4; ++j)
                if (base + e4 + j < n) mom[base + e4 + j] = ys[j];
        }
    }
}

}  // namespace deto
