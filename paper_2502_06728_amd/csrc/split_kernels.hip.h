// Lane per chunk, wavefront per coefficient class: compress from chunk 96 on (on small shards from 64,
// without top-k from 16; top-k at 256 with k <= 32 in half_tile_kernels.hip.h), decompress at chunk
// 16 ... 256 by the rules in tiled_launch.h.
//
// A chunk of more than 64 elements does not fit one lane's registers at two wavefronts per
// SIMD.  Splitting it between two lanes of ONE wavefront makes the lanes run different
// half-size transforms (a DCT-II and a DCT-IV) one after the other.  Here the split is between
// the W wavefronts of a workgroup instead: the workgroup owns a tile of 64 chunks in LDS
// (row = chunk), lane t of EVERY wavefront works on chunk t, and wavefront w computes one class
// of the chunk's coefficients, S/W of them, in its lanes' registers.  Every wavefront runs
// straight-line code with no divergence, and the classes meet in LDS at workgroup barriers.
//
//   W = 2, first level of the DCT-II recursion of fast_dct.hip.h:
//     class 0: u_n = x_n + x_{S-1-n}, coefficients 2m   = dct2_{S/2}(u)
//     class 1: w_n = x_n - x_{S-1-n}, coefficients 2m+1 = dct4_{S/2}(w)
//   W = 4, two levels, Q = S/4:
//     class 0: coefficients 4m   = dct2_Q(u_n + u_{S/2-1-n})
//     class 1: coefficients 4m+2 = dct4_Q(u_n - u_{S/2-1-n})
//     class 2, 3: the DCT-IV of w (length S/2) by plane rotations into two DCT-IIs of length
//              Q, A (class 2) and B (class 3); after an exchange through LDS class 2 holds the
//              coefficients 4m+1 = A_m + B_{Q-m} and class 3 the coefficients
//              4m+3 = A_{m+1} - B_{Q-1-m}.
// The inverse runs the same splits backwards (DCT-III / DCT-IV).
//
// Selection (top-k, any k at run time): every lane sorts the magnitudes of its S/W coefficients
// with a sorting network; the sorted lists of a chunk meet in the chunk's LDS row.  For W = 4
// the lists of classes (0,1) and (2,3) are first merged into two sorted lists of 128 (one
// bitonic half-cleaner across the two wavefronts, then a bitonic merge network per lane).  The
// k-th largest of the union of two sorted lists follows from a binary search over how many of
// the k come from the first list.  A tie at the threshold sends the chunk through the
// whole-wavefront pass that keeps the lowest indices among the equals.
//
// Emission: every class knows the other classes' kept sets as bit masks (exchanged through
// LDS), so a lane can tell the payload position of each of its kept coefficients: its rank
// among all kept coefficients of the chunk with a smaller index.  Values and indices are staged
// in the chunk's row and leave with coalesced stores.
#pragma once

#include "fast_dct.hip.h"
#include "generic_kernels.hip.h"
#include "mfma_kernels.hip.h"
#include "sort_network.hip.h"

namespace deto {

template <int S, int W>
struct SplitGeom {
    static_assert(W == 2 || W == 4, "two or four coefficient classes");
    static_assert(S % (4 * W) == 0, "16-byte pieces per class");
    static constexpr int Q = S / W;                 // coefficients per lane
    static constexpr int kRow = S + 4;              // floats per LDS row (16 B of padding)
    static constexpr int kTile = kWave * kRow;
    static constexpr int kThreads = kWave * W;
    static constexpr int NW = (Q + 31) / 32;        // mask words per lane
    // payload staging inside a chunk's row: values at row[pos], indices at row[kIdx0 + pos]
    // (k <= S/2); what a lane drops goes to a dump slot of its own past the tile
    static constexpr int kIdx0 = S / 2 + 4;
    static constexpr int kBufFloats = kTile + kThreads + kIdx0;
};

// index of coefficient m of class w: W*m + split_off(w)
template <int W>
__device__ __forceinline__ int split_off(int w) {
    if constexpr (W == 2) return w;
    else return ((w & 1) << 1) | (w >> 1);          // 0, 2, 1, 3
}

// k-th largest of the union of two descending lists of length L in LDS: i of the k largest
// come from list 0 and k - i from list 1, i being the smallest count for which list0[i] (the
// first one left out) does not exceed list1[k-i-1] (the last one taken).
template <int L>
__device__ __forceinline__ uint32_t kth_of_two_lists(const uint32_t* l0, const uint32_t* l1,
                                                     int k) {
    int lo = k > L ? k - L : 0, hi = k < L ? k : L;
    constexpr int kSteps = L <= 63 ? 6 : (L <= 127 ? 7 : 8);   // ceil(log2(L + 1))
#pragma unroll
    for (int it = 0; it < kSteps; ++it) {
        const bool open = lo < hi;
        const int mid = (lo + hi) >> 1;
        const uint32_t x0 = l0[open ? mid : 0];
        const uint32_t x1 = l1[open ? k - mid - 1 : 0];
        if (open) {
            if (x0 > x1) lo = mid + 1;
            else hi = mid;
        }
    }
    const int n0 = lo, n1 = k - lo;
    const uint32_t t0 = l0[n0 > 0 ? n0 - 1 : 0], t1 = l1[n1 > 0 ? n1 - 1 : 0];
    return min(n0 > 0 ? t0 : 0xFFFFFFFFu, n1 > 0 ? t1 : 0xFFFFFFFFu);
}

template <int Q>
__device__ __forceinline__ void regs_to_lds(float* dst, const float (&v)[Q]) {
#pragma unroll
    for (int q = 0; q < Q / 4; ++q)
        *reinterpret_cast<float4*>(dst + 4 * q) =
            make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
}

template <int Q>
__device__ __forceinline__ void lds_to_regs(const float* src, float (&v)[Q]) {
#pragma unroll
    for (int q = 0; q < Q / 4; ++q) {
        const float4 t = *reinterpret_cast<const float4*>(src + 4 * q);
        v[4 * q] = t.x; v[4 * q + 1] = t.y; v[4 * q + 2] = t.z; v[4 * q + 3] = t.w;
    }
}

// src[Q-1-i] for i < Q (a list read back to front)
template <int Q>
__device__ __forceinline__ void lds_to_regs_reversed(const float* src, float (&v)[Q]) {
#pragma unroll
    for (int q = 0; q < Q / 4; ++q) {
        const float4 t = *reinterpret_cast<const float4*>(src + Q - 4 - 4 * q);
        v[4 * q] = t.w; v[4 * q + 1] = t.z; v[4 * q + 2] = t.y; v[4 * q + 3] = t.x;
    }
}

// Ends one of several branches that do the same with different parts of a register array: merged into
// one (by a chosen address) they would keep the array in scratch memory.
#define DETO_KEEP_APART(text) asm volatile("; " text)

// dst[i] = src[i] for i = B .. E-1 of a register array
template <int B, int E, int Q>
__device__ __forceinline__ void regs_range_to_lds(float* dst, const float (&v)[Q]) {
    static_assert((E - B) % 4 == 0, "whole pieces");
#pragma unroll
    for (int i = B; i < E; i += 4)
        *reinterpret_cast<float4*>(dst + i - B) = make_float4(v[i], v[i + 1], v[i + 2], v[i + 3]);
}
// dst[i] = v[E-1-i] for i = 0 .. E-B-1
template <int B, int E, int Q>
__device__ __forceinline__ void reversed_range_to_lds(float* dst, const float (&v)[Q]) {
    static_assert((E - B) % 4 == 0, "whole pieces");
#pragma unroll
    for (int i = 0; i < E - B; i += 4)
        *reinterpret_cast<float4*>(dst + i) =
            make_float4(v[E - 1 - i], v[E - 2 - i], v[E - 3 - i], v[E - 4 - i]);
}
template <int B, int E, int Q>
__device__ __forceinline__ void lds_to_regs_range(const float* src, float (&v)[Q]) {
#pragma unroll
    for (int i = B; i < E; i += 4) {
        const float4 t = *reinterpret_cast<const float4*>(src + i - B);
        v[i] = t.x; v[i + 1] = t.y; v[i + 2] = t.z; v[i + 3] = t.w;
    }
}

// The sums A_i + B_j and differences A_i - B_j that end (and, in the inverse, begin) the split of
// the DCT-IV over classes 2 and 3.  FUSED: a and b come from dct2_open, and where one of them still
// lacks its last multiplication, that and the addition round once.  This is how the compiler
// rounds them inside FastDct::dct4, hence in the two-lanes-per-chunk kernels, which hold both
// operands in one lane; the narrow payload formats keep their results by it (rounded twice,
// values differ in the last bit, and from a chunk's second call on so do near ties: chunk 128,
// 192, 256 with 16-bit values, 12 M parameters, fourth call: up to 4 chunks).
template <int Q, bool FUSED, int I, int J>
__device__ __forceinline__ float class_sum(float a, float b) {
    constexpr float fa = FUSED ? FastDct<Q>::dct2_factor(I) : 1.0f;
    constexpr float fb = FUSED ? FastDct<Q>::dct2_factor(J) : 1.0f;
    if constexpr (fa != 1.0f && fb != 1.0f) return fmaf(a, fa, b * fb);
    else if constexpr (fa != 1.0f) return fmaf(a, fa, b);
    else if constexpr (fb != 1.0f) return fmaf(b, fb, a);
    else return a + b;
}
template <int Q, bool FUSED, int I, int J>
__device__ __forceinline__ float class_difference(float a, float b) {
    constexpr float fa = FUSED ? FastDct<Q>::dct2_factor(I) : 1.0f;
    constexpr float fb = FUSED ? FastDct<Q>::dct2_factor(J) : 1.0f;
    if constexpr (fa != 1.0f && fb != 1.0f) return fmaf(a, fa, -(b * fb));
    else if constexpr (fa != 1.0f) return fmaf(a, fa, -b);
    else if constexpr (fb != 1.0f) return fmaf(b, -fb, a);
    else return a - b;
}

// W = 4: f(class as a compile-time number).  Branches on the class inside an unrolled loop would cut it
// up, or keep the operands of both sides live: with the inputs and the inverse's rotations by class,
// compress alone, us, before and with it: 10.8 M fp32 128/16 fp16 36.3, 34.1; 60 M bf16 128/16 136,
// 129, 192/24 158, 149, 256/64 209, 196.  (Two classes differ by a sign only: 96/12 130, 138.)
template <class F>
__device__ __forceinline__ void by_class(int w, F f) {
    if (w == 0) f(std::integral_constant<int, 0>{});
    else if (w == 1) f(std::integral_constant<int, 1>{});
    else if (w == 2) f(std::integral_constant<int, 2>{});
    else f(std::integral_constant<int, 3>{});
}

// W = 4: class CLS's inputs of the transform from the chunk's row
template <int S, int CLS>
__device__ __forceinline__ void split_forward_inputs(const float* __restrict__ row,
                                                     float (&c)[S / 4]) {
    constexpr int Q = S / 4, H = S / 2;
    // four elements at a time: x[n], x[S-1-n], x[H-1-n], x[H+n] for n = 4q .. 4q+3
    static_for<0, Q / 4>([&](auto q) {
        const float4 f0 = *reinterpret_cast<const float4*>(row + 4 * q);
        const float4 r1 = *reinterpret_cast<const float4*>(row + S - 4 - 4 * q);
        const float4 r2 = *reinterpret_cast<const float4*>(row + H - 4 - 4 * q);
        const float4 f3 = *reinterpret_cast<const float4*>(row + H + 4 * q);
        const float x0[4] = {f0.x, f0.y, f0.z, f0.w};
        const float x1[4] = {r1.w, r1.z, r1.y, r1.x};
        const float x2[4] = {r2.w, r2.z, r2.y, r2.x};
        const float x3[4] = {f3.x, f3.y, f3.z, f3.w};
        static_for<0, 4>([&](auto i) {
            constexpr int j = 4 * q + i;
            if constexpr (CLS < 2) {
                constexpr float sgn = CLS ? -1.0f : 1.0f;
                c[j] = fmaf(sgn, x2[i] + x3[i], x0[i] + x1[i]);
            } else {
                // rotations of the DCT-IV of w (length H): pair (w_j, w_{H-1-j})
                constexpr float cs = Rot<H, j>::c, sn = Rot<H, j>::s;
                const float wj = x0[i] - x1[i], wr = x2[i] - x3[i];
                if constexpr (CLS == 2) {
                    c[j] = fmaf(wj, cs, wr * sn);
                } else {
                    const float bv = fmaf(wr, cs, -(wj * sn));
                    c[j] = (j % 2) ? -bv : bv;
                }
            }
        });
    });
}

// The lane's class of coefficients (unscaled; FUSED: classes 2 and 3 without the multiplications that
// class_sum does).
template <int S, int W, bool FUSED = false>
__device__ __forceinline__ void split_forward_local(const float* __restrict__ row, int w,
                                                    float (&c)[S / W]) {
    constexpr int Q = S / W;
    if constexpr (W == 2) {
        const float sgn = w ? -1.0f : 1.0f;
#pragma unroll
        for (int q = 0; q < Q / 4; ++q) {
            const float4 a = *reinterpret_cast<const float4*>(row + 4 * q);
            const float4 b = *reinterpret_cast<const float4*>(row + S - 4 - 4 * q);
            c[4 * q] = fmaf(sgn, b.w, a.x);
            c[4 * q + 1] = fmaf(sgn, b.z, a.y);
            c[4 * q + 2] = fmaf(sgn, b.y, a.z);
            c[4 * q + 3] = fmaf(sgn, b.x, a.w);
        }
        if (w == 0) FastDct<Q>::dct2(c);
        else FastDct<Q>::dct4(c);
    } else {
        by_class(w, [&](auto CLS) { split_forward_inputs<S, CLS>(row, c); });
        if (w == 1) {
            FastDct<Q>::dct4(c);
        } else if constexpr (FUSED) {
            FastDct<Q>::dct2_open(c);
            if (w == 0) FastDct<Q>::dct2_close(c);
        } else {
            FastDct<Q>::dct2(c);
        }
    }
}

// W = 4: classes 2 and 3 hold A and B; after this class 2 holds the coefficients 4m+1 and
// class 3 the coefficients 4m+3.  The tile rows must be free; contains workgroup barriers,
// every wavefront calls it.
template <int S, bool FUSED = false>
__device__ __forceinline__ void split_forward_exchange(float* __restrict__ row, int w,
                                                       float (&c)[S / 4]) {
    constexpr int Q = S / 4;
    if (w >= 2) regs_to_lds<Q>(row + (w - 2) * Q, c);
    __syncthreads();
    if (w == 2) {
        // c[l] = A[l] + B[Q-l] for l >= 1
        float br[Q];
        lds_to_regs_reversed<Q>(row + Q, br);        // br[i] = B[Q-1-i]
        static_for<1, Q>([&](auto l) { c[l] = class_sum<Q, FUSED, l, Q - l>(c[l], br[l - 1]); });
    } else if (w == 3) {
        // c[l] = A[l+1] - B[Q-1-l] for l < Q-1, c[Q-1] = -B[0]
        float a[Q], d[Q];
        lds_to_regs<Q>(row, a);
        static_for<0, Q - 1>([&](auto l) {
            d[l] = class_difference<Q, FUSED, l + 1, Q - 1 - l>(a[l + 1], c[Q - 1 - l]);
        });
        d[Q - 1] = -c[0];
#pragma unroll
        for (int l = 0; l < Q; ++l) c[l] = d[l];
    }
    __syncthreads();
}

// Classes 2 and 3 (CLS) of the inverse of W = 4: the rotations of the pairs of odd coefficients, `other`
// being the other class's coefficients.  v[j] = coefficient 2j+1 of the chunk, v[2l] = class 2's c[l],
// v[2l+1] = class 3's c[l].  c[l] makes r[2l] and c[Q-1-l] makes r[2l+1].
template <int S, int CLS>
__device__ __forceinline__ void inverse_rotations(const float* __restrict__ other,
                                                  const float (&c)[S / 4], float (&r)[S / 4]) {
    constexpr int Q = S / 4, H = S / 2;
    static_assert(Q % 8 == 0, "whole blocks of eight pairs");
    static_for<0, Q / 8>([&](auto q) {
        const float4 fo = *reinterpret_cast<const float4*>(other + 4 * q);
        const float4 ro = *reinterpret_cast<const float4*>(other + Q - 4 - 4 * q);
        const float o[4] = {fo.x, fo.y, fo.z, fo.w};              // other[l]
        const float orv[4] = {ro.w, ro.z, ro.y, ro.x};            // other[Q-1-l]
        static_for<0, 8>([&](auto i) {
            constexpr int j = 8 * q + i;
            constexpr int l = j / 2, li = l - 4 * q;
            constexpr float cs = Rot<H, j>::c, sn = Rot<H, j>::s;
            // pair (v[j], v[H-1-j]): j even: (c2[l], c3[Q-1-l]); j odd: (c3[l], c2[Q-1-l])
            if constexpr (CLS == 2) {
                const float pj = (j % 2) ? o[li] : c[l];
                const float qj = (j % 2) ? c[Q - 1 - l] : orv[li];
                r[j] = fmaf(pj, cs, qj * sn);
            } else {
                const float pj = (j % 2) ? c[l] : o[li];
                const float qj = (j % 2) ? orv[li] : c[Q - 1 - l];
                const float bv = fmaf(qj, cs, -(pj * sn));
                r[j] = (j % 2) ? -bv : bv;
            }
        });
    });
}

// ---- inverse: the classes' scaled coefficients back into the rows as [E | O] (W = 2) or
// [E (2Q) | O even (Q) | O odd (Q)] (W = 4), ready for split_output.  Contains workgroup
// barriers; the rows must be free on entry.
template <int S, int W, bool FUSED = false>
__device__ __forceinline__ void split_inverse_to_rows(float* __restrict__ row, int w,
                                                      float (&c)[S / W]) {
    constexpr int Q = S / W;
    if constexpr (W == 2) {
        if (w == 0) FastDct<Q>::dct3(c);
        else FastDct<Q>::dct4(c);
        regs_to_lds<Q>(row + w * Q, c);
        __syncthreads();
    } else {
        // classes 2 and 3 exchange their coefficients
        constexpr int H = S / 2;
        if (w >= 2) regs_to_lds<Q>(row + H + (w - 2) * Q, c);
        __syncthreads();
        if (w == 0) {
            FastDct<Q>::dct3(c);
        } else if (w == 1) {
            FastDct<Q>::dct4(c);
        } else {
            float r[Q];
            if (w == 2) inverse_rotations<S, 2>(row + H + Q, c, r);
            else inverse_rotations<S, 3>(row + H, c, r);
            if constexpr (FUSED) FastDct<Q>::dct2_open(r);
            else FastDct<Q>::dct2(r);
#pragma unroll
            for (int j = 0; j < Q; ++j) c[j] = r[j];
        }
        __syncthreads();
        // EE | EO | A | B.  The results take the places of what they are made of, so that no second
        // array of Q is live: E[i] at c[i]; E[Q+m] at c[Q-1-m]; O[2l] at c[l]; O[2l+1] at c[Q-1-l]
        // (but for the sign of the last one, which the store turns.  Turned in the branch, by a bare
        // negation of c[0] after which nothing else is done to it, it is in the compiler's intermediate code
        // and missing in what ROCm 7.2 generates from it at chunk 192: structurising the branches it takes
        // the negation out of the last one as free, and that branch then merges the unturned value.)
        regs_to_lds<Q>(row + w * Q, c);
        __syncthreads();
        float o[Q];
        if (w == 0) {
            lds_to_regs<Q>(row + Q, o);
#pragma unroll
            for (int i = 0; i < Q; ++i) c[i] = c[i] + o[i];              // EE[i] + EO[i]
        } else if (w == 1) {
            lds_to_regs<Q>(row, o);
#pragma unroll
            for (int i = 0; i < Q; ++i) c[i] = o[i] - c[i];              // EE[i] - EO[i]
        } else if (w == 2) {
            lds_to_regs_reversed<Q>(row + 3 * Q, o);                     // o[i] = B[Q-1-i]
            static_for<1, Q>([&](auto l) {                               // A[l] + B[Q-l]
                c[l] = class_sum<Q, FUSED, l, Q - l>(c[l], o[l - 1]);
            });
        } else {
            lds_to_regs<Q>(row + 2 * Q, o);
            static_for<0, Q - 1>([&](auto l) {                           // A[l+1] - B[Q-1-l]
                c[Q - 1 - l] = class_difference<Q, FUSED, l + 1, Q - 1 - l>(o[l + 1], c[Q - 1 - l]);
            });
        }
        __syncthreads();
        if (w == 1) {
            reversed_range_to_lds<0, Q>(row + Q, c);
            DETO_KEEP_APART("upper half of E");
        } else if (w == 3) {
            reversed_range_to_lds<0, Q>(row + 3 * Q, c);
            row[4 * Q - 1] = -c[0];
            DETO_KEEP_APART("odd entries of O");
        } else {
            regs_to_lds<Q>(row + w * Q, c);
            DETO_KEEP_APART("lower half of E, even entries of O");
        }
        __syncthreads();
    }
}

// four consecutive elements col .. col+3 of the chunk whose row was left by
// split_inverse_to_rows
template <int S, int W>
__device__ __forceinline__ float4 split_output(const float* __restrict__ row, int col) {
    constexpr int H = S / 2;
    const bool upper = col >= H;
    const int n0 = upper ? S - 4 - col : col;     // elements col+i mirror n0+3-i when upper
    const float4 e = *reinterpret_cast<const float4*>(row + n0);
    float4 o;
    if constexpr (W == 2) {
        o = *reinterpret_cast<const float4*>(row + H + n0);
    } else {
        const float2 oe = *reinterpret_cast<const float2*>(row + H + n0 / 2);
        const float2 oo = *reinterpret_cast<const float2*>(row + H + H / 2 + n0 / 2);
        o = make_float4(oe.x, oo.x, oe.y, oo.y);
    }
    if (!upper) return make_float4(e.x + o.x, e.y + o.y, e.z + o.z, e.w + o.w);
    return make_float4(e.w - o.w, e.z - o.z, e.y - o.y, e.x - o.x);
}

// The Random scheme's kept places of one chunk: the first k steps of a Fisher-Yates shuffle of
// 0 .. S-1 in `places` (S bytes of LDS private to the calling lane), each place handed to `take`
// as it is drawn.  Only places[t] is written back: place j is never read again after step j.
// What bounds it is the LDS latency of a step (its write needs what it has read, the next step
// reads after it), so four steps read at once and settle among themselves in registers what an
// earlier one of the four has moved.
template <int S, class Take>
__device__ __forceinline__ void shuffle_places(uint64_t seed, uint64_t step, uint64_t chunk, int k,
                                               uint8_t* places, Take take) {
#pragma unroll
    for (int q = 0; q < S / 4; ++q)
        reinterpret_cast<uint32_t*>(places)[q] = 0x03020100u + 0x04040404u * q;
    const uint64_t key = chunk_key(seed, step, chunk);
    constexpr int kBatch = 4;
    for (int j = 0; j < k; j += kBatch) {
        uint32_t t[kBatch], pj[kBatch], pt[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            // (steps past the last one stay inside 0 .. S-1 and are not carried out: k <= S/2)
            t[i] = j + i + bounded(draw(key, j + i), S - j - i);
            pj[i] = places[j + i];
            pt[i] = places[t[i]];
        }
#pragma unroll
        for (int i = 1; i < kBatch; ++i) {
#pragma unroll
            for (int l = 0; l < i; ++l) {
                pj[i] = (t[l] == static_cast<uint32_t>(j + i)) ? pj[l] : pj[i];
                pt[i] = (t[l] == t[i]) ? pj[l] : pt[i];
            }
        }
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            if (j + i < k) {
                places[t[i]] = static_cast<uint8_t>(pj[i]);
                take(pt[i]);
            }
        }
    }
}

// Compress half (top-k, DCT domain, k <= S/2) on full tiles of 64 chunks; the chunks past the
// last full tile form one partial tile (one more workgroup).
// TOP > 0: for launches with k <= TOP (see the selection step).
// NARROW: any payload format, chosen at run time by p.val_dtype and p.idx_u8 (16-bit values or
// two-bit signs, byte or int32 indices); otherwise fp32 values and int32 indices.  Only the
// staging step (what a kept coefficient leaves behind) and the payload's way out look at the
// format, each behind one uniform branch, so one kernel serves all of them.
// SCHEME (with NARROW, TOP = 0): Striding or Random on the coefficients (p.scheme) instead of
// top-k: the kept sets do not depend on the values, so one wavefront shuffles all 64 chunks
// (Random) or every wavefront writes the same pattern (Striding).
// Occupancy: the workgroups of a CU are each in one phase at a time (barriers), so the number
// of workgroups per CU is what overlaps memory phases with arithmetic.  Chunk 192 with the
// partial sort fits three (168 registers, 52 KB of LDS with the lists of places in the mask words);
// chunk 256 two (a 64-row tile alone is 65 KB); chunk 96 / 128 four to six of two wavefronts.
// GANG: tiles in gangs (run_log2); fp32 values and int32 indices, top-k.
template <int S, int W, bool GRAD_BF16, int TOP = 0, bool NARROW = false, bool SCHEME = false,
          bool GANG = false>
__global__ __launch_bounds__(kWave * W)
__attribute__((amdgpu_waves_per_eu((S == 192 && TOP > 0) ? 3 : 2))) void compress_split(
    KParams p, int64_t tiles, int64_t n, int64_t n_chunks, const void* __restrict__ grad,
    float* __restrict__ mom, void* __restrict__ idx_out, void* __restrict__ val_out,
    float* __restrict__ coeff_dbg) {
    using G = SplitGeom<S, W>;
    constexpr int Q = G::Q, kRow = G::kRow, NW = G::NW, kThreads = G::kThreads;
    constexpr int kIdx0 = G::kIdx0, kTile = G::kTile;
    // (class_sum; chunk 64: two classes and four round alike, so the shard's size does not matter)
    constexpr bool kFused = W == 4 && (NARROW || S == 64) && !SCHEME;
    // a launch with the partial sort keeps few: their places are listed (payload staging), up to 16 of
    // a chunk in its row's padding, more in its mask words if these are as many bytes (chunk 192: 2 KB
    // more would cost one of three workgroups per CU, 60 M parameters 156 -> 190 us)
    constexpr bool kList = TOP > 0;
    constexpr bool kOwnPlaces = TOP > 16 && TOP > 4 * W * NW, kMaskPlaces = TOP > 16 && !kOwnPlaces;
    static_assert(!(kList && SCHEME), "the kept sets of top-k");
    __shared__ __attribute__((aligned(16))) float buf[kList ? G::kTile : G::kBufFloats];
    __shared__ __attribute__((aligned(16))) uint8_t s_places[kOwnPlaces ? kWave * TOP : 16];
    __shared__ __attribute__((aligned(16))) uint32_t s_mask[kWave][W][NW];   // kept sets: chunk, class, word
    auto places = [&](uint32_t r) -> uint8_t* {
        if constexpr (kOwnPlaces) return &s_places[r * TOP];
        else if constexpr (kMaskPlaces) return reinterpret_cast<uint8_t*>(s_mask[r]);
        else return reinterpret_cast<uint8_t*>(&buf[r * kRow + S]);
    };
    __shared__ uint8_t s_cnt[kWave][W];          // kept per class (at most Q <= 64)
    __shared__ unsigned long long s_tie;         // chunks of the tile that took the tie pass

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int k = p.k;

    // Workgroups [0, tiles): full tiles.  The chunks left over (fewer than 64, the last of them
    // possibly ragged: the shard need not end on a chunk boundary) form ONE partial tile: its
    // first `live` rows are chunks, the other lanes idle; positions past the end of the shard
    // read as zero and are never written.
    const int64_t tile = blockIdx.x;
    const bool partial = tile >= tiles;    // (a partial tile can have 64 rows, the last ragged)
    const int live = partial ? static_cast<int>(n_chunks - tiles * kWave) : kWave;
    const bool alive = lane < live;
    static_assert(!GANG || (!NARROW && !SCHEME), "one payload format");
    const TileRows rows = GANG ? tile_rows(tile, tiles, p.run_lg) : TileRows{tile * kWave, 0u, 6};
    const int64_t chunk0 = rows.first;
    const int64_t base = chunk0 * S;
    // where the thread's piece `it` of the tile (element 4 * (tid + kThreads * it)) is in an array
    auto piece = [&](auto* array, int it) {
        if constexpr (GANG) return array + (base + rows.quads<S>(4 * kWave * (w + W * it))) + 4u * lane;
        else return array + base + 4 * (tid + kThreads * it);
    };
    float* row = &buf[lane * kRow];
    if (tid == 0) s_tie = 0ull;

    // ---- m1 = beta*m + g for the tile's contiguous elements, coalesced, into the rows (the
    // rows past a partial tile's chunks become zero)
    {
        constexpr int kIt = Q / 4;               // 16-byte pieces per thread
        auto fold_piece = [&](int it) {
            const int e4 = 4 * (tid + kThreads * it);
            const int r = e4 / S, col = e4 - r * S;
            const float4 m = ld_f4<false>(piece(mom, it));
            float4 g;
            if constexpr (GRAD_BF16) {
                const uint2 gb = ld_u2<false>(piece(static_cast<const uint16_t*>(grad), it));
                g = make_float4(__uint_as_float(gb.x << 16), __uint_as_float(gb.x & 0xFFFF0000u),
                                __uint_as_float(gb.y << 16), __uint_as_float(gb.y & 0xFFFF0000u));
            } else {
                g = ld_f4<false>(piece(static_cast<const float*>(grad), it));
            }
            *reinterpret_cast<float4*>(&buf[r * kRow + col]) =
                make_float4(fmaf(p.beta, m.x, g.x), fmaf(p.beta, m.y, g.y),
                            fmaf(p.beta, m.z, g.z), fmaf(p.beta, m.w, g.w));
        };
        if (!partial) {
#pragma unroll
            for (int it = 0; it < kIt; ++it) fold_piece(it);
        } else {
            for (int it = 0; it < kIt; ++it) {
                const int e4 = 4 * (tid + kThreads * it);
                const int64_t i0 = base + e4;
                if (i0 + 3 < n) {
                    fold_piece(it);
                } else {
                    // the piece that straddles the end of the shard, and everything past it
                    const int r = e4 / S, col = e4 - r * S;
                    float x[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        x[j] = 0.0f;
                        if (i0 + j < n) {
                            const float g = GRAD_BF16
                                ? bf16_to_f32(static_cast<const uint16_t*>(grad)[i0 + j])
                                : static_cast<const float*>(grad)[i0 + j];
                            x[j] = fmaf(p.beta, mom[i0 + j], g);
                        }
                    }
                    *reinterpret_cast<float4*>(&buf[r * kRow + col]) =
                        make_float4(x[0], x[1], x[2], x[3]);
                }
            }
        }
    }
    __syncthreads();

    // ---- the lane's coefficients c[m] = coefficient W*m + off of chunk `lane`
    const int off = split_off<W>(w);
    float c[Q];
    split_forward_local<S, W, kFused>(row, w, c);
    __syncthreads();                              // every class has read the chunk: rows free
    if constexpr (W == 4) split_forward_exchange<S, kFused>(row, w, c);
    c[0] *= (w == 0) ? p.alpha0 : p.alpha;
#pragma unroll
    for (int m = 1; m < Q; ++m) c[m] *= p.alpha;
    if (coeff_dbg && alive) {
        float* dbg = coeff_dbg + (chunk0 + rows.chunk(lane)) * S + off;
#pragma unroll
        for (int m = 0; m < Q; ++m) dbg[W * m] = c[m];
    }

    uint32_t own[NW];     // this class's kept set: bit m = coefficient W*m + off
    int need = 0;         // entries equal to the threshold that a tied chunk still takes
    if constexpr (SCHEME) {
        if (p.scheme == 2) {
            // one wavefront, a lane per chunk (which one alternates, to spread over the SIMDs);
            // the chunk's free row holds the places that are being shuffled
            if (w == static_cast<int>(tile) % W) {
#pragma unroll
                for (int j = 0; j < W; ++j)
#pragma unroll
                    for (int i = 0; i < NW; ++i) s_mask[lane][j][i] = 0u;
                shuffle_places<S>(p.seed, p.step, static_cast<uint64_t>(chunk0 + lane), k,
                                  reinterpret_cast<uint8_t*>(row), [&](uint32_t at) {
                    atomicOr(&s_mask[lane][split_off<W>(at % W)][(at / W) / 32],
                             1u << ((at / W) % 32));
                });
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < NW; ++j) own[j] = s_mask[lane][w][j];
        } else {
            const int stride = S / k;
            int at = static_cast<int>(p.step % static_cast<uint64_t>(stride));
#pragma unroll
            for (int j = 0; j < NW; ++j) own[j] = 0u;
            for (int j = 0; j < k; ++j, at += stride) {
                const uint32_t bit = (at % W == off) ? 1u << ((at / W) % 32) : 0u;
#pragma unroll
                for (int i = 0; i < NW; ++i) own[i] |= ((at / W) / 32 == i) ? bit : 0u;
            }
#pragma unroll
            for (int j = 0; j < NW; ++j) s_mask[lane][w][j] = own[j];
            __syncthreads();
        }
    } else {
    // ---- k-th largest magnitude T of the chunk
    uint32_t T;
    {
        // (the magnitudes are formed again when the kept sets are marked: keeping these
        // copies alive across the sort would cost Q registers)
        uint32_t a[Q];
#pragma unroll
        for (int m = 0; m < Q; ++m) {
            a[m] = __float_as_uint(c[m]) & 0x7FFFFFFFu;
            asm volatile("" : "+v"(a[m]));
        }
        uint32_t* lists = reinterpret_cast<uint32_t*>(row);
        auto publish = [&]() {
#pragma unroll
            for (int q = 0; q < Q / 4; ++q)
                *reinterpret_cast<uint4*>(lists + w * Q + 4 * q) =
                    make_uint4(a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]);
        };
        // each class contributes at most k of the k largest: a launch with k <= TOP sorts out
        // only every lane's largest TOP (TOP = 0: the full sort)
        if constexpr (TOP > 0) sort_top_desc<Q, TOP>(a);
        else sort_desc<Q>(a);
        publish();
        __syncthreads();
        if constexpr (W == 4 && TOP > 0) {
            // only the TOP largest of each class are in the lists (k <= TOP): the TOP largest
            // of a pair of classes are the maxima of one list against the mirror image of the
            // other, a bitonic sequence that the even class of the pair sorts; the odd class
            // waits.  The pair's merged list has TOP entries.
            uint32_t x[TOP];
            if ((w & 1) == 0) {
                const uint32_t* mine = lists + w * Q;
                const uint32_t* partner = lists + (w + 1) * Q;
                static_for<0, TOP / 4>([&](auto q) {
                    const uint4 m4 = *reinterpret_cast<const uint4*>(mine + 4 * q);
                    const uint4 t = *reinterpret_cast<const uint4*>(partner + TOP - 4 - 4 * q);
                    x[4 * q] = max(m4.x, t.w);
                    x[4 * q + 1] = max(m4.y, t.z);
                    x[4 * q + 2] = max(m4.z, t.y);
                    x[4 * q + 3] = max(m4.w, t.x);
                });
                bitonic_merge_desc<TOP>(x);
            }
            __syncthreads();
            if ((w & 1) == 0) {
                uint32_t* merged = lists + (w >> 1) * 2 * Q;
#pragma unroll
                for (int q = 0; q < TOP / 4; ++q)
                    *reinterpret_cast<uint4*>(merged + 4 * q) =
                        make_uint4(x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]);
            }
            __syncthreads();
            T = kth_of_two_lists<TOP>(lists, lists + 2 * Q, k);
        } else if constexpr (W == 4) {
            // classes (0,1) and (2,3): the larger half of the two lists' union to the even
            // class, the smaller half to the odd one; each half is bitonic and is sorted in
            // place.  Lists are padded with zeros (the smallest magnitude) to a power of two
            // QP; the even class ends up with the QP largest, the odd one with the other
            // 2Q - QP followed by padding, so the pair's merged list has 2Q entries again.
            constexpr int QP = SortNet<Q>::P;
            const uint32_t* partner = lists + (w ^ 1) * Q;
            uint32_t x[QP];
            static_for<0, QP / 4>([&](auto q) {
                constexpr int j0 = QP - 4 - 4 * q;               // partner's entries j0 .. j0+3
                uint4 t = make_uint4(0u, 0u, 0u, 0u);
                if constexpr (j0 < Q) t = *reinterpret_cast<const uint4*>(partner + j0);
                const uint32_t theirs[4] = {t.w, t.z, t.y, t.x};  // partner[QP-1-i], i = 4q ..
                uint4 m4 = make_uint4(0u, 0u, 0u, 0u);            // own entries 4q .. 4q+3
                if constexpr (4 * q < Q) m4 = *reinterpret_cast<const uint4*>(lists + w * Q + 4 * q);
                const uint32_t mine[4] = {m4.x, m4.y, m4.z, m4.w};
                static_for<0, 4>([&](auto e) {
                    constexpr int i = 4 * q + e;
                    x[i] = (w & 1) ? min(mine[e], theirs[e]) : max(mine[e], theirs[e]);
                });
            });
            bitonic_merge_desc<QP>(x);
            __syncthreads();
            uint32_t* merged = lists + (w >> 1) * 2 * Q + ((w & 1) ? QP : 0);
            if ((w & 1) == 0) {
#pragma unroll
                for (int q = 0; q < QP / 4; ++q)
                    *reinterpret_cast<uint4*>(merged + 4 * q) =
                        make_uint4(x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]);
            } else {
#pragma unroll
                for (int q = 0; q < (2 * Q - QP) / 4; ++q)
                    *reinterpret_cast<uint4*>(merged + 4 * q) =
                        make_uint4(x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]);
            }
            __syncthreads();
            T = kth_of_two_lists<2 * Q>(lists, lists + 2 * Q, k);
        } else {
            T = kth_of_two_lists<Q>(lists, lists + Q, k);
        }
    }

    // ---- kept sets: magnitude >= T, unless more than k magnitudes reach T (a tie at the
    // threshold): then only those above T, and the chunk goes through the whole-wavefront
    // pass that adds the lowest indices among the equals
    auto mark = [&](uint32_t thr) -> int {
#pragma unroll
        for (int j = 0; j < NW; ++j) own[j] = 0u;
        auto mag = [&](int m) { return __float_as_uint(c[m]) & 0x7FFFFFFFu; };
        static_for<0, Q / 4>([&](auto I) {
            constexpr int m = Q - 4 - 4 * I;   // descending so that shifting lands bit m at m
            own[m / 32] = push_if_at_least(own[m / 32], mag(m + 3), mag(m + 2), mag(m + 1), mag(m), thr);
        });
        int cnt = 0;
#pragma unroll
        for (int j = 0; j < NW; ++j) {
            cnt += __popc(own[j]);
            s_mask[lane][w][j] = own[j];
        }
        s_cnt[lane][w] = static_cast<uint8_t>(cnt);
        __syncthreads();                          // also: every class is done with the lists
        int total = 0;
#pragma unroll
        for (int j = 0; j < W; ++j) total += s_cnt[lane][j];
        return total;
    };
    uint32_t thr_gt = T, thr_eq = 0xFFFFFFFFu;
    {
        const int cnt = mark(T);
        const bool tie = alive && cnt != k;      // the idle rows of a partial tile are all zero
        if (__syncthreads_or(tie ? 1 : 0)) {
            if (tie) {
                thr_gt = T + 1u;     // <= 0x80000000: no magnitude reaches that
                thr_eq = T;
            }
            const int above = mark(thr_gt);
            if (tie) need = k - above;
            // the tied chunks' coefficients in natural order in their rows, for wavefront 0
#pragma unroll
            for (int m = 0; m < Q; ++m) row[W * m + off] = c[m];
            __syncthreads();
            if (w == 0) {
                const unsigned long long tl = __ballot(need != 0);
                if (lane == 0) s_tie = tl;
                emit_tied_chunks<S, kWave>(buf, p, lane, need, thr_gt, thr_eq, rows, idx_out,
                                           val_out, nullptr);
            }
            __syncthreads();
            if (need != 0) {
#pragma unroll
                for (int m = 0; m < Q; ++m) c[m] = row[W * m + off];   // alpha_j * remainder
            }
            __syncthreads();
        }
    }

    }

    // ---- payload staging, remainder in (settled chunks).  The position of coefficient m of
    // this class is the number of kept coefficients of the chunk with a smaller index: the
    // class's own bits below m, and of another class w' its bits below m (+ 1 if that class's
    // offset is the smaller one).
    if constexpr (kList) {
        // k <= TOP: the coefficients go into the row class by class, and a lane goes through its kept
        // ones alone, writing down each one's index at its position.  The payload's threads take the values
        // out of the rows and leave there what stays in the momentum.  (The walk below is a quarter of the
        // kernel's vector instructions, 619 of 2,350 a wavefront at 128/16 with 16-bit values, and writes
        // to a dump slot at seven of eight steps; here a lane takes the steps of the fullest class of 64
        // chunks, about 9 there.  Compress, us, walk -> list: 10.8 M 128/16 fp16 34.9 -> 32.6, 128/4 33.8 ->
        // 30.9; fp32 5 M 64/5 17.6 -> 16.6, 1 M 64/1 8.1 -> 7.6, 64/8 8.9 -> 8.7; 60 M 96/3 fp16 133 -> 117,
        // 192/7 146 -> 135.  Large launches of 128 and two classes wait for memory either way.  A launch
        // without the partial sort keeps too many: its lanes would take as many steps as the walk.)
        regs_to_lds<Q>(row + w * Q, c);
        uint32_t others[W - 1][NW];
        uint32_t at = 0u;                             // (the classes' bits lined up as below)
#pragma unroll
        for (int o = 1; o < W; ++o) {
            const int wo = (w + o) % W;
            const uint32_t adj = split_off<W>(wo) < off ? 1u : 0u;
            uint32_t ow[NW];
#pragma unroll
            for (int j = 0; j < NW; ++j) ow[j] = s_mask[lane][wo][j];
            at += ow[0] & adj;
#pragma unroll
            for (int j = 0; j < NW; ++j)
                others[o - 1][j] = __builtin_amdgcn_alignbit((j + 1 < NW) ? ow[j + 1] : 0u, ow[j], adj);
        }
        if constexpr (kMaskPlaces) __syncthreads();
        if (need == 0 && alive) {
            uint8_t* out = places(lane);
#pragma unroll
            for (int j = 0; j < NW; ++j) {
                uint32_t left = own[j];
                while (left != 0u) {
                    const uint32_t m = __builtin_ctz(left);
                    const uint32_t low = (1u << m) - 1u;
                    uint32_t to = at;
#pragma unroll
                    for (int o = 0; o < W - 1; ++o) to += __popc(others[o][j] & low);
                    out[to] = static_cast<uint8_t>(W * (32 * j + m) + off);
                    ++at;
                    left &= left - 1u;
                }
#pragma unroll
                for (int o = 0; o < W - 1; ++o) at += __popc(others[o][j]);
            }
        }
    } else if (need == 0 && alive) {
        // the other classes' bits lined up with this class's steps, and counted into the start
        uint32_t plane0[NW], plane1[NW];
        uint32_t start = 0u;
#pragma unroll
        for (int j = 0; j < NW; ++j) plane0[j] = plane1[j] = 0u;
#pragma unroll
        for (int o = 1; o < W; ++o) {
            const int wo = (w + o) % W;
            const uint32_t adj = split_off<W>(wo) < off ? 1u : 0u;
            uint32_t ow[NW];
#pragma unroll
            for (int j = 0; j < NW; ++j) ow[j] = s_mask[lane][wo][j];
            start += ow[0] & adj;
#pragma unroll
            for (int j = 0; j < NW; ++j) {
                const uint32_t up = (j + 1 < NW) ? ow[j + 1] : 0u;
                const uint32_t sh = __builtin_amdgcn_alignbit(up, ow[j], adj);
                // add one-bit numbers into a two-bit counter per position
                const uint32_t carry = plane0[j] & sh;
                plane0[j] ^= sh;
                plane1[j] |= carry;
            }
        }
        char* lds = reinterpret_cast<char*>(buf);
        const uint32_t dump = static_cast<uint32_t>(sizeof(float)) * (kTile + tid);
        uint32_t at = static_cast<uint32_t>(sizeof(float)) * (lane * kRow + start);
        const int idx0 = off;
        // what a kept coefficient leaves behind: the rounding error of a 16-bit format, nothing
        // otherwise.  Both roundings are computed and one is picked: with a branch per format
        // around this loop the compiler hoists the loop's common part and keeps it live across
        // the branch (chunk 128: 193 registers instead of 128, two wavefronts per SIMD instead
        // of four)
        const bool as_bf16 = p.val_dtype == 1, as_f16 = p.val_dtype == 2;
        static_for<0, Q>([&](auto m) {
            const uint32_t kb = (own[m / 32] >> (m % 32)) & 1u;
            const uint32_t b0 = (plane0[m / 32] >> (m % 32)) & 1u;
            const bool keep = kb != 0u;
            const uint32_t a = keep ? at : dump;
            *reinterpret_cast<float*>(lds + a) = c[m];
            *reinterpret_cast<float*>(lds + a + sizeof(float) * kIdx0) =
                __int_as_float(idx0 + W * m);
            at += 4u * kb + 4u * b0;
            if constexpr (W == 4) at += 8u * ((plane1[m / 32] >> (m % 32)) & 1u);
            float left = 0.0f;
            if constexpr (NARROW) {
                float r = c[m];
                r = as_bf16 ? __uint_as_float(pack_bf16x2(c[m], 0.0f) << 16) : r;
                r = as_f16 ? f16_to_f32(f32_to_f16(c[m])) : r;
                left = c[m] - r;
            }
            c[m] = (keep ? left : c[m]) * ((m == 0 && w == 0) ? p.alpha0 : p.alpha);
        });
    }
    __syncthreads();
    {
        // the tile's 64*k entries, in order (contiguous in both payload arrays, or in gangs a run of chunks at a time)
        const uint32_t magic = entry_magic(k);
        const unsigned long long tie_chunks = s_tie;
        // entries e .. e+3 of the tile (k a multiple of 4: they belong to one chunk)
        // (gangs: entry e of row r is this many entries further on)
        auto further = [&](uint32_t r) -> uint32_t { return GANG ? rows.item(0u, r, k) : 0u; };
        auto store_index4 = [&](uint32_t e, const int4& i4) {
            if (SCHEME && !idx_out) return;       // not transmitted
            if (NARROW && p.idx_u8)
                *reinterpret_cast<uint32_t*>(static_cast<uint8_t*>(idx_out) + chunk0 * k + e) =
                    static_cast<uint32_t>(i4.x | (i4.y << 8) | (i4.z << 16) | (i4.w << 24));
            else
                st_u4<GANG>(static_cast<int32_t*>(idx_out) + chunk0 * k + e,
                             make_uint4(i4.x, i4.y, i4.z, i4.w));
        };
        // takes coefficient i of row r out of the row: what a kept one leaves behind there is the
        // rounding error of a 16-bit format, nothing otherwise
        auto take = [&](uint32_t r, uint32_t i) -> float {
            const uint32_t cls = W == 2 ? i & 1u : ((i & 1u) << 1) | ((i >> 1) & 1u);    // (split_off)
            float* from = &buf[r * kRow + cls * Q + i / W];
            const float v = *from;
            *from = NARROW ? v - payload_roundtrip(p.val_dtype, v) : 0.0f;
            return v;
        };
        if (k % 4 == 0) {
            const int quads = live * k / 4;                // 16-byte pieces of the tile
            for (int q = tid; q < quads; q += kThreads) {
                const uint32_t e = 4u * static_cast<uint32_t>(q);
                const uint32_t r = __umulhi(e, magic);     // chunk of the tile, k >= 4
                const uint32_t j = e - r * static_cast<uint32_t>(k);
                if ((tie_chunks >> r) & 1ull) continue;    // written by the tie pass
                const uint32_t to = e + further(r);
                float4 v;
                int4 i4;
                if constexpr (kList) {
                    const uint32_t four = *reinterpret_cast<const uint32_t*>(places(r) + j);
                    i4 = make_int4(four & 0xFFu, (four >> 8) & 0xFFu, (four >> 16) & 0xFFu, four >> 24);
                    v = make_float4(take(r, i4.x), take(r, i4.y), take(r, i4.z), take(r, i4.w));
                } else {
                    const float* src = &buf[r * kRow + j];
                    v = *reinterpret_cast<const float4*>(src);
                    const float4 iv = *reinterpret_cast<const float4*>(src + kIdx0);
                    i4 = make_int4(__float_as_int(iv.x), __float_as_int(iv.y), __float_as_int(iv.z),
                                   __float_as_int(iv.w));
                }
                if (!NARROW || p.val_dtype == 0) {
                    st_f4<GANG>(static_cast<float*>(val_out) + chunk0 * k + to, v);
                } else if (p.val_dtype != 3) {
                    uint2 h;
                    if (p.val_dtype == 1) {
                        h.x = pack_bf16x2(v.x, v.y);
                        h.y = pack_bf16x2(v.z, v.w);
                    } else {
                        h.x = f32_to_f16(v.x) | (static_cast<uint32_t>(f32_to_f16(v.y)) << 16);
                        h.y = f32_to_f16(v.z) | (static_cast<uint32_t>(f32_to_f16(v.w)) << 16);
                    }
                    *reinterpret_cast<uint2*>(static_cast<uint16_t*>(val_out) + chunk0 * k + to) = h;
                }
                store_index4(to, i4);
            }
        } else {
            // four entries of a lane could straddle two chunks (and the arrays need not be
            // 16-byte aligned): one entry per lane
            for (uint32_t e = tid; e < static_cast<uint32_t>(live * k); e += kThreads) {
                const uint32_t r = (k == 1) ? e : __umulhi(e, magic);
                const uint32_t j = e - r * static_cast<uint32_t>(k);
                if ((tie_chunks >> r) & 1ull) continue;
                const float* src = &buf[r * kRow + j];
                const int at = kList ? places(r)[j] : __float_as_int(src[kIdx0]);
                const float v = kList ? take(r, at) : src[0];
                if constexpr (NARROW) {
                    if (p.val_dtype != 3)
                        store_payload_value(val_out, chunk0 * k + e, p.val_dtype, v);
                    if (!SCHEME || idx_out)
                        store_payload_index(idx_out, chunk0 * k + e, p.idx_u8, at);
                } else {
                    static_cast<float*>(val_out)[chunk0 * k + e + further(r)] = v;
                    static_cast<int32_t*>(idx_out)[chunk0 * k + e + further(r)] = at;
                }
            }
        }
        if (SCHEME && p.val_dtype == 3) {
            // two-bit signs: a thread builds one 16-entry word from the staged values (the
            // tile's words are contiguous)
            const uint32_t nw = static_cast<uint32_t>(ternary_words_per_chunk(k));
            uint32_t* words = static_cast<uint32_t*>(val_out) + chunk0 * nw;
            for (uint32_t q = tid; q < live * nw; q += kThreads) {
                const uint32_t r = q / nw;
                const uint32_t j0 = 16u * (q - r * nw);
                if ((tie_chunks >> r) & 1ull) continue;
                const float* src = &buf[r * kRow + j0];
                uint32_t word = 0u;
#pragma unroll
                for (uint32_t v = 0; v < 4; ++v) {
                    const float4 x = *reinterpret_cast<const float4*>(src + 4 * v);
                    const float xs[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
                    for (uint32_t i = 0; i < 4; ++i) {
                        const uint32_t j = 4 * v + i;
                        if (j0 + j < static_cast<uint32_t>(k)) word |= ternary_code(xs[i]) << (2 * j);
                    }
                }
                words[q] = word;
            }
        }
    }
    __syncthreads();
    if constexpr (kList) {
        lds_to_regs<Q>(row + w * Q, c);
        if (need == 0) {                              // (a tied chunk's are scaled)
            c[0] *= (w == 0) ? p.alpha0 : p.alpha;
#pragma unroll
            for (int m = 1; m < Q; ++m) c[m] *= p.alpha;
        }
    }

    // ---- new momentum = inverse transform of the remainder
    split_inverse_to_rows<S, W, kFused>(row, w, c);
    {
        auto output4 = [&](int r, int col) -> float4 {
            return split_output<S, W>(&buf[r * kRow], col);
        };
        constexpr int kIt = Q / 4;
        if (!partial) {
            // (non-temporal: a program reads the new momentum only a step later.  Whole steps on
            // rotating buffers, without -> with: 11 M fp32 64/16 62.2 -> 60.7 us, 28 M 130.7 ->
            // 128.4, 16 M bf16 256/32 114.7 -> 113.1; 1 M, all of it in the caches, the same.  The
            // lane-per-chunk kernels lose by the same hint: 376 -> 405 us at 147 M parameters)
#pragma unroll 8
            for (int it = 0; it < kIt; ++it) {
                const int e4 = 4 * (tid + kThreads * it);
                const int r = e4 / S, col = e4 - r * S;
                st_f4<true>(piece(mom, it), output4(r, col));
            }
        } else {
            for (int it = 0; it < kIt; ++it) {
                const int e4 = 4 * (tid + kThreads * it);
                const int r = e4 / S, col = e4 - r * S;
                const int64_t i0 = base + e4;
                if (i0 + 3 < n) {
                    st_f4<false>(mom + i0, output4(r, col));
                } else if (i0 < n) {
                    const float4 y = output4(r, col);
                    const float v[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (i0 + j < n) mom[i0 + j] = v[j];
                }
            }
        }
    }
}

// One lane's piece of a replica's payload as it is loaded and until it is applied: VEC consecutive
// entries (four, or one where k is not a multiple of 4).  VAL: value format (0 fp32, 1 bf16,
// 2 fp16, 3 two-bit signs); U8: byte indices.
template <int VEC, int VAL, bool U8>
struct SplitPiece {
    static_assert(VEC == 1 || VEC == 4, "one entry or four");
    static constexpr int kIdxWords = U8 ? 1 : VEC;
    static constexpr int kValWords = (VAL == 0) ? VEC : ((VAL == 3 || VEC == 1) ? 1 : 2);
    uint32_t i[kIdxWords], v[kValWords];

    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int c = 0; c < kIdxWords; ++c) i[c] = 0u;
#pragma unroll
        for (int c = 0; c < kValWords; ++c) v[c] = 0u;
    }
    // entries ie .. / ve .. counted from the arrays' bases; word_byte: the byte with these
    // entries' signs
    __device__ __forceinline__ void load(const void* idx, int64_t ie, const void* val, int64_t ve,
                                         int64_t word_byte) {
        if constexpr (VEC == 4) {
            if constexpr (U8) {
                i[0] = ld_u1<true>(static_cast<const uint8_t*>(idx) + ie);
            } else {
                const uint4 t = ld_u4<true>(static_cast<const int32_t*>(idx) + ie);
                i[0] = t.x; i[1] = t.y; i[2] = t.z; i[3] = t.w;
            }
        } else {
            i[0] = U8 ? static_cast<uint32_t>(static_cast<const uint8_t*>(idx)[ie])
                      : static_cast<const uint32_t*>(idx)[ie];
        }
        load_values(val, ve, word_byte);
    }
    // The same from a uniform part u (and its byte uw) and a 32-bit one of the lane: a scalar base for
    // the access.
    __device__ __forceinline__ void load_from(const void* idx, int64_t iu, const void* val, int64_t vu,
                                              uint32_t e, int64_t wu, uint32_t word_byte) {
        load(static_cast<const char*>(idx) + iu * (U8 ? 1 : 4), e,
             static_cast<const char*>(val) + (VAL == 3 ? wu : vu * (VAL == 0 ? 4 : 2)), e, word_byte);
    }
    __device__ __forceinline__ void load_values(const void* val, int64_t ve, int64_t word_byte) {
        if constexpr (VEC == 4) {
            if constexpr (VAL == 0) {
                const uint4 t = ld_u4<true>(static_cast<const float*>(val) + ve);
                v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
            } else if constexpr (VAL == 3) {
                v[0] = static_cast<const uint8_t*>(val)[word_byte];
            } else {
                const uint2 t = ld_u2<true>(static_cast<const uint16_t*>(val) + ve);
                v[0] = t.x; v[1] = t.y;
            }
        } else {
            if constexpr (VAL == 0) v[0] = static_cast<const uint32_t*>(val)[ve];
            else if constexpr (VAL == 3) v[0] = static_cast<const uint8_t*>(val)[word_byte];
            else v[0] = static_cast<const uint16_t*>(val)[ve];
        }
    }
    // indices and values; j: the first entry's place in its chunk
    __device__ __forceinline__ void get(uint32_t j, uint32_t (&at)[VEC], float (&x)[VEC]) const {
#pragma unroll
        for (int c = 0; c < VEC; ++c)
            at[c] = (U8 && VEC == 4) ? (i[0] >> (8 * c)) & 0xFFu : i[U8 ? 0 : c];
        values(j, x);
    }
    __device__ __forceinline__ void values(uint32_t j, float (&x)[VEC]) const {
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
            if constexpr (VAL == 0) x[c] = __uint_as_float(v[c]);
            else if constexpr (VAL == 3) x[c] = ternary_decode(v[0], VEC == 4 ? c : (j & 3u));
            else x[c] = decode16<VAL>(static_cast<uint16_t>(v[VEC == 1 ? 0 : c / 2] >> (16 * (c & 1))));
        }
    }
};

// Scatter-add of R replicas' entries into `rows` (my_rows chunk rows of kRow floats that belong to
// the calling wavefront), replica after replica; entry0 / chunk0: the first entry / chunk of
// those rows.  A step = one batch of replicas for one group of 64 pieces of VEC entries, one
// piece per lane; the loads of the next step are requested before the present one is applied.
// Inside a group a replica's entries hit distinct accumulators when the indices of every lane,
// and the step from the previous lane, ascend strictly (what compress emits): a plain
// read-add-write then; LDS atomics otherwise (duplicates add; they cost about 3 cycles a lane).
// GANG: `rows` are the tile's rows row0 .., whose chunks `gang` knows (entry0 and chunk0 are those of its
// first one).
template <int S, int VEC, int VAL, bool U8, bool GANG>
__device__ __forceinline__ void split_scatter(const KParams& p, int lane, float* rows, int my_rows,
                                              const void* __restrict__ idx, int64_t idx_stride,
                                              const void* __restrict__ val, int64_t val_stride,
                                              int64_t entry0, int64_t chunk0, uint32_t magic,
                                              const TileRows& gang, int row0) {
    constexpr int kRow = S + 4;
    constexpr int kBatch = 4;                              // replicas per batch
    using Piece = SplitPiece<VEC, VAL, U8>;
    const int k = p.k;
    const int pieces = my_rows * k / VEC;                  // per replica
    const int chunk_bytes = 4 * ternary_words_per_chunk(k);
    const int n_batches = (p.R + kBatch - 1) / kBatch;
    const int steps = ((pieces + kWave - 1) / kWave) * n_batches;
    // entry number e of the wavefront's rows, its row and its place j in that row's chunk
    auto locate = [&](int t, bool& in, uint32_t& e, uint32_t& r, uint32_t& j) {
        const int q = (t / n_batches) * kWave + lane;
        in = q < pieces;
        e = VEC * static_cast<uint32_t>(in ? q : 0);
        if constexpr (VEC == 4) r = (k == 4) ? (e >> 2) : __umulhi(e, magic);
        else r = (k == 1) ? e : __umulhi(e, magic);
        j = e - r * static_cast<uint32_t>(k);
    };
    auto request = [&](int t, Piece (&b)[kBatch]) {
        bool in;
        uint32_t e, r, j;
        locate(t, in, e, r, j);
        const int r0 = (t % n_batches) * kBatch;
        const int64_t word_byte = (chunk0 + r) * chunk_bytes + j / 4;
        const uint32_t at = gang.item(row0 * k + e, row0 + r, k);
        const uint32_t byte = gang.item((row0 + r) * chunk_bytes + j / 4, row0 + r, chunk_bytes);
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            if (r0 + i < p.R && in) {
                const int64_t rep = r0 + i;
                if constexpr (GANG)
                    b[i].load_from(idx, rep * idx_stride + entry0, val, rep * val_stride + entry0, at,
                                   rep * val_stride * 4 + chunk0 * chunk_bytes, byte);
                else
                    b[i].load(idx, rep * idx_stride + entry0 + e, val,
                              rep * val_stride + entry0 + e, rep * val_stride * 4 + word_byte);
            } else {
                b[i].clear();
            }
        }
    };
    auto apply = [&](int t, const Piece (&b)[kBatch]) {
        bool in;
        uint32_t e, r, j;
        locate(t, in, e, r, j);
        const int r0 = (t % n_batches) * kBatch;
        const bool chunk_start = lane == 0 || j == 0u;
        float* arow = rows + r * kRow;
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            if (r0 + i < p.R) {
                uint32_t at[VEC];
                float v[VEC];
                b[i].get(j, at, v);
                // (what an index outside the chunk, or a lane without a piece, adds goes to the
                // row's padding; unsigned: a negative index is a large one)
#pragma unroll
                for (int c = 0; c < VEC; ++c)
                    at[c] = in ? min(at[c], static_cast<uint32_t>(S)) : static_cast<uint32_t>(S);
                // the previous lane's last index (a shift over the whole wavefront)
                const uint32_t prev = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
                    0, static_cast<int>(at[VEC - 1]), 0x138, 0xf, 0xf, false));
                bool asc = chunk_start || prev < at[0];
#pragma unroll
                for (int c = 1; c < VEC; ++c) asc = asc && at[c - 1] < at[c];
                if (__any(in && !asc)) {
#pragma unroll
                    for (int c = 0; c < VEC; ++c) atomicAdd(&arow[at[c]], v[c]);
                } else {
                    float old[VEC];
#pragma unroll
                    for (int c = 0; c < VEC; ++c) old[c] = arow[at[c]];
#pragma unroll
                    for (int c = 0; c < VEC; ++c) arow[at[c]] = old[c] + v[c];
                }
                wave_lds_sync();
            }
        }
    };
    Piece b0[kBatch], b1[kBatch];
    if (steps > 0) request(0, b0);
    for (int t = 0; t < steps; t += 2) {
        if (t + 1 < steps) request(t + 1, b1);
        apply(t, b0);
        if (t + 2 < steps) request(t + 2, b0);
        if (t + 1 < steps) apply(t + 1, b1);
    }
}

// The same without transmitted indices (Striding, Random): every replica kept the same places, so
// the R values of an entry are summed in registers, replica 0 first, and written to their
// place once.  place(r, j): the place of entry j of the wavefront's row r.
template <int S, int VEC, int VAL, class Place>
__device__ __forceinline__ void split_place_sums(const KParams& p, int lane, float* rows,
                                                 int my_rows, const void* __restrict__ val,
                                                 int64_t val_stride, int64_t entry0,
                                                 int64_t chunk0, uint32_t magic, Place place) {
    constexpr int kRow = S + 4;
    constexpr int kBatch = 8;                              // replicas requested at a time
    using Piece = SplitPiece<VEC, VAL, true>;
    const int k = p.k;
    const int pieces = my_rows * k / VEC;
    const int chunk_bytes = 4 * ternary_words_per_chunk(k);
    for (int q = lane; q < pieces; q += kWave) {
        const uint32_t e = VEC * static_cast<uint32_t>(q);
        const uint32_t r = (k == 1) ? e : __umulhi(e, magic);
        const uint32_t j = e - r * static_cast<uint32_t>(k);
        const int64_t word_byte = (chunk0 + r) * chunk_bytes + j / 4;
        float sum[VEC];
#pragma unroll
        for (int c = 0; c < VEC; ++c) sum[c] = 0.0f;
        for (int r0 = 0; r0 < p.R; r0 += kBatch) {
            Piece b[kBatch];
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                b[i].clear();
                const int64_t rep = r0 + i;
                if (rep < p.R)
                    b[i].load_values(val, rep * val_stride + entry0 + e,
                                     rep * val_stride * 4 + word_byte);
            }
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                float x[VEC];
                b[i].values(j, x);
#pragma unroll
                for (int c = 0; c < VEC; ++c) sum[c] += x[c];   // (zero past the last replica)
            }
        }
#pragma unroll
        for (int c = 0; c < VEC; ++c) rows[r * kRow + place(r, j + c)] = sum[c];
    }
}

// The same for two-bit signs of many replicas: a word of 16 entries per lane.
template <int S, class Place>
__device__ __forceinline__ void split_count_sums(const KParams& p, int lane, float* rows, int my_rows,
                                                 const void* __restrict__ val, int64_t val_stride,
                                                 int64_t chunk0, Place place) {
    const int k = p.k, nw = ternary_words_per_chunk(k);
    const uint32_t* words = static_cast<const uint32_t*>(val) + chunk0 * nw;
    for (int q = lane; q < my_rows * nw; q += kWave) {
        const SignCounts counts(words, q, val_stride, p.R);
        const int r = q / nw, j0 = 16 * (q - r * nw);
#pragma unroll
        for (int f = 0; f < 16; ++f)
            if (j0 + f < k) rows[r * (S + 4) + place(r, j0 + f)] = counts.sum(f);
    }
}

// Decompress-and-update half (transmitted indices, DCT domain) on full tiles of 64 chunks, W
// wavefronts per workgroup; NARROW as in compress_split.  SCHEME (with NARROW): Striding or Random on
// coefficients without transmitted indices; one wavefront shuffles all 64 chunks of the tile
// and lists their places in ascending order.
//
// Scatter-add: wavefront w owns the rows [64w/W, 64(w+1)/W) of the tile, so no two wavefronts
// ever add into the same accumulator and, inside a wavefront, LDS operations complete in program
// order: replica after replica, deterministic.  Two batches of four replicas are in flight per
// wavefront (the wavefronts of a workgroup are in this phase together, so what each keeps in
// flight decides how busy the memory is).  Then every class gathers its coefficients from
// the rows, the inverse transform runs as in compress_split, and all wavefronts stream the
// parameters (and the moments of Decoupled AdamW) through the update.
//
// AMSGRAD: Decoupled AdamW with the running maximum, in kernels of their own.  Its maximum is requested
// with the rest of its batch; beside the plain update in one kernel that sets aside 16 registers in
// every launch, and a copy of the loop without it nearly doubles the kernel.  us, as a copy with
// checks in the same kernel and like this: amsgrad, signs, bf16, 256/32 10 M 92, 70, 128/16 10 M 66,
// 57; fp32 64/8 2 M 17.7, 15.8; and the other launches: 64/20 signs 60 M SGD 122, 109, Random 32/5 60 M
// 90, 71, 16/3 signs 30 M 61, 57.
// GANG: tiles in gangs (run_log2), transmitted indices.  (80 registers are six wavefronts per SIMD, 81 five.)
// COUNT (with SCHEME): two-bit signs of many replicas, counted a word at a time (count_signs), in kernels of their own:
// in one kernel the words of a batch cost every other payload up to three wavefronts per SIMD (16/2: 50 registers, 71;
// 16/1 R = 16 1.2 M 5.8 us, 6.6).
template <int S, int W, bool PARAM_BF16, bool NARROW = false, bool SCHEME = false, bool AMSGRAD = false,
          bool GANG = false, bool COUNT = false>
__global__ __launch_bounds__(kWave * W)
__attribute__((amdgpu_waves_per_eu(GANG && S == 32 ? 6 : 1))) void decompress_split(
    KParams p, int64_t tiles, int64_t n, int64_t n_chunks, const void* __restrict__ idx,
    int64_t idx_stride, const void* __restrict__ val, int64_t val_stride,
    void* __restrict__ params, AdamPtrs ad, float* __restrict__ presign_dbg) {
    using G = SplitGeom<S, W>;
    constexpr int Q = G::Q, kRow = G::kRow, kThreads = G::kThreads, kTile = G::kTile;
    constexpr int kRowsPerWave = kWave / W;
    __shared__ __attribute__((aligned(16))) float buf[kTile];

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int k = p.k;

    // full tiles, then one partial tile of the chunks left over, the last of them possibly
    // ragged (as in compress_split)
    const int64_t tile = blockIdx.x;
    const bool partial = tile >= tiles;    // (a partial tile can have 64 rows, the last ragged)
    const int live = partial ? static_cast<int>(n_chunks - tiles * kWave) : kWave;
    // rows of this wavefront's share that are chunks
    const int my_rows = min(max(live - w * kRowsPerWave, 0), kRowsPerWave);
    static_assert(!GANG || (!SCHEME && !AMSGRAD), "transmitted indices");
    const TileRows gang = GANG ? tile_rows(tile, tiles, p.run_lg) : TileRows{tile * kWave, 0u, 6};
    const int64_t base = gang.first * S;
    // where the thread's piece `it` of the tile (element 4 * (tid + kThreads * it)) is, as a uniform part and
    // the lane's
    auto piece = [&](int it) -> int64_t {
        if constexpr (GANG) return base + gang.quads<S>(4 * kWave * (w + W * it));
        else return base + 4 * (tid + kThreads * it);
    };
    const uint32_t lane4 = GANG ? 4u * lane : 0u;
    float* row = &buf[lane * kRow];

    // ---- the tile's bf16 parameters, requested first: they are needed only after the
    // transform (plain update of a full tile.  fp32 parameters, or the moments of Decoupled
    // AdamW, held that long would cost a wavefront per SIMD in registers: they are loaded
    // where they are used)
    constexpr int kPieces = Q / 4;                // 4-element pieces of the tile per thread
    uint2 early[kPieces];
    const bool adam = AMSGRAD || p.adam;
    const bool params_early = PARAM_BF16 && !partial && !adam && (SCHEME || p.use_dct);
    if constexpr (PARAM_BF16) {
        if (params_early) {
#pragma unroll
            for (int it = 0; it < kPieces; ++it)
                early[it] = ld_u2<true>(static_cast<const uint16_t*>(params) + piece(it) + lane4);
        }
    }

    // ---- Random: the places of every chunk, ascending, as bytes (entry e of the tile at byte e)
    __shared__ __attribute__((aligned(16))) uint8_t s_places[SCHEME ? kWave * S / 2 : 4];
    __shared__ uint32_t s_bits[SCHEME ? kWave * (S / 32 > 0 ? S / 32 : 1) : 1];
    if constexpr (SCHEME) {
        if (p.scheme == 2) {
            if (w == static_cast<int>(tile) % W) {
                constexpr int kWords = S / 32 > 0 ? S / 32 : 1;
                uint32_t* bits = &s_bits[lane * kWords];
#pragma unroll
                for (int i = 0; i < kWords; ++i) bits[i] = 0u;
                shuffle_places<S>(p.seed, p.step, static_cast<uint64_t>(tile * kWave + lane), k,
                                  reinterpret_cast<uint8_t*>(row),
                                  [&](uint32_t at) { atomicOr(&bits[at / 32], 1u << (at % 32)); });
                uint8_t* out = &s_places[lane * k];
                for (int i = 0; i < kWords; ++i) {
                    uint32_t left = bits[i];
                    while (left) {
                        *out++ = static_cast<uint8_t>(32 * i + __ffs(left) - 1);
                        left &= left - 1u;
                    }
                }
            }
            __syncthreads();
        }
    }

    // ---- zero this wavefront's rows
    {
        float* mine = &buf[w * kRowsPerWave * kRow];
        for (int v = lane; v < kRowsPerWave * kRow / 4; v += kWave)
            *reinterpret_cast<float4*>(mine + 4 * v) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    wave_lds_sync();

    // ---- scatter-add of this wavefront's rows, replica after replica
    {
        const int64_t row0 = GANG ? gang.first : tile * kWave + w * kRowsPerWave;
        float* rows = &buf[w * kRowsPerWave * kRow];
        const uint32_t magic = entry_magic(k);
        // (the format is settled once, out here: a branch on it at every piece would cut the
        // loads and the additions of a batch apart)
        auto scatter = [&](auto val_tag, auto u8_tag) {
            constexpr int VAL = decltype(val_tag)::value;
            constexpr bool U8 = decltype(u8_tag)::value;
            if (k % 4 == 0)
                split_scatter<S, 4, VAL, U8, GANG>(p, lane, rows, my_rows, idx, idx_stride, val,
                                                   val_stride, row0 * k, row0, magic, gang,
                                                   GANG ? w * kRowsPerWave : 0);
            else
                split_scatter<S, 1, VAL, U8, GANG>(p, lane, rows, my_rows, idx, idx_stride, val,
                                                   val_stride, row0 * k, row0, magic, gang,
                                                   GANG ? w * kRowsPerWave : 0);
        };
        // Striding / Random without transmitted indices
        [[maybe_unused]] auto place_sums = [&](auto val_tag) {
            constexpr int VAL = decltype(val_tag)::value;
            const int stride = S / k;
            const int first = static_cast<int>(p.step % static_cast<uint64_t>(stride));
            const uint8_t* listed = &s_places[SCHEME ? w * kRowsPerWave * k : 0];
            auto place = [&](uint32_t r, uint32_t j) -> int {
                return p.scheme == 2 ? static_cast<int>(listed[r * k + j])
                                     : first + static_cast<int>(j) * stride;
            };
            if constexpr (COUNT)
                split_count_sums<S>(p, lane, rows, my_rows, val, val_stride, row0, place);
            else if (k % 4 == 0)
                split_place_sums<S, 4, VAL>(p, lane, rows, my_rows, val, val_stride, row0 * k, row0,
                                            magic, place);
            else
                split_place_sums<S, 1, VAL>(p, lane, rows, my_rows, val, val_stride, row0 * k, row0,
                                            magic, place);
        };
        using std::integral_constant;
        static_assert(!COUNT || SCHEME, "no transmitted indices");
        if constexpr (COUNT) {
            place_sums(integral_constant<int, 3>{});
        } else if constexpr (SCHEME) {
            if (p.val_dtype == 1) place_sums(integral_constant<int, 1>{});
            else if (p.val_dtype == 2) place_sums(integral_constant<int, 2>{});
            else if (p.val_dtype == 3) place_sums(integral_constant<int, 3>{});
            else place_sums(integral_constant<int, 0>{});
        } else if constexpr (!NARROW) {
            scatter(integral_constant<int, 0>{}, std::false_type{});
        } else {
            auto by_value = [&](auto u8_tag) {
                if (p.val_dtype == 1) scatter(integral_constant<int, 1>{}, u8_tag);
                else if (p.val_dtype == 2) scatter(integral_constant<int, 2>{}, u8_tag);
                else if (p.val_dtype == 3) scatter(integral_constant<int, 3>{}, u8_tag);
                else scatter(integral_constant<int, 0>{}, u8_tag);
            };
            if (p.idx_u8) by_value(std::true_type{});
            else by_value(std::false_type{});
        }
    }
    __syncthreads();

    // ---- the lane's class of the averaged coefficients: a[W*m + off] * alpha_j / R, and back
    // (transmitted indices in the raw domain: the rows hold the sums themselves)
    if (SCHEME || p.use_dct) {
        const int off = split_off<W>(w);
        const float scale = p.alpha * p.inv_R;
        float c[Q];
        const float* src = row + off;
#pragma unroll
        for (int m = 0; m < Q; ++m) c[m] = src[W * m] * scale;
        if (w == 0) c[0] = row[0] * (p.alpha0 * p.inv_R);
        __syncthreads();
        split_inverse_to_rows<S, W>(row, w, c);
    }
    // (the domain is settled outside the update loops: a branch in every piece would cut their
    // loads apart)
    auto output4 = [&](int e4, auto raw_tag) -> float4 {
        const int r = e4 / S, col = e4 - r * S;
        if constexpr (decltype(raw_tag)::value) {
            const float4 a = *reinterpret_cast<const float4*>(&buf[r * kRow + col]);
            return make_float4(a.x * p.inv_R, a.y * p.inv_R, a.z * p.inv_R, a.w * p.inv_R);
        } else {
            return split_output<S, W>(&buf[r * kRow], col);
        }
    };

    // ---- y out of the rows, optional sign, parameter update, coalesced; the parameters (and
    // moments) of a batch of iterations are requested before the first is used
    {
        constexpr int kIt = Q / 4;                // 16-byte pieces per thread
        // (fewer at a time where the LDS leaves room for more than two wavefronts per SIMD: eight
        // pieces of parameters and moments would hold over 200 registers)
        constexpr int kBatch = Q >= 64 ? 8 : (kIt % 4 == 0 ? 4 : (kIt % 3 == 0 ? 3 : 2));
        static_assert(kIt % kBatch == 0, "whole batches");
        // (full tiles run the code without the checks against the end of the shard: with them
        // the loads of a batch are no longer issued together)
        auto update = [&](auto guarded_tag, auto raw_tag) {
        constexpr bool kGuarded = decltype(guarded_tag)::value;
#pragma unroll 1
        for (int b0 = 0; b0 < kIt; b0 += kBatch) {
            float4 old4[kBatch], m4[kBatch], v4[kBatch], x4[AMSGRAD ? kBatch : 1];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                const int64_t u = piece(b0 + j), i = u + lane4;
                if constexpr (kGuarded) {
                    old4[j] = m4[j] = v4[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    if constexpr (AMSGRAD) x4[j] = old4[j];
                    if (i + 3 >= n) continue;   // the shard's end: handled below
                }
                if constexpr (PARAM_BF16) {
                    const uint2 pb = ld_u2<true>(static_cast<const uint16_t*>(params) + u + lane4);
                    old4[j] = make_float4(__uint_as_float(pb.x << 16),
                                          __uint_as_float(pb.x & 0xFFFF0000u),
                                          __uint_as_float(pb.y << 16),
                                          __uint_as_float(pb.y & 0xFFFF0000u));
                } else {
                    old4[j] = ld_f4<true>(static_cast<const float*>(params) + u + lane4);
                }
                if (adam) {
                    m4[j] = ld_f4<true>(ad.m + u + lane4);
                    v4[j] = ld_f4<true>(ad.v + u + lane4);
                    if constexpr (AMSGRAD) x4[j] = ld_f4<true>(ad.vmax + u + lane4);
                }
            }
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                const int e4 = 4 * (tid + kThreads * (b0 + j));
                const int64_t u = piece(b0 + j), i = u + lane4;
                if (kGuarded && i + 3 >= n) {
                    // the piece that straddles the end of the shard: element by element
                    if (i < n) {
                        const float4 y4 = output4(e4, raw_tag);
                        const float yv[4] = {y4.x, y4.y, y4.z, y4.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            if (i + e >= n) break;
                            if (presign_dbg) presign_dbg[i + e] = yv[e];
                            const float q = sign_or_self(yv[e], p.use_sign);
                            const float th = PARAM_BF16
                                ? bf16_to_f32(static_cast<const uint16_t*>(params)[i + e])
                                : static_cast<const float*>(params)[i + e];
                            float nw;
                            if (adam) {
                                float vm = AMSGRAD ? ad.vmax[i + e] : 0.0f;
                                nw = adamw_step<AMSGRAD>(p, th, q, ad.m[i + e], ad.v[i + e], vm);
                                if constexpr (AMSGRAD) ad.vmax[i + e] = vm;
                            } else {
                                nw = fmaf(-p.lr, q, th * p.wd_scale);
                            }
                            if constexpr (PARAM_BF16)
                                static_cast<uint16_t*>(params)[i + e] = f32_to_bf16(nw);
                            else
                                static_cast<float*>(params)[i + e] = nw;
                        }
                    }
                    continue;
                }
                const float4 y4 = output4(e4, raw_tag);
                if (presign_dbg) st_f4<false>(presign_dbg + u + lane4, y4);
                const float y[4] = {y4.x, y4.y, y4.z, y4.w};
                const float old[4] = {old4[j].x, old4[j].y, old4[j].z, old4[j].w};
                float nw[4];
                if (adam) {
                    float m[4] = {m4[j].x, m4[j].y, m4[j].z, m4[j].w};
                    float v[4] = {v4[j].x, v4[j].y, v4[j].z, v4[j].w};
                    float4 vm = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    if constexpr (AMSGRAD) vm = x4[j];
                    float x[4] = {vm.x, vm.y, vm.z, vm.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        nw[e] = adamw_step<AMSGRAD>(p, old[e], sign_or_self(y[e], p.use_sign), m[e],
                                                    v[e], x[e]);
                    st_f4<true>(ad.m + u + lane4, make_float4(m[0], m[1], m[2], m[3]));
                    st_f4<true>(ad.v + u + lane4, make_float4(v[0], v[1], v[2], v[3]));
                    if constexpr (AMSGRAD) st_f4<true>(ad.vmax + u + lane4, make_float4(x[0], x[1], x[2], x[3]));
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        nw[e] = fmaf(-p.lr, sign_or_self(y[e], p.use_sign), old[e] * p.wd_scale);
                }
                if constexpr (PARAM_BF16) {
                    uint2 o;
                    o.x = pack_bf16x2(nw[0], nw[1]);
                    o.y = pack_bf16x2(nw[2], nw[3]);
                    st_u2<true>(static_cast<uint16_t*>(params) + u + lane4, o);
                } else {
                    st_f4<true>(static_cast<float*>(params) + u + lane4,
                                make_float4(nw[0], nw[1], nw[2], nw[3]));
                }
            }
        }
        };
        auto update_early = [&] {
#pragma unroll
            for (int it = 0; it < kPieces; ++it) {
                const int e4 = 4 * (tid + kThreads * it);
                const int64_t u = piece(it);
                const float4 y4 = output4(e4, std::false_type{});
                if (presign_dbg) st_f4<false>(presign_dbg + u + lane4, y4);
                const float y[4] = {y4.x, y4.y, y4.z, y4.w};
                const float old[4] = {__uint_as_float(early[it].x << 16),
                                      __uint_as_float(early[it].x & 0xFFFF0000u),
                                      __uint_as_float(early[it].y << 16),
                                      __uint_as_float(early[it].y & 0xFFFF0000u)};
                float nw[4];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    nw[e] = fmaf(-p.lr, sign_or_self(y[e], p.use_sign), old[e] * p.wd_scale);
                uint2 o;
                o.x = pack_bf16x2(nw[0], nw[1]);
                o.y = pack_bf16x2(nw[2], nw[3]);
                st_u2<true>(static_cast<uint16_t*>(params) + u + lane4, o);
            }
        };
        if (params_early) {
            update_early();
        } else {
            // (nothing is in flight here, but to the compiler the early parameters may be: without
            // this it waits between the loads of a batch that share registers with them.  vmcnt(0);
            // AdamW, bf16 parameters, us, without and with it: Random 256/32 30 M 140, 134; top-k 32/8
            // 1 M 9.0, 8.2, 32/2 with 8 replicas 9.4, 8.3.  Not below chunk 192 without indices: Random and
            // Striding 32/16 80 M 258, 272, 32/4 147 M 519, 532)
            if constexpr (PARAM_BF16 && !AMSGRAD && (!SCHEME || S >= 192))
                __builtin_amdgcn_s_waitcnt(0x0F70);
            if (!SCHEME && !p.use_dct) {
                // (transmitted indices in the raw domain: rare, one copy of the loop with the checks)
                update(std::true_type{}, std::integral_constant<bool, !SCHEME>{});
            } else if (partial) {
                update(std::true_type{}, std::false_type{});
            } else {
                update(std::false_type{}, std::false_type{});
            }
        }
    }
}

}  // namespace deto
