// Top-k compress at chunk 256, k <= 32: a lane per chunk and a wavefront per coefficient class as in
// split_kernels.hip.h (four classes of Q = 64 coefficients), with half of the tile in LDS at a time.
//
// Why halves: a tile of 64 chunks is 65 KB, and two workgroups per CU were all that fit; the vector
// units then ran two thirds of the time and the memory waited with them.  Everything that goes through
// LDS can go in two halves: the transform's inputs (n, S-1-n and the mirror images of both in the
// chunk's halves meet, so a half is n < Q/2), the exchanges between the classes, the coefficients
// (class-major, so a half is the indices below S/2), and the inverse's outputs.  A workgroup is then
// 38 KB; what bounds occupancy are the registers that hold a class's coefficients, three wavefronts
// per SIMD.  (At chunk 96, 128 and 192 those allow what the whole tile allows or one more, and the
// added barriers cost more than it gives: 67 M parameters, 192/24 195 -> 259 us, 128/16 151 -> 184.)
//
// Why a list of places instead of a walk over the coefficients: seven of eight steps of that walk
// write to a dump slot.  Here a chunk's kept set becomes S/32 mask words in index order (one atomic OR
// per class and word), a thread per word lists its set bits as bytes, and the payload's threads (four
// consecutive entries each) gather the values from the parked coefficients and leave behind what stays
// in the momentum.  A tie at the threshold is settled in the words: the lowest of the equal places
// fill up what is left to k.
//
// The arithmetic is that of compress_split, operation by operation, so its results keep their bits
// (the sign of a NaN aside, as fp16 values that overflow leave them in the momentum).
// Measured, compress alone, us, compress_split (whole tiles) and this kernel: 67 M parameters, bf16
// gradients 256/32 212 and 172, 256/8 204 and 151; 10.8 M fp32 256/32 53 and 45, with fp16 + byte indices
// 55 and 43; 1.2 M 22 and 22.
#pragma once

#include "split_kernels.hip.h"

namespace deto {

// (S: chunk size, W: classes, Q: coefficients per lane, H: S/2, L: half a class)
struct HalfGeom {
    static constexpr int S = 256, W = 4;
    static constexpr int Q = S / W, H = S / 2, L = Q / 2;
    static constexpr int kThreads = kWave * W;
    static constexpr int kRow = H + 4;                   // odd multiple of 4: 16 rows hit all banks
    static constexpr int kWords = S / 32;                // mask words of a chunk, in index order
    static constexpr int kWordRow = kWords | 1;
    static constexpr int NW = Q / 32;                    // mask words of a class
};

// The TOP largest magnitudes (bit patterns) of a class, descending: sort_top_desc on magnitudes that
// are formed group by group, so that no more than 2 TOP keys are live beside c.
template <int Q, int TOP>
__device__ __forceinline__ void largest_magnitudes(const float (&c)[Q], uint32_t (&a)[TOP]) {
    static_assert(Q % TOP == 0, "whole groups");
    static_for<0, Q / TOP>([&](auto g) {
        uint32_t x[TOP];
#pragma unroll
        for (int m = 0; m < TOP; ++m) {
            x[m] = __float_as_uint(c[g * TOP + m]) & 0x7FFFFFFFu;
            asm volatile("" : "+v"(x[m]));                 // (not formed again where c is used)
        }
        sort_desc<TOP>(x);
#pragma unroll
        for (int m = 0; m < TOP; ++m)                      // the larger of each and its mirror image:
            a[m] = g == 0 ? x[m] : max(a[m], x[TOP - 1 - m]);   // a bitonic sequence
        if constexpr (g > 0) bitonic_merge_desc<TOP>(a);
        __builtin_amdgcn_sched_barrier(0);
    });
}

// bit m of x (m < 8) to bit 4m
__device__ __forceinline__ uint32_t spread8(uint32_t x) {
    x = (x | (x << 12)) & 0x000F000Fu;
    x = (x | (x << 6)) & 0x03030303u;
    return (x | (x << 3)) & 0x11111111u;
}

// Half P of class CLS's transform inputs, from a row that holds the pieces of half P (load_place): what
// split_forward_local does for q in [P Q/8, (P+1) Q/8).
template <int P, int CLS>
__device__ __forceinline__ void half_forward_inputs(const float* __restrict__ row,
                                                    float (&c)[HalfGeom::Q]) {
    constexpr int Q = HalfGeom::Q, H = HalfGeom::H, L = HalfGeom::L;
    static_for<0, Q / 8>([&](auto qq) {
        constexpr int q = P * (Q / 8) + qq;
        const float4 f0 = *reinterpret_cast<const float4*>(row + 4 * qq);
        const float4 r2 = *reinterpret_cast<const float4*>(row + 2 * L - 4 - 4 * qq);
        const float4 f3 = *reinterpret_cast<const float4*>(row + 2 * L + 4 * qq);
        const float4 r1 = *reinterpret_cast<const float4*>(row + 4 * L - 4 - 4 * qq);
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

// Where element column `col` of a chunk goes before the transform: its half and its place in the row.
// half_forward_inputs reads four segments of L floats, ascending columns inside each: n, the ones
// below S/2, those from S/2 on, and S-1-n; half 0 is the blocks 0, 3, 4 and 7 of L columns.
__device__ __forceinline__ int load_place(int col, int& half) {
    constexpr int L = HalfGeom::L;
    const int block = col / L;
    half = (block & 1) ^ ((block >> 1) & 1);
    return (block >> 1) * L + col % L;
}

// Inverse, up to the outputs' even and odd parts in registers (what split_inverse_to_rows leaves in the
// rows): classes 0 and 1 the two halves of E (1: back to front), 2 and 3 the even and the odd entries
// of O (3: back to front, O's last entry with the other sign).  On entry a lane may still be reading its
// own quarter of its row; on return the rows are free.
template <bool FUSED>
__device__ __forceinline__ void half_inverse(float* __restrict__ row, int w, float (&c)[HalfGeom::Q]) {
    constexpr int Q = HalfGeom::Q, L = HalfGeom::L;
    __syncthreads();
    if (w >= 2) regs_to_lds<Q>(row + (w - 2) * Q, c);
    __syncthreads();
    if (w == 0) {
        FastDct<Q>::dct3(c);
    } else if (w == 1) {
        FastDct<Q>::dct4(c);
    } else {
        float r[Q];
        if (w == 2) inverse_rotations<HalfGeom::S, 2>(row + Q, c, r);
        else inverse_rotations<HalfGeom::S, 3>(row, c, r);
        if constexpr (FUSED) FastDct<Q>::dct2_open(r);
        else FastDct<Q>::dct2(r);
#pragma unroll
        for (int j = 0; j < Q; ++j) c[j] = r[j];
    }
    __syncthreads();
    // EE, EO, A and the upper half of B; then the other halves (B[Q-l] faces A[l]).  The results
    // take the places of what they are made of, so that no second array of Q is live:
    // E[i] at c[i]; E[Q+m] at c[Q-1-m]; O[2l] at c[l]; O[2l+1] at c[Q-1-l].
    float o[L];
    if (w == 3) {
        regs_range_to_lds<L, Q>(row + 3 * L, c);
        DETO_KEEP_APART("upper half of B");
    } else {
        regs_range_to_lds<0, L>(row + w * L, c);
        DETO_KEEP_APART("lower half");
    }
    __syncthreads();
    float middle = 0.0f;                              // O[Q]: c[L] is still to be published
    if (w == 0) {
        lds_to_regs<L>(row + L, o);
#pragma unroll
        for (int i = 0; i < L; ++i) c[i] = c[i] + o[i];               // EE[i] + EO[i]
    } else if (w == 1) {
        lds_to_regs<L>(row, o);
#pragma unroll
        for (int i = 0; i < L; ++i) c[i] = o[i] - c[i];               // EE[i] - EO[i]
    } else if (w == 2) {
        lds_to_regs_reversed<L>(row + 3 * L, o);                      // o[i] = B[Q-1-i]
        static_for<1, L>([&](auto l) {
            c[l] = class_sum<Q, FUSED, l, Q - l>(c[l], o[l - 1]);
        });
        middle = class_sum<Q, FUSED, L, Q - L>(c[L], o[L - 1]);
    } else {
        lds_to_regs<L>(row + 2 * L, o);                               // o[i] = A[i]
        static_for<0, L - 1>([&](auto l) {
            c[Q - 1 - l] = class_difference<Q, FUSED, l + 1, Q - 1 - l>(o[l + 1], c[Q - 1 - l]);
        });
    }
    __syncthreads();
    if (w == 3) {
        regs_range_to_lds<0, L>(row + 3 * L, c);
        DETO_KEEP_APART("lower half of B");
    } else {
        regs_range_to_lds<L, Q>(row + w * L, c);
        DETO_KEEP_APART("upper half");
    }
    __syncthreads();
    if (w == 0) {
        lds_to_regs<L>(row + L, o);
#pragma unroll
        for (int i = 0; i < L; ++i) c[L + i] = c[L + i] + o[i];
    } else if (w == 1) {
        lds_to_regs<L>(row, o);
#pragma unroll
        for (int i = 0; i < L; ++i) c[L + i] = o[i] - c[L + i];
    } else if (w == 2) {
        lds_to_regs_reversed<L>(row + 3 * L, o);                      // o[i] = B[L-1-i]
        static_for<L + 1, Q>([&](auto l) {
            c[l] = class_sum<Q, FUSED, l, Q - l>(c[l], o[l - 1 - L]);
        });
        c[L] = middle;
    } else {
        lds_to_regs<L>(row + 2 * L, o);                               // o[i] = A[L+i]
        static_for<L - 1, Q - 1>([&](auto l) {
            c[Q - 1 - l] =
                class_difference<Q, FUSED, l + 1, Q - 1 - l>(o[l + 1 - L], c[Q - 1 - l]);
        });
        // (c[0] stays B[0] = -O[2Q-1]: half_outputs_to_rows turns its sign)
    }
    __syncthreads();
}

// Half P of that into the rows: entries [P Q, (P+1) Q) of E, then [P L, (P+1) L) of the even and the
// same of the odd entries of O.
template <int P>
__device__ __forceinline__ void half_outputs_to_rows(float* __restrict__ row, int w,
                                                     const float (&c)[HalfGeom::Q]) {
    constexpr int Q = HalfGeom::Q, L = HalfGeom::L;
    if (w == 2) {
        regs_range_to_lds<P * L, (P + 1) * L>(row + 2 * L, c);
        DETO_KEEP_APART("even entries of O");
    } else if (w == 3) {
        reversed_range_to_lds<(1 - P) * L, (2 - P) * L>(row + 3 * L, c);
        if constexpr (P == 1) row[4 * L - 1] = -c[0];
        DETO_KEEP_APART("odd entries of O");
    } else if (w == P) {
        if constexpr (P == 0) regs_to_lds<Q>(row, c);
        else reversed_range_to_lds<0, Q>(row, c);
        DETO_KEEP_APART("half of E");
    }
}

// Top-k compress, k <= TOP.  NARROW as in compress_split.
template <bool GRAD_BF16, int TOP, bool NARROW>
__global__ __launch_bounds__(HalfGeom::kThreads) __attribute__((amdgpu_waves_per_eu(3))) void
compress_halves(
    KParams p, int64_t tiles, int64_t n, int64_t n_chunks, const void* __restrict__ grad,
    float* __restrict__ mom, void* __restrict__ idx_out, void* __restrict__ val_out,
    float* __restrict__ coeff_dbg) {
    using G = HalfGeom;
    constexpr int S = G::S, W = G::W, Q = G::Q, H = G::H, L = G::L, NW = G::NW;
    constexpr int N = TOP / W;                             // payload entries per thread
    static_assert(N % 4 == 0 && W * TOP <= H, "whole quads; the classes' sorted lists in the row");
    constexpr int kRow = G::kRow, kThreads = G::kThreads, kWords = G::kWords, kWordRow = G::kWordRow;
    constexpr bool kFused = NARROW;                        // (class_sum)
    __shared__ __attribute__((aligned(16))) float buf[kWave * kRow];
    __shared__ uint32_t s_kept[kWave * kWordRow];          // kept places of a chunk, index order
    __shared__ __attribute__((aligned(16))) uint8_t s_places[kWave * TOP];   // entry e of the tile

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int k = p.k;
    // full tiles, then one partial tile of the chunks left over (as in compress_split)
    const int64_t tile = blockIdx.x;
    const bool partial = tile >= tiles;
    const int live = partial ? static_cast<int>(n_chunks - tiles * kWave) : kWave;
    const int64_t base = tile * static_cast<int64_t>(kWave * S);
    const int64_t chunk0 = tile * kWave;
    float* row = &buf[lane * kRow];

    for (int q = tid; q < kWave * kWordRow; q += kThreads) s_kept[q] = 0u;

    // ---- m1 = beta*m + g, requested in whole, into the rows half by half; a thread's pieces of half P
    // are P Q/8 ... (P+1) Q/8 - 1
    float c[Q];
    {
        float4 x[Q / 4];
        if (!partial) {
            float4 m4[Q / 4], g4[Q / 4];
            uint2 gb[Q / 4];
#pragma unroll
            for (int v = 0; v < Q / 4; ++v) {
                const int64_t e = base + 4 * (tid + kThreads * v);
                m4[v] = ld_f4<false>(mom + e);
                if constexpr (GRAD_BF16) gb[v] = ld_u2<false>(static_cast<const uint16_t*>(grad) + e);
                else g4[v] = ld_f4<false>(static_cast<const float*>(grad) + e);
            }
#pragma unroll
            for (int v = 0; v < Q / 4; ++v) {
                if constexpr (GRAD_BF16)
                    g4[v] = make_float4(__uint_as_float(gb[v].x << 16),
                                        __uint_as_float(gb[v].x & 0xFFFF0000u),
                                        __uint_as_float(gb[v].y << 16),
                                        __uint_as_float(gb[v].y & 0xFFFF0000u));
                x[v] = make_float4(fmaf(p.beta, m4[v].x, g4[v].x), fmaf(p.beta, m4[v].y, g4[v].y),
                                   fmaf(p.beta, m4[v].z, g4[v].z), fmaf(p.beta, m4[v].w, g4[v].w));
            }
        } else {
#pragma unroll
            for (int v = 0; v < Q / 4; ++v) {
                const int64_t e = base + 4 * (tid + kThreads * v);
                float y[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    y[j] = 0.0f;
                    if (e + j < n) {
                        const float g = GRAD_BF16
                            ? bf16_to_f32(static_cast<const uint16_t*>(grad)[e + j])
                            : static_cast<const float*>(grad)[e + j];
                        y[j] = fmaf(p.beta, mom[e + j], g);
                    }
                }
                x[v] = make_float4(y[0], y[1], y[2], y[3]);
            }
        }
        // (dealt to the threads as they lie in memory: a thread's pieces all have the same column,
        // hence the same half)
        static_for<0, 2>([&](auto P) {
            if constexpr (P == 1) __syncthreads();
#pragma unroll
            for (int v = 0; v < Q / 4; ++v) {
                const int e4 = 4 * (tid + kThreads * v);
                const int r = e4 / S;
                int half;
                const int at = load_place(e4 - r * S, half);
                if (half == P) *reinterpret_cast<float4*>(&buf[r * kRow + at]) = x[v];
            }
            __syncthreads();
            by_class(w, [&](auto CLS) { half_forward_inputs<P, CLS>(row, c); });
        });
    }
    // ---- the lane's class of coefficients
    if (w == 1) {
        FastDct<Q>::dct4(c);
    } else if constexpr (kFused) {
        FastDct<Q>::dct2_open(c);
        if (w == 0) FastDct<Q>::dct2_close(c);
    } else {
        FastDct<Q>::dct2(c);
    }
    __syncthreads();
    split_forward_exchange<S, kFused>(row, w, c);
    const int off = split_off<W>(w);
    c[0] *= (w == 0) ? p.alpha0 : p.alpha;
#pragma unroll
    for (int m = 1; m < Q; ++m) c[m] *= p.alpha;
    if (coeff_dbg && lane < live) {
        float* dbg = coeff_dbg + (chunk0 + lane) * S + off;
#pragma unroll
        for (int m = 0; m < Q; ++m) dbg[W * m] = c[m];
    }

    // ---- k-th largest magnitude T of the chunk
    uint32_t T;
    {
        uint32_t a[TOP];
        largest_magnitudes<Q, TOP>(c, a);
        uint32_t* lists = reinterpret_cast<uint32_t*>(row);
        auto publish = [&](uint32_t* to) {
#pragma unroll
            for (int q = 0; q < TOP / 4; ++q)
                *reinterpret_cast<uint4*>(to + 4 * q) =
                    make_uint4(a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]);
        };
        // the odd class of a pair hands its list to the even one, which folds it into its own
        if (w & 1) publish(lists + w * TOP);
        __syncthreads();
        if ((w & 1) == 0) {
            const uint32_t* partner = lists + (w + 1) * TOP;
            static_for<0, TOP / 4>([&](auto q) {
                const uint4 t = *reinterpret_cast<const uint4*>(partner + TOP - 4 - 4 * q);
                a[4 * q] = max(a[4 * q], t.w);
                a[4 * q + 1] = max(a[4 * q + 1], t.z);
                a[4 * q + 2] = max(a[4 * q + 2], t.y);
                a[4 * q + 3] = max(a[4 * q + 3], t.x);
            });
            bitonic_merge_desc<TOP>(a);
            publish(lists + w * TOP);
        }
        __syncthreads();
        T = kth_of_two_lists<TOP>(lists, lists + 2 * TOP, k);
    }

    // ---- kept sets as mask words in index order
    auto publish_bits = [&](uint32_t* words, const uint32_t (&own)[NW]) {
#pragma unroll
        for (int i = 0; i < kWords; ++i)
            atomicOr(&words[lane * kWordRow + i],
                     spread8((own[i / 4] >> (8 * (i % 4))) & 0xFFu) << off);
    };
    {
        uint32_t own[NW];
#pragma unroll
        for (int j = 0; j < NW; ++j) own[j] = 0u;
        const float thr = __uint_as_float(T);
        static_for<0, Q / 2>([&](auto I) {
            constexpr int m = Q - 2 - 2 * I;   // descending so that shifting lands bit m at m
            own[m / 32] = push_unless_below(own[m / 32], c[m + 1], c[m], thr);
        });
        publish_bits(s_kept, own);
    }
    __syncthreads();                                       // (also: the lists are free)
    // the chunk `lane`'s words; this wavefront lists words w, w + W, ...
    uint32_t word[kWords];
    int total = 0;
#pragma unroll
    for (int i = 0; i < kWords; ++i) {
        word[i] = s_kept[lane * kWordRow + i];
        total += __popc(word[i]);
    }
    if (__syncthreads_or(lane < live && total != k)) {
        // a tie: the places above T, and those at T in words of their own
        uint32_t* s_equal = reinterpret_cast<uint32_t*>(buf);
        for (int q = tid; q < kWave * kWordRow; q += kThreads) s_kept[q] = s_equal[q] = 0u;
        __syncthreads();
        uint32_t above[NW], equal[NW];
#pragma unroll
        for (int j = 0; j < NW; ++j) above[j] = equal[j] = 0u;
        static_for<0, Q>([&](auto m) {
            const uint32_t mag = __float_as_uint(c[m]) & 0x7FFFFFFFu;
            above[m / 32] |= mag > T ? 1u << (m % 32) : 0u;
            equal[m / 32] |= mag == T ? 1u << (m % 32) : 0u;
        });
        publish_bits(s_kept, above);
        publish_bits(s_equal, equal);
        __syncthreads();
        int need = k;
#pragma unroll
        for (int i = 0; i < kWords; ++i) need -= __popc(s_kept[lane * kWordRow + i]);
#pragma unroll
        for (int i = 0; i < kWords; ++i) {
            uint32_t e = s_equal[lane * kWordRow + i];
            word[i] = s_kept[lane * kWordRow + i];
            while (e != 0u && need > 0) {                  // the lowest ones
                word[i] |= e & (0u - e);
                e &= e - 1u;
                --need;
            }
        }
        __syncthreads();
    }
    if (lane < live) {
        int before = 0;
        static_for<0, kWords>([&](auto i) {
            if (i % W == w) {
                uint8_t* out = &s_places[lane * k + before];
                uint32_t left = word[i];
                while (left != 0u) {
                    *out++ = static_cast<uint8_t>(32 * i + __ffs(left) - 1);
                    left &= left - 1u;
                }
            }
            before += __popc(word[i]);
        });
    }
    __syncthreads();

    // ---- payload: every thread's entries, and where their coefficients will be parked: class-major,
    // index i at (i mod S/2 in its class), the half i / (S/2) in the upper bits
    auto emit = [&](auto vec_tag) {
        constexpr int VEC = decltype(vec_tag)::value;
        const uint32_t magic = entry_magic(k);
        const uint32_t entries = static_cast<uint32_t>(live * k);
        auto entry = [&](int i) -> uint32_t {              // number of this thread's entry i
            return VEC == 4 ? 4u * (tid + kThreads * (i / 4)) + i % 4 : tid + kThreads * i;
        };
        uint32_t at[N];
        float v[N];
#pragma unroll
        for (int i0 = 0; i0 < N; i0 += VEC) {
            const uint32_t e = entry(i0);                  // (a quad's entries belong to one chunk)
            const bool in = e < entries;
            const uint32_t r = k == 1 ? e : __umulhi(e, magic);
            uint32_t places = 0u;
            if (in) places = VEC == 4 ? *reinterpret_cast<const uint32_t*>(&s_places[e]) : s_places[e];
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                const uint32_t j = (places >> (8 * i)) & 0xFFu;
                const uint32_t half = j >= H ? 1u : 0u, jh = j - half * H;
                const uint32_t cls = ((jh & 1u) << 1) | ((jh >> 1) & 1u);   // (split_off)
                at[i0 + i] = in ? (4u * (r * kRow + cls * L + jh / W)) | (half << 30) : 2u << 30;
                v[i0 + i] = 0.0f;
            }
        }
        char* lds = reinterpret_cast<char*>(buf);
        static_for<0, 2>([&](auto P) {
            regs_range_to_lds<P * L, (P + 1) * L>(row + w * L, c);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < N; ++i)
                if ((at[i] >> 30) == P)
                    v[i] = *reinterpret_cast<const float*>(lds + (at[i] & 0x3FFFFFFFu));
            // what a kept coefficient leaves behind: the rounding error of a 16-bit format
#pragma unroll
            for (int i = 0; i < N; ++i)
                if ((at[i] >> 30) == P)
                    *reinterpret_cast<float*>(lds + (at[i] & 0x3FFFFFFFu)) =
                        NARROW ? v[i] - payload_roundtrip(p.val_dtype, v[i]) : 0.0f;
            __syncthreads();
            lds_to_regs_range<P * L, (P + 1) * L>(row + w * L, c);
        });
        // the tile's entries are contiguous in both arrays
        const int64_t e0 = chunk0 * k;
        const int value_bytes = !NARROW || p.val_dtype == 0 ? 4 : 2, index_bytes = NARROW && p.idx_u8 ? 1 : 4;
        char* vals = static_cast<char*>(val_out) + e0 * value_bytes;
        char* idxs = static_cast<char*>(idx_out) + e0 * index_bytes;
#pragma unroll
        for (int i = 0; i < N; i += VEC) {
            const uint32_t e = entry(i);
            if (e >= entries) continue;
            if constexpr (VEC == 4) {
                const uint32_t four = *reinterpret_cast<const uint32_t*>(&s_places[e]);
                if (NARROW && p.idx_u8)
                    *reinterpret_cast<uint32_t*>(idxs + e) = four;
                else
                    *reinterpret_cast<uint4*>(idxs + 4u * e) =
                        make_uint4(four & 0xFFu, (four >> 8) & 0xFFu, (four >> 16) & 0xFFu, four >> 24);
                if (!NARROW || p.val_dtype == 0) {
                    *reinterpret_cast<float4*>(vals + 4u * e) =
                        make_float4(v[i], v[i + 1], v[i + 2], v[i + 3]);
                } else {
                    uint2 h;
                    if (p.val_dtype == 1) {
                        h.x = pack_bf16x2(v[i], v[i + 1]);
                        h.y = pack_bf16x2(v[i + 2], v[i + 3]);
                    } else {
                        h.x = f32_to_f16(v[i]) | (static_cast<uint32_t>(f32_to_f16(v[i + 1])) << 16);
                        h.y = f32_to_f16(v[i + 2]) | (static_cast<uint32_t>(f32_to_f16(v[i + 3])) << 16);
                    }
                    *reinterpret_cast<uint2*>(vals + 2u * e) = h;
                }
            } else {
                if (!NARROW || p.val_dtype == 0) *reinterpret_cast<float*>(vals + 4u * e) = v[i];
                else
                    *reinterpret_cast<uint16_t*>(vals + 2u * e) =
                        p.val_dtype == 1 ? encode16<1>(v[i]) : encode16<2>(v[i]);
                if (NARROW && p.idx_u8) *reinterpret_cast<uint8_t*>(idxs + e) = s_places[e];
                else *reinterpret_cast<uint32_t*>(idxs + 4u * e) = s_places[e];
            }
        }
    };
    if (k % 4 == 0) emit(std::integral_constant<int, 4>{});
    else emit(std::integral_constant<int, 1>{});

    // ---- new momentum = inverse transform of the remainder
    c[0] *= (w == 0) ? p.alpha0 : p.alpha;
#pragma unroll
    for (int m = 1; m < Q; ++m) c[m] *= p.alpha;
    half_inverse<kFused>(row, w, c);
    static_for<0, 2>([&](auto P) {
        if constexpr (P == 1) __syncthreads();
        half_outputs_to_rows<P>(row, w, c);
        __syncthreads();
        // elements n0 .. n0+3 = E + O and their mirror images E - O
        constexpr int kPer = S / 16;                       // pieces of n0 per row and half
#pragma unroll
        for (int it = 0; it < Q / 16; ++it) {
            const int g = tid + kThreads * it;
            const int r = g / kPer, u = g - r * kPer;
            const float* src = &buf[r * kRow];
            const float4 e = *reinterpret_cast<const float4*>(src + 4 * u);
            const float2 oe = *reinterpret_cast<const float2*>(src + 2 * L + 2 * u);
            const float2 oo = *reinterpret_cast<const float2*>(src + 3 * L + 2 * u);
            const float4 o = make_float4(oe.x, oo.x, oe.y, oo.y);
            const int n0 = P * Q + 4 * u;
            auto put = [&](int col, float4 y) {
                const int64_t i0 = base + r * S + col;
                if (!partial || i0 + 3 < n) {
                    st_f4<true>(mom + i0, y);
                } else {
                    const float ys[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (i0 + j < n) mom[i0 + j] = ys[j];
                }
            };
            put(n0, make_float4(e.x + o.x, e.y + o.y, e.z + o.z, e.w + o.w));
            put(S - 4 - n0, make_float4(e.w - o.w, e.z - o.z, e.y - o.y, e.x - o.x));
        }
    });
}

}  // namespace deto
