// Device-side helpers shared by the gfx950 kernels: dtype conversion, the counter-based
// generator of the Random scheme, kernel parameter block.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace deto {

constexpr int kWave = 64;        // CDNA wavefront width
constexpr int kMaxChunk = 256;   // largest chunk size s the library accepts
constexpr int kMaxReplicas = 64;  // largest replication group R the library accepts

// Everything a kernel needs from deto_config, resolved on the host.
struct KParams {
    int s;              // chunk size
    int k;              // kept entries per chunk
    int scheme;         // deto_scheme
    int use_dct;        // transform domain (always for TOPK)
    int use_sign;       // DETO_FLAG_SIGN
    int R;              // replicas (decompress)
    int val_dtype;      // payload values: 0 fp32, 1 bf16, 2 fp16
    int idx_u8;         // payload indices as bytes instead of int32
    float beta;         // momentum decay
    float lr;           // eta
    float wd_scale;     // 1 - eta*lambda
    float alpha0;       // sqrt(1/s): scale of DCT row 0
    float alpha;        // sqrt(2/s): scale of the other rows
    float inv_R;        // 1/R
    uint64_t seed;
    uint64_t step;
    // Decoupled AdamW as the underlying optimizer (adam != 0)
    int adam;
    int amsgrad;
    float b1, b2;       // betas
    float omb1, omb2;   // 1 - beta
    float eps;
    float step_size;    // eta / (1 - beta1^t)
    float inv_sqrt_bc2; // 1 / sqrt(1 - beta2^t)
    int run_lg;         // run_log2 of this call (6: no gangs)
    int count_signs;    // this call's two-bit signs are counted a word at a time (count_signs)
};

// ---- Which 64 chunks a tile is made of.  Not 64 in a row: kGang consecutive tiles (a gang) share
// kGang * 64 chunks and take them in turn, a run of 2^lg chunks each, so that the workgroups in flight walk
// through every array side by side, in windows of a run each, instead of each through a window of its own.
// Memory is faster that way.  The traffic alone, without arithmetic (membench), 147 M parameters, us, tiles in a
// row / in gangs: eight streams of 8 KiB a tile read and one rewritten 517 / 465; 24 KiB read and 32 KiB written 379 /
// 368 (plain stores 389 / 384: an interleaved stream wants non-temporal ones); AdamW's three rewritten 548 / 521.
// Which launches are in gangs: compress_run_log2, decompress_gangs and decompress_run_log2 in tiled_launch.h.  The
// chunks that do not fill a gang are tiles of 64 in a row (lg = 6: no gangs at all).
//
// A run is 512 elements or more (2 KiB of fp32: a wavefront's loads stay whole), and at least `run_bytes` of
// every payload array, below which runs cost more lines than they save: decompress, plain update, us,
// in a row / runs of that many bytes: 64/4, 32 replicas, fp32 parameters, 60 M 253 / 128 319, 64/16,
// 8 replicas, 147 M bf16 487 / 512 472, 1,024 455, 128/32, 4 replicas 373 (fp32) / 512 380, 1,024 373.  More
// than 16 chunks a run (32 at chunk 16) gain nothing: 32/16 signs 546 / 553.  Chunk 96 loses 3 - 6 %, chunk
// 192 and 256 are bound by their arithmetic (256/32 decompress 246 / 262).
constexpr int kGang = 32;
constexpr int kRunElems = 512, kRunBytes = 128, kSchemeRunBytes = 1024;
constexpr bool in_gangs(int s) { return s == 16 || s == 32 || s == 64 || s == 128; }
// idx_bytes: of one transmitted index, 0 without indices
__host__ __device__ constexpr int run_log2(int s, int k, int val_dtype, int idx_bytes, int run_bytes) {
    if (!in_gangs(s)) return 6;
    int payload = val_dtype == 3 ? 4 * ((k + 15) / 16) : k * (val_dtype == 0 ? 4 : 2);
    if (idx_bytes != 0 && k * idx_bytes < payload) payload = k * idx_bytes;
    int lg = 0;
    while (lg < 6 && ((s << lg) < kRunElems || (payload << lg) < run_bytes)) ++lg;
    return lg <= (s == 16 ? 5 : 4) ? lg : 6;
}
// Decompress reads a payload per replica: the more of the traffic that is, the longer its runs (us, in a
// row / runs of that many bytes.  AdamW, 64/4: 4 replicas 147 M 550 / 128 530, 32 replicas 60 M 388 / 128
// 427.  Plain update, 4 replicas, fp32 parameters, 60 M: 64/8 116 / 256 113, 64/4 100 / 256 103, 32/4 147 M
// 284 / 256 272).
__host__ __device__ constexpr int decompress_run_bytes(int s, int k, int R, bool adam) {
    if (adam) return R * k <= s ? 128 : 256;
    return 2 * R * k <= s && (s <= 32 || k >= 8) ? 256 : 1024;
}

// Striding and Random on coefficients, a lane per chunk, fp32 values: decompress kernels in gangs
__host__ __device__ constexpr bool scheme_gangs(int s, int k) { return k >= 16 && (s == 32 || s == 64); }

struct TileRows {
    int64_t first;      // chunk of row 0
    uint32_t skip;      // chunks between a run's end and the next one's start
    int lg;
    // row r's chunk, counted from `first`
    __host__ __device__ __forceinline__ uint32_t chunk(uint32_t r) const { return r + (r >> lg) * skip; }
    // item e (of row r) of the tile's, `unit` a chunk, counted from the first chunk's first item.  (Below
    // 2^24: 24-bit products.)
    __device__ __forceinline__ uint32_t item(uint32_t e, uint32_t r, uint32_t unit) const {
        return e + __umul24(r >> lg, skip * unit);
    }
    // The accesses below are a uniform base and a 32-bit offset of the lane; what these functions give is
    // added to the pointer one after the other, so that it stays that way.
    // Elements e .. e + 4 * kWave - 1 that a wavefront takes at a time, S a chunk (a run is a multiple of
    // that): where the first one is
    template <int S>
    __device__ __forceinline__ uint32_t quads(uint32_t e) const {
        return e + ((e / S) >> lg) * (skip * S);
    }
    // item it * BLOCK + within (within < BLOCK), UNIT a chunk, LG = lg: the block's part and the lane's
    template <int UNIT, int LG, int BLOCK>
    __device__ __forceinline__ uint32_t block(int it) const {
        constexpr int kRun = UNIT << LG;
        if constexpr (LG >= 6 || (kRun % BLOCK != 0 && BLOCK % kRun != 0)) return 0u;
        else return it * BLOCK + (it * BLOCK / kRun) * (skip * UNIT);
    }
    template <int UNIT, int LG, int BLOCK>
    __device__ __forceinline__ uint32_t within_block(int it, uint32_t within) const {
        constexpr int kRun = UNIT << LG;
        if constexpr (LG >= 6) return it * BLOCK + within;
        else if constexpr (kRun % BLOCK == 0) return within;
        else if constexpr (BLOCK % kRun == 0) return within + __umul24(within / kRun, skip * UNIT);
        else return it * BLOCK + within + __umul24((it * BLOCK + within) / kRun, skip * UNIT);
    }
};

__host__ __device__ __forceinline__ TileRows tile_rows(int64_t tile, int64_t tiles, int lg) {
    const int64_t gang = tile / kGang;
    if (lg < 6 && (gang + 1) * kGang <= tiles)
        return {gang * (kGang * kWave) + ((tile % kGang) << lg),
                static_cast<uint32_t>(kGang - 1) << lg, lg};
    return {tile * kWave, 0u, lg};
}

// AdamW moment arrays (device pointers; vmax only with amsgrad)
struct AdamPtrs {
    float* m;
    float* v;
    float* vmax;
};

// ---- 16-byte global accesses with an optional non-temporal hint.  Every tensor on this
// path is touched once per call; on MI355X the hint lifts a many-stream read from about
// 6.3 to 7.0 TB/s.
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

// Per-site policy (measured on MI355X, OLMo-1B shard): the decompress kernel gains from
// the hint on every access; the compress kernel, which rewrites the momentum it has just
// read, on its stores where tiles are in gangs (LG < 6: 64/32 374 us without both, 372 with gangs alone,
// 360 with both; without gangs the hint costs 4 %).
#ifndef DETO_NT_COMPRESS_GRAD
#define DETO_NT_COMPRESS_GRAD 0
#endif
#ifndef DETO_NT_COMPRESS_MOM
#define DETO_NT_COMPRESS_MOM 0
#endif
#ifndef DETO_NT_COMPRESS_PAYLOAD
#define DETO_NT_COMPRESS_PAYLOAD (LG < 6)
#endif
#ifndef DETO_NT_COMPRESS_MOM_ST
#define DETO_NT_COMPRESS_MOM_ST (LG < 6)
#endif
#ifndef DETO_NT_DECOMPRESS_LD
#define DETO_NT_DECOMPRESS_LD 1
#endif
#ifndef DETO_NT_DECOMPRESS_ST
#define DETO_NT_DECOMPRESS_ST 1
#endif

template <bool NT>
__device__ __forceinline__ float4 ld_f4(const float* p) {
    if constexpr (NT) {
        const f32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(p));
        return make_float4(t.x, t.y, t.z, t.w);
    } else {
        return *reinterpret_cast<const float4*>(p);
    }
}

template <bool NT>
__device__ __forceinline__ uint4 ld_u4(const void* p) {
    if constexpr (NT) {
        const u32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
        return make_uint4(t.x, t.y, t.z, t.w);
    } else {
        return *reinterpret_cast<const uint4*>(p);
    }
}

typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

template <bool NT>
__device__ __forceinline__ uint2 ld_u2(const void* p) {
    if constexpr (NT) {
        const u32x2_t t = __builtin_nontemporal_load(reinterpret_cast<const u32x2_t*>(p));
        return make_uint2(t.x, t.y);
    } else {
        return *reinterpret_cast<const uint2*>(p);
    }
}

template <bool NT>
__device__ __forceinline__ uint32_t ld_u1(const void* p) {
    if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(p));
    else return *reinterpret_cast<const uint32_t*>(p);
}

template <bool NT>
__device__ __forceinline__ void st_f4(float* p, float4 v) {
    if constexpr (NT) {
        const f32x4_t t = {v.x, v.y, v.z, v.w};
        __builtin_nontemporal_store(t, reinterpret_cast<f32x4_t*>(p));
    } else {
        *reinterpret_cast<float4*>(p) = v;
    }
}

template <bool NT>
__device__ __forceinline__ void st_u4(void* p, uint4 v) {
    if constexpr (NT) {
        const u32x4_t t = {v.x, v.y, v.z, v.w};
        __builtin_nontemporal_store(t, reinterpret_cast<u32x4_t*>(p));
    } else {
        *reinterpret_cast<uint4*>(p) = v;
    }
}

template <bool NT>
__device__ __forceinline__ void st_u2(void* p, uint2 v) {
    if constexpr (NT) {
        const u32x2_t t = {v.x, v.y};
        __builtin_nontemporal_store(t, reinterpret_cast<u32x2_t*>(p));
    } else {
        *reinterpret_cast<uint2*>(p) = v;
    }
}

// Ordering point between the LDS phases of a single-wavefront workgroup.  The LDS queue of
// one wavefront is processed in program order, so no hardware barrier is needed; this only
// stops the compiler from moving LDS accesses across the phase boundary.  Unlike
// __syncthreads() it does not wait for outstanding global loads and stores, so prefetched
// data stays in flight and finished tiles retire without waiting for their stores.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
    return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// fp32 -> bf16, round to nearest even (finite inputs).
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return static_cast<uint16_t>(u >> 16);
}

// IEEE half <-> fp32 (round to nearest even; half subnormals are kept on gfx950)
__device__ __forceinline__ uint16_t f32_to_f16(float f) {
    return __builtin_bit_cast(uint16_t, static_cast<_Float16>(f));
}

__device__ __forceinline__ float f16_to_f32(uint16_t b) {
    return static_cast<float>(__builtin_bit_cast(_Float16, b));
}

// payload value formats: 0 fp32, 1 bf16, 2 fp16
template <int VAL>
__device__ __forceinline__ uint16_t encode16(float v) {
    static_assert(VAL == 1 || VAL == 2, "16-bit transfer dtype");
    if constexpr (VAL == 1) return f32_to_bf16(v);
    else return f32_to_f16(v);
}

template <int VAL>
__device__ __forceinline__ float decode16(uint16_t b) {
    static_assert(VAL == 1 || VAL == 2, "16-bit transfer dtype");
    if constexpr (VAL == 1) return bf16_to_f32(b);
    else return f16_to_f32(b);
}

// two fp32 -> packed bf16 (lo in bits 0..15), round to nearest even: one v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    const f32x2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// sign(y) in {-1, 0, +1} without compares: scaling by 2^192 (two exact multiplications by
// 2^96, enough to lift the smallest fp32 subnormal above 1) and clamping to [-1, 1] maps
// every non-zero finite y to +-1 and keeps +-0.
__device__ __forceinline__ float sign3(float y) {
    return __builtin_amdgcn_fmed3f(y * 0x1p96f * 0x1p96f, -1.0f, 1.0f);
}

__device__ __forceinline__ float sign_or_self(float y, int use_sign) {
    return use_sign ? sign3(y) : y;
}

// One Decoupled-AdamW step for one element: moments updated in place, returns the new
// parameter value in fp32 (section "Decoupled AdamW"; q is the averaged update).
template <bool AMSGRAD>
__device__ __forceinline__ float adamw_step(const KParams& p, float theta, float q, float& m,
                                            float& v, float& vmax) {
    m = fmaf(p.b1, m, p.omb1 * q);
    v = fmaf(p.b2, v, p.omb2 * q * q);
    float vh = v;
    if constexpr (AMSGRAD) {
        vmax = fmaxf(vmax, v);
        vh = vmax;
    }
    const float denom = fmaf(sqrtf(vh), p.inv_sqrt_bc2, p.eps);
    return fmaf(-p.step_size, m / denom, theta * p.wd_scale);
}
__device__ __forceinline__ float adamw_step(const KParams& p, float theta, float q, float& m,
                                            float& v, float& vmax) {
    return p.amsgrad ? adamw_step<true>(p, theta, q, m, v, vmax)
                     : adamw_step<false>(p, theta, q, m, v, vmax);
}

// ---- Compares into the carry and additions with carry, four at a time.  A carry may be read no earlier
// than two instructions after the compare that wrote it; the compiler pads its own code (s_nop 1) but
// not what is inside an asm statement: four compares into four register pairs, then the four additions, so
// three instructions lie between.  In C++ every compare waits for its own addition: compress, us, C++
// and this, 256/32 bf16 gradients 141 M 384, 379; 128/32 bf16 values 141 M 355, 350; signs 16/8 0.4 M 11.9,
// 11.2, 64/24 0.4 M 11.8, 11.1 (signs 64/8 12.6 M 61.3, 61.8).
#define DETO_FOUR_CARRIES(ADD)                                                                      \
    "v_cmp_ge_u32 %1, %5, %9\n\tv_cmp_ge_u32 %2, %6, %9\n\t"                                        \
    "v_cmp_ge_u32 %3, %7, %9\n\tv_cmp_ge_u32 %4, %8, %9\n\t"                                        \
    "v_addc_co_u32 %0, vcc, " ADD ", %0, %1\n\tv_addc_co_u32 %0, vcc, " ADD ", %0, %2\n\t"          \
    "v_addc_co_u32 %0, vcc, " ADD ", %0, %3\n\tv_addc_co_u32 %0, vcc, " ADD ", %0, %4"

// 16*word + 8*(a >= thr) + 4*(b >= thr) + 2*(c >= thr) + (d >= thr)
__device__ __forceinline__ uint32_t push_if_at_least(uint32_t word, uint32_t a, uint32_t b, uint32_t c,
                                                     uint32_t d, uint32_t thr) {
    uint64_t c0, c1, c2, c3;
    asm(DETO_FOUR_CARRIES("%0")
        : "+v"(word), "=&s"(c0), "=&s"(c1), "=&s"(c2), "=&s"(c3)
        : "v"(a), "v"(b), "v"(c), "v"(d), "v"(thr)
        : "vcc");
    return word;
}
// 4*word + 2*!(|a| < thr) + !(|b| < thr): for magnitudes this is >= as integers (a NaN counts as the
// largest).  Two at a time, which has no registers to spare around it (four: 24 bytes of scratch memory
// and 60 M 256/8 bf16 136, 150 us).
__device__ __forceinline__ uint32_t push_unless_below(uint32_t word, float a, float b, float thr) {
    uint64_t c0;
    asm("v_cmp_nlt_f32 %1, |%2|, %4\n\tv_cmp_nlt_f32 vcc, |%3|, %4\n\ts_nop 0\n\t"
        "v_addc_co_u32 %0, %1, %0, %0, %1\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc"
        : "+v"(word), "=&s"(c0)
        : "v"(a), "v"(b), "v"(thr)
        : "vcc");
    return word;
}
// cnt + how many of the four reach cand
__device__ __forceinline__ uint32_t add_if_at_least(uint32_t cnt, uint32_t a, uint32_t b, uint32_t c,
                                                    uint32_t d, uint32_t cand) {
    uint64_t c0, c1, c2, c3;
    asm(DETO_FOUR_CARRIES("0")
        : "+v"(cnt), "=&s"(c0), "=&s"(c1), "=&s"(c2), "=&s"(c3)
        : "v"(a), "v"(b), "v"(c), "v"(d), "v"(cand)
        : "vcc");
    return cnt;
}

// ---- Random scheme generator (paper, "Replication Schemes": indices are reproduced on
// every replica from a shared seed).  key = mix64(mix64(seed + G*(step+1)) + G*(chunk+1)),
// draw_j = mix32(lo32(key) + 0x9E3779B9*(j+1)) ^ hi32(key), bounded(d,b) = (d*b) >> 32.
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ uint32_t mix32(uint32_t x) {
    x ^= x >> 16;
    x *= 0x7FEB352Du;
    x ^= x >> 15;
    x *= 0x846CA68Bu;
    x ^= x >> 16;
    return x;
}

__device__ __forceinline__ uint64_t chunk_key(uint64_t seed, uint64_t step, uint64_t chunk) {
    const uint64_t G = 0x9E3779B97F4A7C15ull;
    return mix64(mix64(seed + G * (step + 1ull)) + G * (chunk + 1ull));
}

__device__ __forceinline__ uint32_t draw(uint64_t key, uint32_t j) {
    return mix32(static_cast<uint32_t>(key) + 0x9E3779B9u * (j + 1u)) ^
           static_cast<uint32_t>(key >> 32);
}

__device__ __forceinline__ uint32_t bounded(uint32_t d, uint32_t b) {
    return __umulhi(d, b);
}

// The sums over R replicas of a word of 16 two-bit signs; replica r's word is words[r * stride + at], words uniform.
// A field is 0, 1 or 3 (2 counts as 0), so its sum is (fields with bit 0) - 2 (fields with both bits): both are counted
// side by side, three replicas in the two bits of a field, five times that in four bits, up to 64 in eight.  Batches of
// 18 words, not of 33: the registers are worth a wavefront per SIMD more to a launch than a round trip less to 64
// replicas (streaming kernels, geometric mean over 600 random shapes 0.93 of the time, none but 2 % of them longer).
struct SignCounts {
    uint32_t ones[4] = {0u, 0u, 0u, 0u}, both[4] = {0u, 0u, 0u, 0u};      // byte b: field 4b + i

    // (a batch is counted whole, however few replicas are in it)
    __device__ __forceinline__ SignCounts(const uint32_t* __restrict__ words, uint32_t at, int64_t stride,
                                          int R) {
        int r0 = 0;
        for (; R - r0 > 18; r0 += 18) add<18>(words, at, stride, r0, R);
        const int left = R - r0;
        if (left <= 3) add<3>(words, at, stride, r0, R);
        else if (left <= 9) add<9>(words, at, stride, r0, R);
        else add<18>(words, at, stride, r0, R);
    }
    // the replicas r0 .. r0 + BATCH - 1 that there are.  Every load is unconditional (the last replica's again
    // past it): behind a branch a load is masked, and so waited for, before the next one leaves.
    template <int BATCH>
    __device__ __forceinline__ void add(const uint32_t* __restrict__ words, uint32_t at, int64_t stride, int r0,
                                        int R) {
        uint32_t x[BATCH];
#pragma unroll
        for (int i = 0; i < BATCH; ++i) x[i] = (words + min(r0 + i, R - 1) * stride)[at];
#pragma unroll
        for (int i = 0; i < BATCH; ++i) x[i] = r0 + i < R ? x[i] : 0u;
#pragma unroll
        for (int f = 0; f < BATCH; f += 15) {
            uint32_t o4[2] = {0u, 0u}, b4[2] = {0u, 0u};               // nibble b: field 2b + i
#pragma unroll
            for (int t = f; t < f + 15 && t < BATCH; t += 3) {
                uint32_t o2 = 0u, b2 = 0u;
#pragma unroll
                for (int i = t; i < t + 3; ++i) {
                    const uint32_t one = x[i] & 0x55555555u;
                    o2 += one;
                    b2 += one & (x[i] >> 1);
                }
                o4[0] += o2 & 0x33333333u;
                o4[1] += (o2 >> 2) & 0x33333333u;
                b4[0] += b2 & 0x33333333u;
                b4[1] += (b2 >> 2) & 0x33333333u;
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                ones[i] += o4[i] & 0x0F0F0F0Fu;
                ones[i + 2] += (o4[i] >> 4) & 0x0F0F0F0Fu;
                both[i] += b4[i] & 0x0F0F0F0Fu;
                both[i + 2] += (b4[i] >> 4) & 0x0F0F0F0Fu;
            }
        }
    }
    // of field f (a constant where it is called)
    __device__ __forceinline__ float sum(int f) const {
        return static_cast<float>(static_cast<int>((ones[f % 4] >> (8 * (f / 4))) & 0xFFu) -
                                  2 * static_cast<int>((both[f % 4] >> (8 * (f / 4))) & 0xFFu));
    }
};

}  // namespace deto
