// Shared body of tiled_scheme.hip / tiled_scheme_small.hip: instantiates the Striding / Random
// kernels (decompress: raw-momentum or coefficient domain) for the (chunk, k) pairs in DETO_SCHEME_LIST(X)
// and defines the two launchers named by DETO_COMPRESS_SCHEME_FN / DETO_DECOMPRESS_SCHEME_FN.
#include "tiled_kernels.hip.h"
#include "tiled_launch.h"

namespace deto {

namespace {
MaskWords words(const uint32_t (&w)[4]) { return MaskWords{{w[0], w[1], w[2], w[3]}}; }
}  // namespace

bool DETO_COMPRESS_SCHEME_FN(const CompressLaunch& a) {
    if (!a.p.use_dct || a.p.val_dtype != 0 || a.p.idx_u8) return false;   // fp32 values, int32 indices only
    const unsigned grid = tiled_grid(a.tiles, a.n_chunks);
    const TailRange tail{a.n, a.n_chunks};
#define LAUNCH(S, K, BF16, GANG)                                                                \
    compress_tiled_scheme<S, K, BF16, 0, GANG><<<grid, kWave, spare_lds(a), a.stream>>>(        \
        a.p, words(a.stride_mask), a.tiles, tail, a.grad, a.mom, a.idx, a.val, a.coeff_dbg)
#define X(S, K)                                                                                 \
    if (a.p.s == S && a.p.k == K) {                                                             \
        constexpr bool kGangs = run_log2(S, K, 0, 0, kRunBytes) < 6;                            \
        if (kGangs && a.p.run_lg < 6) {                                                         \
            if (a.grad_bf16) LAUNCH(S, K, true, kGangs); else LAUNCH(S, K, false, kGangs);      \
        } else {                                                                                \
            if (a.grad_bf16) LAUNCH(S, K, true, false); else LAUNCH(S, K, false, false);        \
        }                                                                                       \
        return true;                                                                            \
    }
    DETO_SCHEME_LIST(X)
#undef X
#undef LAUNCH
    return false;
}

bool DETO_DECOMPRESS_SCHEME_FN(const DecompressLaunch& a) {
    if (a.idx || a.p.val_dtype != 0 || a.p.adam) return false;
    const unsigned grid = tiled_grid(a.tiles, a.n_chunks);
    const TailRange tail{a.n, a.n_chunks};
#define LAUNCH(S, K, BF16, GANG)                                                                \
    decompress_tiled_scheme<S, K, BF16, 0, GANG, false><<<grid, kWave, spare_lds(a), a.stream>>>(      \
        a.p, words(a.stride_mask), a.tiles, tail, a.val, a.val_stride, a.params,                \
        AdamPtrs{nullptr, nullptr, nullptr}, a.presign_dbg)
#define X(S, K)                                                                                 \
    if (a.p.s == S && a.p.k == K) {                                                             \
        constexpr bool kGangs = scheme_gangs(S, K);                                             \
        if (!a.param_bf16) LAUNCH(S, K, false, false);                                          \
        else if (kGangs && a.p.run_lg < 6) LAUNCH(S, K, true, kGangs);                          \
        else LAUNCH(S, K, true, false);                                                         \
        return true;                                                                            \
    }
    DETO_SCHEME_LIST(X)
#undef X
#undef LAUNCH
    return false;
}

}  // namespace deto
