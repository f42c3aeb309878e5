// Shared body of the tiled_topk_s*.hip units: instantiates the top-k compress kernel and the
// indexed decompress kernel for chunk size DETO_S and the k values in DETO_K_LIST(X), and
// defines the two launchers named by DETO_COMPRESS_FN / DETO_DECOMPRESS_FN.  A unit that
// does not define DETO_COMPRESS_FN has the decompress kernel only (chunk sizes above 64).
#include "tiled_kernels.hip.h"
#include "tiled_launch.h"

namespace deto {

#ifdef DETO_COMPRESS_FN
bool DETO_COMPRESS_FN(const CompressLaunch& a) {
    if (a.p.s != DETO_S || a.p.val_dtype != 0 || a.p.idx_u8) return false;
    const unsigned grid = tiled_grid(a.tiles, a.n_chunks);
    const TailRange tail{a.n, a.n_chunks};
#define LAUNCH(K, BF16, GANG)                                                                   \
    compress_tiled_topk<DETO_S, K, BF16, 0, GANG><<<grid, kWave, spare_lds(a), a.stream>>>(    \
        a.p, a.tiles, tail, a.grad, a.mom, a.idx, a.val, a.coeff_dbg)
#define X(K)                                                                                    \
    if (a.p.k == K) {                                                                           \
        constexpr bool kGangs = run_log2(DETO_S, K, 0, 4, kRunBytes) < 6;                       \
        if (kGangs && a.p.run_lg < 6) {                                                         \
            if (a.grad_bf16) LAUNCH(K, true, kGangs); else LAUNCH(K, false, kGangs);            \
        } else {                                                                                \
            if (a.grad_bf16) LAUNCH(K, true, false); else LAUNCH(K, false, false);              \
        }                                                                                       \
        return true;                                                                            \
    }
    DETO_K_LIST(X)
#undef X
#undef LAUNCH
    return false;
}
#endif

bool DETO_DECOMPRESS_FN(const DecompressLaunch& a) {
    if (a.p.s != DETO_S || !a.idx || a.p.val_dtype != 0 || a.p.idx_u8 || a.p.adam) return false;
    const unsigned grid = tiled_grid(a.tiles, a.n_chunks);
    const TailRange tail{a.n, a.n_chunks};
#define X(K)                                                                                    \
    if (a.p.k == K) {                                                                           \
        if (a.param_bf16)                                                                       \
            decompress_tiled<DETO_S, K, true><<<grid, kWave, spare_lds(a), a.stream>>>(        \
                a.p, a.tiles, tail, a.idx, a.idx_stride, a.val, a.val_stride, a.params,               \
                AdamPtrs{nullptr, nullptr, nullptr}, a.presign_dbg);                                                                 \
        else if constexpr (DETO_S == 16)   /* (always two classes, see decompress_classes) */   \
            return false;                                                                       \
        else                                                                                    \
            decompress_tiled<DETO_S, K, false><<<grid, kWave, spare_lds(a), a.stream>>>(       \
                a.p, a.tiles, tail, a.idx, a.idx_stride, a.val, a.val_stride, a.params,               \
                AdamPtrs{nullptr, nullptr, nullptr}, a.presign_dbg);                                                                 \
        return true;                                                                            \
    }
    DETO_K_LIST(X)
#undef X
    return false;
}

}  // namespace deto
