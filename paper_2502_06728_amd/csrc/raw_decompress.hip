// Striding / Random decompress-and-update on the momentum itself, no transmitted indices, any k <= S/2: plain update
// and values of 16 or 32 bits here; two-bit signs, Decoupled AdamW and amsgrad in units of their own
// (raw_decompress_*.hip).
#ifndef DETO_RAW_FN
#define DETO_RAW_FN launch_decompress_raw_values
#define DETO_RAW_OPT 0
#define DETO_RAW_SIGNS false
#endif
#include "raw_kernels.hip.h"
#include "tiled_launch.h"

namespace deto {

int64_t DETO_RAW_FN(const DecompressLaunch& a) {
    const KParams& p = a.p;
#ifdef DETO_TILED_ONLY_64_32
    return 0;
#else
    const int quads = raw_decompress_quads(p, a.n);
    const int wgs_cu = raw_decompress_workgroups(p, a.n, a.param_bf16);
    auto launch = [&](auto S_tag, auto Q_tag, auto kernel) -> int64_t {
        using G = RawGeom<decltype(S_tag)::value, decltype(Q_tag)::value>;
        const int64_t wgs = (a.n_chunks + G::kChunks - 1) / G::kChunks;
        if (wgs > 0x7FFFFFFF) return 0;
        const unsigned lds = raw_lds(G::decompress_lds(p.k, p.scheme == 2), wgs_cu);
        kernel<<<static_cast<unsigned>(wgs), kRawThreads, lds, a.stream>>>(
            p, a.n, a.n_chunks, a.val, a.val_stride, a.params, a.adam, a.presign_dbg);
        return a.n_chunks;
    };
#define X(S, Q)                                                                              \
    if (p.s == S && quads == Q)                                                              \
        return launch(std::integral_constant<int, S>{}, std::integral_constant<int, Q>{},    \
                      a.param_bf16 ? decompress_raw<S, Q, true, DETO_RAW_OPT, DETO_RAW_SIGNS>  \
                                   : decompress_raw<S, Q, false, DETO_RAW_OPT, DETO_RAW_SIGNS>);
    DETO_RAW_DECOMPRESS_LIST(X)
#if DETO_RAW_OPT == 0
    DETO_RAW_DECOMPRESS_PLAIN_LIST(X)
#endif
#undef X
    return 0;
#endif
}

}  // namespace deto
