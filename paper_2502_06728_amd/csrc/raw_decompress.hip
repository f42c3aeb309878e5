// Striding / Random decompress-and-update on the momentum itself, no transmitted indices: any payload
// format, any k <= S/2, plain update, Decoupled AdamW, amsgrad.
#include "raw_kernels.hip.h"
#include "tiled_launch.h"

namespace deto {

int64_t launch_decompress_raw(const DecompressLaunch& a) {
    const KParams& p = a.p;
#ifdef DETO_TILED_ONLY_64_32
    return 0;
#else
    if (a.idx || p.scheme == 0 || p.use_dct || 2 * p.k > p.s) return 0;
    if (!raw_decompress(p, a.n, a.param_bf16)) return 0;
    const int quads = raw_decompress_quads(p, a.n);
    const int wgs_cu = raw_decompress_workgroups(p, a.n, a.param_bf16);
    auto launch = [&](auto S_tag, auto Q_tag, auto kernel) -> int64_t {
        using G = RawGeom<decltype(S_tag)::value, decltype(Q_tag)::value>;
        const int64_t wgs = (a.n_chunks + G::kChunks - 1) / G::kChunks;
        if (wgs > 0x7FFFFFFF) return 0;
        kernel<<<static_cast<unsigned>(wgs), kRawThreads,
                 raw_lds(G::decompress_lds(p.k, p.scheme == 2), wgs_cu), a.stream>>>(p, a.n, a.n_chunks, a.val, a.val_stride, a.params, a.adam,
                             a.presign_dbg);
        return a.n_chunks;
    };
#define K(S, Q, OPT) (a.param_bf16 ? decompress_raw<S, Q, true, OPT> : decompress_raw<S, Q, false, OPT>)
#define X(S, Q)                                                                              \
    if (p.s == S && quads == Q)                                                              \
        return launch(std::integral_constant<int, S>{}, std::integral_constant<int, Q>{},    \
                      !p.adam ? K(S, Q, 0) : !p.amsgrad ? K(S, Q, 1) : K(S, Q, 2));
    DETO_RAW_DECOMPRESS_LIST(X)
#undef X
#undef K
    return 0;
#endif
}

}  // namespace deto
