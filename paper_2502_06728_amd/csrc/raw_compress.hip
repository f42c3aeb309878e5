// Striding / Random compress on the momentum itself: any payload format, any k <= S/2.
#include "raw_kernels.hip.h"
#include "tiled_launch.h"

namespace deto {

int64_t launch_compress_raw(const CompressLaunch& a) {
    const KParams& p = a.p;
#ifdef DETO_TILED_ONLY_64_32
    return 0;
#else
    if (p.scheme == 0 || p.use_dct || 2 * p.k > p.s || !raw_compress(p, a.n)) return 0;
    const int quads = raw_compress_quads(p);
    const int wgs_cu = raw_compress_workgroups(p, a.n, a.grad_bf16);
    auto launch = [&](auto S_tag, auto Q_tag, auto kernel) -> int64_t {
        using G = RawGeom<decltype(S_tag)::value, decltype(Q_tag)::value>;
        const int64_t wgs = (a.n_chunks + G::kChunks - 1) / G::kChunks;
        if (wgs > 0x7FFFFFFF) return 0;
        const unsigned lds = raw_lds(G::compress_lds(p.k, a.idx != nullptr), wgs_cu);
        kernel<<<static_cast<unsigned>(wgs), kRawThreads, lds, a.stream>>>(
            p, a.n, a.n_chunks, a.grad, a.mom, a.idx, a.val, a.coeff_dbg);
        return a.n_chunks;
    };
#define X(S, Q)                                                                              \
    if (p.s == S && quads == Q)                                                              \
        return launch(std::integral_constant<int, S>{}, std::integral_constant<int, Q>{},    \
                      a.grad_bf16 ? compress_raw<S, Q, true> : compress_raw<S, Q, false>);
    DETO_RAW_COMPRESS_LIST(X)
#undef X
    return 0;
#endif
}

}  // namespace deto
