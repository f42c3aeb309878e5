// Direct sums on the matrix cores: see direct_kernels.hip.h.
#include "direct_kernels.hip.h"
#include "tiled_launch.h"

namespace deto {

int64_t launch_compress_direct(const CompressLaunch& a) {
    const KParams& p = a.p;
    if (!direct_compress(p) || few_direct(p, a.n_chunks)) return 0;
#define X(S)                                                                                       \
    if (p.s == S) {                                                                                \
        constexpr int NC = DirectGeom<S>::NC;                                                      \
        const int64_t tiles = (a.n / S) / NC;                                                      \
        const int64_t grid64 = tiles + (tiles * NC < a.n_chunks ? 1 : 0);                          \
        if (grid64 > 0x7FFFFFFF) return 0;                                                         \
        const unsigned grid = static_cast<unsigned>(grid64);                                       \
        if (a.grad_bf16)                                                                           \
            compress_direct<S, true><<<grid, DirectGeom<S>::kThreads, 0, a.stream>>>(              \
                p, tiles, a.n, a.n_chunks, a.grad, a.mom, a.idx, a.val, a.coeff_dbg);              \
        else                                                                                       \
            compress_direct<S, false><<<grid, DirectGeom<S>::kThreads, 0, a.stream>>>(             \
                p, tiles, a.n, a.n_chunks, a.grad, a.mom, a.idx, a.val, a.coeff_dbg);              \
        return a.n_chunks;                                                                         \
    }
    DETO_DIRECT_COMPRESS_LIST(X)
#undef X
    return 0;
}

}  // namespace deto
