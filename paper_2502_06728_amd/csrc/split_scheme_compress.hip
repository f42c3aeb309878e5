// Striding / Random compress on the wavefront-per-coefficient-class kernels: on coefficients, every
// payload format, any k <= S/2, for what the lane-per-chunk kernels are not instantiated for
// (chunk sizes above 64, low rates with narrow payloads).
#include "split_kernels.hip.h"
#include "tiled_launch.h"

namespace deto {

int64_t launch_compress_split_scheme(const CompressLaunch& a) {
    const KParams& p = a.p;
#ifdef DETO_TILED_ONLY_64_32
    return 0;
#else
    if (p.scheme == 0 || !p.use_dct || 2 * p.k > p.s) return 0;
    const int64_t tiles = (a.n / p.s) / kWave;
    // one workgroup per full tile and one for the chunks left over (a partial tile)
    const int64_t grid64 = tiles + (a.n_chunks > tiles * kWave ? 1 : 0);
    if (grid64 > 0x7FFFFFFF) return 0;
    const unsigned grid = static_cast<unsigned>(grid64);
#define X(S, W)                                                                                 \
    if (p.s == S) {                                                                             \
        if (a.grad_bf16)                                                                        \
            compress_split<S, W, true, 0, true, true><<<grid, W * kWave, 0, a.stream>>>(        \
                p, tiles, a.n, a.n_chunks, a.grad, a.mom, a.idx, a.val, a.coeff_dbg);           \
        else                                                                                    \
            compress_split<S, W, false, 0, true, true><<<grid, W * kWave, 0, a.stream>>>(       \
                p, tiles, a.n, a.n_chunks, a.grad, a.mom, a.idx, a.val, a.coeff_dbg);           \
        return a.n_chunks;   /* the tail chunks ride along */                                   \
    }
    X(16, 2) X(32, 2) X(64, 2) X(96, 4) X(128, 4) X(192, 4) X(256, 4)
#undef X
    return 0;
#endif
}

}  // namespace deto
