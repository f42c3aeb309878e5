// Lane-per-chunk, wavefront-per-coefficient-class compress kernels (chunk size 192: 4 classes;
// top-k selection, fp32 values + int32 indices, k <= 96).
#include "split_kernels.hip.h"
#include "tiled_launch.h"

namespace deto {

int64_t launch_compress_split_192(const CompressLaunch& a) {
    const KParams& p = a.p;
#ifdef DETO_TILED_ONLY_64_32
    return 0;
#else
    if (p.s != 192 || p.scheme != 0 || !p.use_dct || p.val_dtype != 0 || p.idx_u8 || p.k > 96)
        return 0;
    const int64_t tiles = (a.n / p.s) / kWave;
    // one workgroup per full tile and one for the chunks left over (a partial tile)
    const int64_t grid64 = tiles + (a.n_chunks > tiles * kWave ? 1 : 0);
    if (tiles <= 0 || grid64 > 0x7FFFFFFF) return 0;
    const unsigned grid = static_cast<unsigned>(grid64);
    constexpr int kThreads = SplitGeom<192, 4>::kThreads;
    // a launch with k <= 16 (k <= 32) sorts out only every lane's 16 (32) largest magnitudes
#define LAUNCH(BF16, TOP)                                                                  \
    compress_split<192, 4, BF16, TOP><<<grid, kThreads, 0, a.stream>>>(                 \
        p, tiles, a.n, a.n_chunks, a.grad, a.mom, a.idx, a.val, a.coeff_dbg)
    if (p.k <= 16) {
        if (a.grad_bf16) LAUNCH(true, 16);
        else LAUNCH(false, 16);
    } else if (p.k <= 32) {
        if (a.grad_bf16) LAUNCH(true, 32);
        else LAUNCH(false, 32);
    } else {
        if (a.grad_bf16) LAUNCH(true, 0);
        else LAUNCH(false, 0);
    }
#undef LAUNCH
    return a.n_chunks;   // the tail chunks ride along
#endif
}

}  // namespace deto
