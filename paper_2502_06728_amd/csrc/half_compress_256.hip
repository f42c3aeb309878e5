// Half-tile compress kernels of chunk size 256 (top-k, k <= 32; every format but two-bit signs).
#include "half_tile_kernels.hip.h"
#include "tiled_launch.h"

namespace deto {

int64_t launch_compress_halves_256(const CompressLaunch& a) {
    const KParams& p = a.p;
#ifdef DETO_TILED_ONLY_64_32
    return 0;
#else
    if (p.s != HalfGeom::S || p.scheme != 0 || !p.use_dct || p.val_dtype == 3 || p.k > 32) return 0;
    // one workgroup per full tile and one for the chunks left over (a partial tile)
    const int64_t grid64 = a.tiles + (a.n_chunks > a.tiles * kWave ? 1 : 0);
    if (a.tiles <= 0 || grid64 > 0x7FFFFFFF) return 0;
    const unsigned grid = static_cast<unsigned>(grid64);
#define LAUNCH(BF16, TOP, NARROW)                                                              \
    compress_halves<BF16, TOP, NARROW><<<grid, HalfGeom::kThreads, 0, a.stream>>>(             \
        p, a.tiles, a.n, a.n_chunks, a.grad, a.mom, a.idx, a.val, a.coeff_dbg)
    // (a launch with k <= 16 sorts out only every lane's 16 largest magnitudes, with k <= 32 the 32)
#define BY_TOP(BF16, NARROW)                                                                   \
    if (p.k <= 16) LAUNCH(BF16, 16, NARROW);                                                   \
    else LAUNCH(BF16, 32, NARROW)
    const bool narrow = p.val_dtype != 0 || p.idx_u8;
    if (a.grad_bf16) {
        if (narrow) { BY_TOP(true, true); }
        else { BY_TOP(true, false); }
    } else {
        if (narrow) { BY_TOP(false, true); }
        else { BY_TOP(false, false); }
    }
#undef BY_TOP
#undef LAUNCH
    return a.n_chunks;   // the tail chunks ride along
#endif
}

}  // namespace deto
