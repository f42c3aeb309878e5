// Shared body of the split_narrow_*.hip units: the wavefront-per-coefficient-class compress
// kernels of chunk size DETO_S with DETO_W classes for 16-bit values (byte or int32 indices)
// and fp32 values with byte indices, any k <= DETO_S / 2.  Defines the launcher DETO_SPLIT_NARROW_FN.
// DETO_TOP(X): the partial-sort lengths, ascending; a launch takes the first that holds its k.
#include "split_kernels.hip.h"
#include "tiled_launch.h"

namespace deto {

int64_t DETO_SPLIT_NARROW_FN(const CompressLaunch& a) {
    const KParams& p = a.p;
#ifdef DETO_TILED_ONLY_64_32
    return 0;
#else
    if (p.s != DETO_S || p.scheme != 0 || !p.use_dct || 2 * p.k > DETO_S) return 0;
    if (p.val_dtype == 3 || (p.val_dtype == 0 && !p.idx_u8)) return 0;
    const int64_t tiles = (a.n / p.s) / kWave;
    // one workgroup per full tile and one for the chunks left over (a partial tile)
    const int64_t grid64 = tiles + (a.n_chunks > tiles * kWave ? 1 : 0);
    if (tiles <= 0 || grid64 > 0x7FFFFFFF) return 0;
    const unsigned grid = static_cast<unsigned>(grid64);
    constexpr int kThreads = SplitGeom<DETO_S, DETO_W>::kThreads;
#define LAUNCH(BF16, TOP)                                                                  \
    compress_split<DETO_S, DETO_W, BF16, TOP, true><<<grid, kThreads, 0, a.stream>>>(      \
        p, tiles, a.n, a.n_chunks, a.grad, a.mom, a.idx, a.val, a.coeff_dbg)
#define X(TOP)                                                                             \
    if (p.k <= TOP) {                                                                      \
        if (a.grad_bf16) LAUNCH(true, TOP);                                                \
        else LAUNCH(false, TOP);                                                           \
        return a.n_chunks;   /* the tail chunks ride along */                              \
    }
    DETO_TOP(X)
#undef X
    if (a.grad_bf16) LAUNCH(true, 0);
    else LAUNCH(false, 0);
#undef LAUNCH
    return a.n_chunks;
#endif
}

}  // namespace deto
