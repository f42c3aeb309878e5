// Decompress-and-update on the wavefront-per-coefficient-class kernels (transmitted indices; plain
// SGD update or Decoupled AdamW; any k): launchers for fp32 values + int32 indices, and
// (split_decompress_narrow.hip) for every other payload format; both again for amsgrad.
#ifndef DETO_SPLIT_FN
#define DETO_SPLIT_FN launch_decompress_split
#define DETO_SPLIT_NARROW false
#endif
#ifndef DETO_SPLIT_AMSGRAD
#define DETO_SPLIT_AMSGRAD false
#endif
#ifndef DETO_SPLIT_GANG
#define DETO_SPLIT_GANG false
#define DETO_SPLIT_SHAPES(X) \
    X(16, 2) X(32, 2) X(32, 4) X(64, 2) X(64, 4) X(96, 2) X(96, 4) X(128, 2) X(128, 4) X(192, 4) X(256, 4)
#endif
#include "split_kernels.hip.h"
#include "tiled_launch.h"

namespace deto {

int64_t DETO_SPLIT_FN(const DecompressLaunch& a, int classes) {
    const KParams& p = a.p;
#ifdef DETO_TILED_ONLY_64_32
    return 0;
#else
    if (!a.idx || DETO_SPLIT_NARROW != (p.val_dtype != 0 || p.idx_u8)) return 0;
    if (DETO_SPLIT_AMSGRAD != (p.adam && p.amsgrad)) return 0;
    if (DETO_SPLIT_GANG && !decompress_gangs(p, a.n, a.param_bf16, classes)) return 0;
    const int64_t tiles = (a.n / p.s) / kWave;
    // one workgroup per full tile and one for the chunks left over (a partial tile)
    const int64_t grid64 = tiles + (a.n_chunks > tiles * kWave ? 1 : 0);
    if (grid64 > 0x7FFFFFFF) return 0;
    const unsigned grid = static_cast<unsigned>(grid64);
    const unsigned spare = spare_lds(a, classes);
#define LAUNCH(S, W, BF16)                                                                      \
    decompress_split<S, W, BF16, DETO_SPLIT_NARROW, false, DETO_SPLIT_AMSGRAD, DETO_SPLIT_GANG> \
        <<<grid, W * kWave, spare, a.stream>>>(p, tiles, a.n, a.n_chunks, a.idx, a.idx_stride,  \
                                               a.val, a.val_stride, a.params, a.adam,           \
                                               a.presign_dbg)
    // (two classes in gangs: fp32 parameters only)
#define X(S, W)                                                                                 \
    if (p.s == S && classes == W && !(DETO_SPLIT_GANG && W == 2 && a.param_bf16)) {             \
        if (a.param_bf16) LAUNCH(S, W, (!(DETO_SPLIT_GANG && W == 2)));                         \
        else LAUNCH(S, W, false);                                                               \
        return a.n_chunks;   /* the tail chunks ride along */                                   \
    }
    DETO_SPLIT_SHAPES(X)
#undef X
#undef LAUNCH
    return 0;
#endif
}

}  // namespace deto
