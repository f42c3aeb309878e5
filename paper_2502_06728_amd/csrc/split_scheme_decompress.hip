// Striding / Random decompress-and-update without transmitted indices on the
// wavefront-per-coefficient-class kernels: on coefficients, every payload format, any k <= S/2,
// plain SGD update or Decoupled AdamW, for what the lane-per-chunk kernels are not instantiated for.  (In units of
// their own: amsgrad, split_scheme_decompress_amsgrad.hip, and counted signs, split_scheme_decompress_counts.hip.)
#ifndef DETO_SPLIT_FN
#define DETO_SPLIT_FN launch_decompress_split_scheme
#define DETO_SPLIT_AMSGRAD false
#endif
#ifndef DETO_SPLIT_COUNT
#define DETO_SPLIT_COUNT false
#endif
#include "split_kernels.hip.h"
#include "tiled_launch.h"

namespace deto {

int64_t DETO_SPLIT_FN(const DecompressLaunch& a, int classes) {
    const KParams& p = a.p;
#ifdef DETO_TILED_ONLY_64_32
    return 0;
#else
    if (a.idx || p.scheme == 0 || !p.use_dct || 2 * p.k > p.s) return 0;
    if (DETO_SPLIT_AMSGRAD != (p.adam && p.amsgrad) || DETO_SPLIT_COUNT != (p.count_signs != 0)) return 0;
    const int64_t tiles = (a.n / p.s) / kWave;
    // one workgroup per full tile and one for the chunks left over (a partial tile)
    const int64_t grid64 = tiles + (a.n_chunks > tiles * kWave ? 1 : 0);
    if (grid64 > 0x7FFFFFFF) return 0;
    const unsigned grid = static_cast<unsigned>(grid64);
    const unsigned spare = spare_lds(a, classes);
#define LAUNCH(S, W, BF16)                                                                      \
    decompress_split<S, W, BF16, true, true, DETO_SPLIT_AMSGRAD, false, DETO_SPLIT_COUNT>       \
        <<<grid, W * kWave, spare, a.stream>>>(p, tiles, a.n, a.n_chunks, nullptr, 0, a.val,        \
                                           a.val_stride, a.params, a.adam, a.presign_dbg)
#define X(S, W)                                                                                 \
    if (p.s == S && classes == W) {                                                             \
        if (a.param_bf16) LAUNCH(S, W, true);                                                   \
        else LAUNCH(S, W, false);                                                               \
        return a.n_chunks;   /* the tail chunks ride along */                                   \
    }
    X(16, 2) X(32, 2) X(32, 4) X(64, 2) X(64, 4) X(96, 4) X(128, 4) X(192, 4) X(256, 4)
#undef X
#undef LAUNCH
    return 0;
#endif
}

}  // namespace deto
