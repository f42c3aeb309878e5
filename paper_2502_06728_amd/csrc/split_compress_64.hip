// Lane-per-chunk, wavefront-per-coefficient-class compress kernels (chunk size 64: 2 classes,
// 4 on very small shards; top-k selection, fp32 values + int32 indices, k <= 32), for small shards: the
// wavefronts share a tile, so a tile is done sooner than on the lane-per-chunk kernel, which wins on
// throughput once the launch is many occupancy rounds long.  Also for any k the lane-per-chunk
// kernel is not instantiated for, at every shard size.
#include "split_kernels.hip.h"
#include "tiled_launch.h"

namespace deto {

int64_t launch_compress_split_64(const CompressLaunch& a) {
    const KParams& p = a.p;
#ifdef DETO_TILED_ONLY_64_32
    return 0;
#else
    if (p.s != 64 || p.scheme != 0 || !p.use_dct || p.val_dtype != 0 || p.idx_u8 || p.k > 32)
        return 0;
    const int64_t tiles = (a.n / p.s) / kWave;
    // the lane-per-chunk kernels take k as a template argument: at any other k this kernel
    // serves every shard size
    const bool lane_per_chunk_has_k = p.k == 1 || p.k == 2 || p.k == 4 || p.k == 8 || p.k == 16 ||
                                      p.k == 32;
    if (tiles <= 0 || (lane_per_chunk_has_k && tiles > small_shard_tiles())) return 0;
    // one workgroup per full tile and one for the chunks left over (a partial tile)
    const int64_t grid64 = tiles + (a.n_chunks > tiles * kWave ? 1 : 0);
    if (grid64 > 0x7FFFFFFF) return 0;
    const unsigned grid = static_cast<unsigned>(grid64);
#define LAUNCH_CLASSES(W, BF16, TOP)                                                       \
    compress_split<64, W, BF16, TOP><<<grid, SplitGeom<64, W>::kThreads, 0, a.stream>>>(   \
        p, tiles, a.n, a.n_chunks, a.grad, a.mom, a.idx, a.val, a.coeff_dbg)
    // a launch with k <= 16 sorts out only every lane's 16 largest magnitudes
#define LAUNCH(W)                                                                          \
    if (p.k <= 16) {                                                                       \
        if (a.grad_bf16) LAUNCH_CLASSES(W, true, 16);                                      \
        else LAUNCH_CLASSES(W, false, 16);                                                 \
    } else {                                                                               \
        if (a.grad_bf16) LAUNCH_CLASSES(W, true, 0);                                       \
        else LAUNCH_CLASSES(W, false, 0);                                                  \
    }
    // up to two tiles per CU a tile's own duration is what a launch takes: four classes shorten it (2.0 M
    // parameters, 64/1 11.5 -> 10.3 us, 64/8 12.0 -> 10.4, 64/32 13.5 -> 12.7; 3 M 64/16 13.2, 13.9;
    // 8 M 23.1, 25.8).  Both give the same bits: with class_sum's fused additions four classes round
    // as two do.
    if (tiles <= 512) { LAUNCH(4) }
    else { LAUNCH(2) }
#undef LAUNCH
#undef LAUNCH_CLASSES
    return a.n_chunks;   // the tail chunks ride along
#endif
}

}  // namespace deto
