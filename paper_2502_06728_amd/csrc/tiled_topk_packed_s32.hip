// Tiled top-k compress and indexed decompress with byte indices and bf16 or fp16 values at
// chunk size 32, the chunk size of the paper's experiments ("Overall Setup"), for the
// compression rates 1/2 ... 1/32.
#define DETO_NARROW_LIST(X) DETO_LANE_16BIT_32(X)
#define DETO_COMPRESS_NARROW_FN launch_compress_topk_packed_s32
#define DETO_DECOMPRESS_NARROW_FN launch_decompress_idx_packed_s32
#include "tiled_narrow_impl.hip.h"
