// Tiled top-k compress and indexed decompress with the narrow payload: byte indices and
// bf16 or fp16 values (chunk size 64).
#define DETO_NARROW_LIST(X) DETO_LANE_16BIT_64(X)
#define DETO_COMPRESS_NARROW_FN launch_compress_topk_packed
#define DETO_DECOMPRESS_NARROW_FN launch_decompress_idx_packed
#include "tiled_narrow_impl.hip.h"
