// Tiled top-k compress and indexed decompress, chunk size 32.
#define DETO_S 32
#define DETO_K_LIST(X) DETO_LANE_TOPK_32(X)
#define DETO_COMPRESS_FN launch_compress_topk_s32
#define DETO_DECOMPRESS_FN launch_decompress_idx_s32
#include "tiled_topk_impl.hip.h"
