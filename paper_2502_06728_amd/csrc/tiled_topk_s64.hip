// Tiled top-k compress and indexed decompress, chunk size 64.
#define DETO_S 64
#define DETO_K_LIST(X) DETO_LANE_TOPK_64(X)
#define DETO_COMPRESS_FN launch_compress_topk_s64
#define DETO_DECOMPRESS_FN launch_decompress_idx_s64
#include "tiled_topk_impl.hip.h"
