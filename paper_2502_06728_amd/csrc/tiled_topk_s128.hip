// Indexed decompress on 64-chunk tiles, chunk size 128 (one wavefront per SIMD: a chunk
// occupies 128 VGPRs of its lane).  The compress half at this chunk size runs with a
// wavefront per coefficient class.
#define DETO_S 128
#define DETO_K_LIST(X) DETO_LANE_TOPK_128(X)
#define DETO_DECOMPRESS_FN launch_decompress_idx_s128
#include "tiled_topk_impl.hip.h"
