// Indexed decompress on 64-chunk tiles, chunk size 96 (Appendix B sweep): the fast DCT ends in
// 3-point transforms.  The compress half at this chunk size runs with a wavefront per
// coefficient class.
#define DETO_S 96
#define DETO_K_LIST(X) DETO_LANE_TOPK_96(X)
#define DETO_DECOMPRESS_FN launch_decompress_idx_s96
#include "tiled_topk_impl.hip.h"
