// Tiled top-k compress and indexed decompress with the ternary payload: byte indices and the
// signs of the kept coefficients, two bits per entry.  Chunk size 64 at rates 1/2 and 1/4, and
// chunk size 32 at rates 1/2 ... 1/32: sign-only synchronisation at chunk size 32 is the
// configuration of the paper's experiments ("Overall Setup").
#define DETO_NARROW_TERNARY
#define DETO_NARROW_LIST(X) DETO_LANE_SIGNS(X)
#define DETO_COMPRESS_NARROW_FN launch_compress_topk_ternary
#define DETO_DECOMPRESS_NARROW_FN launch_decompress_idx_ternary
#include "tiled_narrow_impl.hip.h"
