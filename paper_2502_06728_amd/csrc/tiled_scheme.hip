// Tiled Striding / Random kernels (compress, and decompress without transmitted indices):
// compression rates 1/2 ... 1/8 at chunk sizes 64 and 32.
#define DETO_SCHEME_LIST(X) DETO_LANE_SCHEME(X)
#define DETO_COMPRESS_SCHEME_FN launch_compress_scheme
#define DETO_DECOMPRESS_SCHEME_FN launch_decompress_scheme
#include "tiled_scheme_impl.hip.h"
