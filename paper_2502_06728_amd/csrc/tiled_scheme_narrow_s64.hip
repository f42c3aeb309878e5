// Striding / Random with a narrow payload at chunk size 64, rates 1/2 ... 1/16.
#define DETO_SCHEME_NARROW_LIST(X) DETO_LANE_SCHEME_NARROW_64(X)
#define DETO_COMPRESS_SCHEME_NARROW_FN launch_compress_scheme_narrow_s64
#define DETO_DECOMPRESS_SCHEME_NARROW_FN launch_decompress_scheme_narrow_s64
#include "tiled_scheme_narrow_impl.hip.h"
