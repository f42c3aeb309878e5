// Striding / Random with a narrow payload at chunk size 32, rates 1/2 ... 1/32: the setting of
// the paper's experiments (chunk size 32, only signs synchronised, "Overall Setup").
#define DETO_SCHEME_NARROW_LIST(X) DETO_LANE_SCHEME_NARROW_32(X)
#define DETO_COMPRESS_SCHEME_NARROW_FN launch_compress_scheme_narrow_s32
#define DETO_DECOMPRESS_SCHEME_NARROW_FN launch_decompress_scheme_narrow_s32
#include "tiled_scheme_narrow_impl.hip.h"
