// Wavefront-per-coefficient-class compress, chunk size 256, narrow payloads (four
// classes; up to k = 32 half_compress_256.hip comes first).
#define DETO_S 256
#define DETO_W 4
#define DETO_TOP(X)
#define DETO_SPLIT_NARROW_FN launch_compress_split_narrow_256
#include "split_narrow_impl.hip.h"
