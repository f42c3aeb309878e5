// Wavefront-per-coefficient-class compress, chunk size 192, narrow payloads (four classes).
#define DETO_S 192
#define DETO_W 4
#define DETO_TOP(X) X(16) X(32)
#define DETO_SPLIT_NARROW_FN launch_compress_split_narrow_192
#include "split_narrow_impl.hip.h"
