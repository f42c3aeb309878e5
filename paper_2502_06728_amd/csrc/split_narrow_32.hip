// Wavefront-per-coefficient-class compress, chunk size 32, narrow payloads (two classes).
#define DETO_S 32
#define DETO_W 2
#define DETO_TOP(X)
#define DETO_SPLIT_NARROW_FN launch_compress_split_narrow_32
#include "split_narrow_impl.hip.h"
