// Wavefront-per-coefficient-class compress, chunk size 64, narrow payloads (two classes).
#define DETO_S 64
#define DETO_W 2
#define DETO_TOP(X) X(16)
#define DETO_SPLIT_NARROW_FN launch_compress_split_narrow_64
#include "split_narrow_impl.hip.h"
