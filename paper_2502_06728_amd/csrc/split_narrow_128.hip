// Wavefront-per-coefficient-class compress, chunk size 128, narrow payloads (four classes at every shard
// size: up to 4 % slower than two on large shards, 4 - 13 % faster on small ones; one choice keeps
// one set of kernels, where fp32 + int32 has both).
#define DETO_S 128
#define DETO_W 4
#define DETO_TOP(X) X(16)
#define DETO_SPLIT_NARROW_FN launch_compress_split_narrow_128
#include "split_narrow_impl.hip.h"
