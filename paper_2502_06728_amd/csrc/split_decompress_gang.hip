// The kernels of split_decompress.hip on tiles in gangs (run_log2): large launches.
#define DETO_SPLIT_FN launch_decompress_split_gang
#define DETO_SPLIT_NARROW false
#define DETO_SPLIT_GANG true
#define DETO_SPLIT_SHAPES(X) X(32, 2) X(32, 4) X(64, 2) X(64, 4) X(128, 4)
#include "split_decompress.hip"
