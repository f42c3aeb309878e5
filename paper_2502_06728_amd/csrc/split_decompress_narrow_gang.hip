// The kernels of split_decompress_narrow.hip on tiles in gangs (run_log2): AdamW on large launches.
#define DETO_SPLIT_FN launch_decompress_split_narrow_gang
#define DETO_SPLIT_NARROW true
#define DETO_SPLIT_GANG true
#define DETO_SPLIT_SHAPES(X) X(64, 4) X(128, 4)
#include "split_decompress.hip"
