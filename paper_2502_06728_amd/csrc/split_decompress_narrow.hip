// The kernels of split_decompress.hip for every other payload format (16-bit values or two-bit
// signs, byte or int32 indices, fp32 values with byte indices), chosen at run time.
#define DETO_SPLIT_FN launch_decompress_split_narrow
#define DETO_SPLIT_NARROW true
#include "split_decompress.hip"
