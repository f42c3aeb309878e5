// The kernels of raw_decompress.hip: two-bit signs.
#define DETO_RAW_FN launch_decompress_raw_signs
#define DETO_RAW_OPT 0
#define DETO_RAW_SIGNS true
#include "raw_decompress.hip"
