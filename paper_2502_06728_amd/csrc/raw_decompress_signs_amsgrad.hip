// The kernels of raw_decompress.hip: two-bit signs, Decoupled AdamW with amsgrad.
#define DETO_RAW_FN launch_decompress_raw_signs_amsgrad
#define DETO_RAW_OPT 2
#define DETO_RAW_SIGNS true
#include "raw_decompress.hip"
