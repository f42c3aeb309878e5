// The kernels of raw_decompress.hip: two-bit signs, Decoupled AdamW.
#define DETO_RAW_FN launch_decompress_raw_signs_adamw
#define DETO_RAW_OPT 1
#define DETO_RAW_SIGNS true
#include "raw_decompress.hip"
