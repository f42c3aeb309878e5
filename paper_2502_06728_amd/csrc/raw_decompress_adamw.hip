// The kernels of raw_decompress.hip: Decoupled AdamW.
#define DETO_RAW_FN launch_decompress_raw_adamw
#define DETO_RAW_OPT 1
#define DETO_RAW_SIGNS false
#include "raw_decompress.hip"
