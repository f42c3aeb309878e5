// The kernels of raw_decompress.hip: Decoupled AdamW with amsgrad.
#define DETO_RAW_FN launch_decompress_raw_amsgrad
#define DETO_RAW_OPT 2
#define DETO_RAW_SIGNS false
#include "raw_decompress.hip"
