// The kernels of split_decompress.hip for Decoupled AdamW with amsgrad.
#define DETO_SPLIT_FN launch_decompress_split_amsgrad
#define DETO_SPLIT_NARROW false
#define DETO_SPLIT_AMSGRAD true
#include "split_decompress.hip"
