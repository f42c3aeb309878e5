// The kernels of split_decompress_narrow.hip for Decoupled AdamW with amsgrad.
#define DETO_SPLIT_FN launch_decompress_split_narrow_amsgrad
#define DETO_SPLIT_NARROW true
#define DETO_SPLIT_AMSGRAD true
#include "split_decompress.hip"
