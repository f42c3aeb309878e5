// The kernels of split_scheme_decompress.hip for Decoupled AdamW with amsgrad.
#define DETO_SPLIT_FN launch_decompress_split_scheme_amsgrad
#define DETO_SPLIT_AMSGRAD true
#include "split_scheme_decompress.hip"
