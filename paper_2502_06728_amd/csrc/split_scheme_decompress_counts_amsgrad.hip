// The same, Decoupled AdamW with amsgrad.
#define DETO_SPLIT_FN launch_decompress_split_scheme_counts_amsgrad
#define DETO_SPLIT_AMSGRAD true
#define DETO_SPLIT_COUNT true
#include "split_scheme_decompress.hip"
