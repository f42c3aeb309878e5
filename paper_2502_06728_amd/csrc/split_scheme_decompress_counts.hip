// The kernels of split_scheme_decompress.hip: two-bit signs of many replicas, counted a word at a time.
#define DETO_SPLIT_FN launch_decompress_split_scheme_counts
#define DETO_SPLIT_AMSGRAD false
#define DETO_SPLIT_COUNT true
#include "split_scheme_decompress.hip"
