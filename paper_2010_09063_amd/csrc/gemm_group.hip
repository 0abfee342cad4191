// One group of the tiled contraction's instantiations: compiled once per group with -DDP_GEMM_GROUP=<number>.
#include "problems.h"

#define DP_CAT_(a, b) a##b
#define DP_CAT(a, b) DP_CAT_(a, b)
DP_CAT(DP_GEMM_GROUP_, DP_GEMM_GROUP)()
