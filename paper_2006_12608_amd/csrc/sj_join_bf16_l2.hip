// sj_join_bf16_l2.hip -- the fused join kernels for bf16 rows, squared-Euclidean test.
#include "sj_join_kernels.h"

namespace sjk {

SJ_JOIN_UNIT(bf16_l2, DT_BF16, MET_L2)

}  // namespace sjk
