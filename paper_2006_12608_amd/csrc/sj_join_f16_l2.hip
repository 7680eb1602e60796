// sj_join_f16_l2.hip -- the fused join kernels for f16 rows, squared-Euclidean test.
#include "sj_join_kernels.h"

namespace sjk {

SJ_JOIN_UNIT(f16_l2, DT_F16, MET_L2)

}  // namespace sjk
