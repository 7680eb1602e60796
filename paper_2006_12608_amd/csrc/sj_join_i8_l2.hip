// sj_join_i8_l2.hip -- the fused join kernels for int8 rows, squared-Euclidean test.
#include "sj_join_kernels.h"

namespace sjk {

SJ_JOIN_UNIT(i8_l2, DT_I8, MET_L2)

}  // namespace sjk
