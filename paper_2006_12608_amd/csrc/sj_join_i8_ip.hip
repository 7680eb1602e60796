// sj_join_i8_ip.hip -- the fused join kernels for int8 rows, inner-product test.
#include "sj_join_kernels.h"

namespace sjk {

SJ_JOIN_UNIT(i8_ip, DT_I8, MET_IP)

}  // namespace sjk
