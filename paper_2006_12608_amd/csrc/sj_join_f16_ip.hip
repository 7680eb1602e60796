// sj_join_f16_ip.hip -- the fused join kernels for f16 rows, inner-product test.
#include "sj_join_kernels.h"

namespace sjk {

SJ_JOIN_UNIT(f16_ip, DT_F16, MET_IP)

}  // namespace sjk
