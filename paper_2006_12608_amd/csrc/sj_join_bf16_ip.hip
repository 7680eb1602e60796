// sj_join_bf16_ip.hip -- the fused join kernels for bf16 rows, inner-product test.
#include "sj_join_kernels.h"

namespace sjk {

SJ_JOIN_UNIT(bf16_ip, DT_BF16, MET_IP)

}  // namespace sjk
