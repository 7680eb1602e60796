// sj_join_fp4_ip.hip -- the fused join kernels for 4-bit float rows (the Hamming
// front end's +-1 codes), inner-product test.
#include "sj_join_kernels.h"

namespace sjk {

SJ_JOIN_UNIT(fp4_ip, DT_FP4, MET_IP)

}  // namespace sjk
