// Launches of k_qpass in FP32.
#include "launch_qpass.h"

namespace chfpe {

CHFPE_INST(float, float, true, EPI_ACC, FQ, FQ)
CHFPE_INST_STAGE(float, EPI_H1)
CHFPE_INST_STAGE(float, EPI_H2)
CHFPE_INST_STAGE(float, EPI_H4)

}  // namespace chfpe
