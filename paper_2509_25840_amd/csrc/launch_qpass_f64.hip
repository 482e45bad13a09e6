// Launches of k_qpass in FP64.
#include "launch_qpass.h"

namespace chfpe {

CHFPE_INST(double, double, true, EPI_ACC, FQ, FQ)
CHFPE_INST(double, double, false, EPI_ACC, FX, FQ)
CHFPE_INST(double, float, false, EPI_ACC, FX, FQ)
CHFPE_INST_STAGE(double, EPI_OUT)
CHFPE_INST_STAGE(double, EPI_H1)
CHFPE_INST_STAGE(double, EPI_H2)
CHFPE_INST_STAGE(double, EPI_H4)

}  // namespace chfpe
