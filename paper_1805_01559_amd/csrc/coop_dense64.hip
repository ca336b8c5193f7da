// Cooperative kernels in FP64 of the dense cost sources (launchers.h).
#include "launchers.h"

using namespace otk;
OT_COOP64(, DenseSrc<float>)
OT_COOP64(, DenseSrc<double>)
