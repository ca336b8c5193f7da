// Cooperative kernels of the dense cost sources (launchers.h).
#include "launchers.h"

using namespace otk;
OT_COOP(, DenseSrc<float>)
OT_COOP(, DenseSrc<double>)
