// Cooperative kernels of the rates cost sources (launchers.h).
#include "launchers.h"

using namespace otk;
OT_COOP(, RatesSrc<float>)
OT_COOP(, RatesSrc<double>)
