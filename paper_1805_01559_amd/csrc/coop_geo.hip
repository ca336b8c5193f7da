// Cooperative kernels of the geo cost sources (launchers.h).
#include "launchers.h"

using namespace otk;
OT_COOP(, GeoSrc)
OT_COOP(, EuclidSrc)
