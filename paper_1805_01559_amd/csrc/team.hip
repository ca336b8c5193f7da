// The team kernel of the batched engine (team_kernels.h), compiled on its own.
#include "team_kernels.h"

using namespace otk;

const void* otk_team_kernel() { return (const void*)k_team; }
