// The flux-limited step kernel of the version-3 equilibria alone, for a test
// of what the compiler makes of it.
#include "../../paper_1106_0785_amd/csrc/lbm_kernels.h"

template __global__ void lbm::k_step_fused<3, false, 4, 2, true>(Field, const Hot*, const Cold*, MarchGeom, int*);
