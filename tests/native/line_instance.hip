// The persistent line kernel of the version-3 equilibria at region 128 alone,
// for a test of what the compiler makes of it.
#include "../../paper_1106_0785_amd/csrc/lbm_batch_kernels.h"

template __global__ void lbm::k_batch_line_persistent<3, 128>(double*, double*, const LineInst*, const LineChunk*, int,
                                                              const int*, int, int, int*, int*, long long);
