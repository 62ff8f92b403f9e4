// Host build of the ghost-layer rule, for a CPU test against its definition.
#include <hip/hip_runtime.h>

#include "../../paper_1106_0785_amd/csrc/lbm_kernels.h"

using namespace lbm;

extern "C" void host_resolve(int i, int n, int bc_lo, int bc_hi, int side_lo, int* out) {
  const Src s = resolve(i, n, bc_lo, bc_hi, side_lo);
  out[0] = s.idx;
  out[1] = s.mode;
  out[2] = s.side;
  out[3] = s.kind;
}
