// Symmetric pair kernels of the F32 family (templates in pair_sym.h).
#include "pair_sym.h"

namespace nb {
hipError_t launch_sym_f32(const Args& a, const SymBand& b, int grid, bool mask, bool pot, hipStream_t s) {
  return launch_sym_family<FAM_F32>(a, b, grid, mask, pot, s);
}
}  // namespace nb
