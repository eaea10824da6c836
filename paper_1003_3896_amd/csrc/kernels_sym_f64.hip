// Symmetric pair kernels of the F64 family (templates in pair_sym.h).
#include "pair_sym.h"

namespace nb {
hipError_t launch_sym_f64(const Args& a, const SymBand& b, int grid, bool mask, bool pot, hipStream_t s) {
  return launch_sym_family<FAM_F64>(a, b, grid, mask, pot, s);
}
}  // namespace nb
