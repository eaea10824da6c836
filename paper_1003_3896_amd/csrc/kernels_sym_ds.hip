// Symmetric pair kernels of the DS family (templates in pair_sym.h).
#include "pair_sym.h"

namespace nb {
hipError_t launch_sym_ds(const Args& a, const SymBand& b, int grid, bool mask, bool pot, hipStream_t s) {
  return launch_sym_family<FAM_DS>(a, b, grid, mask, pot, s);
}
}  // namespace nb
