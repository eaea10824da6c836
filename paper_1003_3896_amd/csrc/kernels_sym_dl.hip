// Symmetric pair kernels of the DL family (templates in pair_sym.h).
#include "pair_sym.h"

namespace nb {
hipError_t launch_sym_dl(const Args& a, const SymBand& b, int grid, bool mask, bool pot, hipStream_t s) {
  return launch_sym_family<FAM_DL>(a, b, grid, mask, pot, s);
}
}  // namespace nb
