// Launch of the pair kernels (one-sided: kernels_pair_{f32,ds,f64,dl}.hip, symmetric:
// kernels_sym_{f32,ds,f64,dl}.hip).
#include "nb_internal.h"

namespace nb {

bool tile_supported(int family, const TileCfg& t) {
  const bool kw = (t.k == 1 && (t.w == 4 || t.w == 2 || (family != FAM_DL && t.w == 1))) ||
                  (t.k == 2 && (t.w == 2 || t.w == 4));
  const bool ph = t.phase == 0 || ((family == FAM_F32 || family == FAM_DS) &&
                                   ((t.k == 1 && t.w == 4 && t.tile == 256) ||
                                    (t.k == 2 && t.w == 2 && t.tile == 256) || (t.k == 2 && t.w == 4)));
  return kw && ph && (t.tile == 128 || t.tile == 256) && t.bpc >= 1 && t.bpc <= 8;
}

bool wide_compiled(int family, const TileCfg& t) {
  return (family == FAM_F32 || family == FAM_DS) && t.w == 4 && t.tile == 128;
}

PairFn pair_kernel(int prec, const TileCfg& t, bool mask, bool potmode) {
  if (prec == 4) return pair_kernel_dl(t, true, mask, potmode);
  if (prec == 3) return pair_kernel_f64(t, true, mask, potmode);
  if (prec == 2) return pair_kernel_ds(t, true, mask, potmode);
  return pair_kernel_f32(t, prec != 0, mask, potmode);  // pure FP32 (0) keeps one FP32 sum
}

hipError_t launch_pair(PairFn fn, const Args& a, int grid, bool kick, hipStream_t s) {
  hipLaunchKernelGGL(fn, dim3(grid), dim3(kBlock), 0, s, a, kick ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_pair_sym(const Args& a, const SymBand& b, int grid, bool mask, bool potmode, hipStream_t s) {
  switch (a.prec) {
    case 4: return launch_sym_dl(a, b, grid, mask, potmode, s);
    case 3: return launch_sym_f64(a, b, grid, mask, potmode, s);
    case 2: return launch_sym_ds(a, b, grid, mask, potmode, s);
    default: return launch_sym_f32(a, b, grid, mask, potmode, s);
  }
}

}  // namespace nb
