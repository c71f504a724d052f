// The FP64 forward of psi_tri.h at chi padded to 64.
#include "psi_tri.h"

namespace nqs {
hipError_t launch_tri_64(const TriParams& P, const uint64_t* m, int64_t R, double* lphi, int8_t* sphi, hipStream_t st,
                         const PsiStates<double>& X, int mode, double* phs) {
  return run_tri_ch<double, 64>(P, m, R, lphi, sphi, st, X, mode, phs);
}
}  // namespace nqs
