// The marching kernels that hand moments from pass to pass (march.h), of one
// storage form and field kind (STEP_FORM, MARCH_FIELD).
#include <atomic>

#include "march.h"

namespace tflbm {

// Launches one pass, or with `occ` only reports its resident workgroups per CU.
template <int P, int KF, bool CAP, int NS, bool MI, bool MO, bool G0, int PF, int U>
static hipError_t go(const StepArgs &A, int *occ, hipStream_t s) {
  auto *k = march_kernel<P, KF, CAP, NS, MI, MO, G0, PF, U>;
  if (occ) {
    static std::atomic<int> known{0};  // a property of the kernel
    hipError_t e = hipSuccess;
    *occ = known.load();
    if (*occ == 0 && (e = hipOccupancyMaxActiveBlocksPerMultiprocessor(occ, k, 64, 0)) == hipSuccess) known = *occ;
    return e;
  }
  k<<<dim3(8 * A.per_xcd), dim3(64), 0, s>>>(A);
  return hipGetLastError();
}

// Rows in flight (PF) and rows per turn of the loop (U) of each pass: as much of
// both as the 256 registers of two wavefronts per SIMD hold.  Measured at 4096^2,
// us per step: FP32 three steps PF, U = 1, 1 75.4; 1, 6 71.7; 3, 3 70.4; 3, 6
// 68.5 (which needs g = 0's shorter collision); FP64 1, 6 136.3; 3, 3 132.5.
// Two steps at 2048^2: FP32 3, 6 23.6; 2, 6 23.1; FP64 2, 6 36.7; 3, 6 35.7; three
// wavefronts per SIMD (1, 6 with chunks for twelve per CU) 30.3 and 39.0.
template <int P, int KF, bool CAP, bool G0> static hipError_t pass(int kind, const StepArgs &A, int *occ, hipStream_t s) {
  constexpr bool F32 = P == kF32;
  switch (kind) {
    case kPopMom2: return go<P, KF, CAP, 2, false, true, false, 1, 3>(A, occ, s);
    case kMom2: return go<P, KF, CAP, 2, true, true, G0, F32 ? 2 : 3, 6>(A, occ, s);
    case kMom3: return go<P, KF, CAP, 3, true, true, G0, F32 && CAP ? 1 : 3, F32 && G0 && KF == kKappa ? 6 : 3>(A, occ, s);
    case kMomPop2: return go<P, KF, CAP, 2, true, false, false, 3, 3>(A, occ, s);
    case kMomPop3: return go<P, KF, CAP, 3, true, false, false, F32 && CAP ? 1 : 3, 3>(A, occ, s);
    default: return hipErrorInvalidValue;
  }
}
template <int P, int KF> hipError_t march_form(int kind, const StepArgs &A, bool cap, int *occ, hipStream_t s) {
  if (cap) return pass<P, KF, true, false>(kind, A, occ, s);
  return A.g == 0.0 ? pass<P, KF, false, true>(kind, A, occ, s) : pass<P, KF, false, false>(kind, A, occ, s);
}
template hipError_t march_form<STEP_FORM, MARCH_FIELD>(int, const StepArgs &, bool, int *, hipStream_t);

}  // namespace tflbm
