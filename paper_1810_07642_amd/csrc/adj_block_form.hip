// The reverse block kernels of one working type and collision stage
// (ADJ_TYPE, STEP_W1).
#include "adj_block.h"

namespace tflbm {

template <typename T, bool W1, int I> static hipError_t go(const AdjBlockArgs &A, hipStream_t s) {
  constexpr BlockShape sh = AdjBlockShapes<T, W1>::list[I];
  adj_block_kernel<T, W1, sh.r, sh.nw><<<dim3(8 * A.per_xcd), dim3(64 * sh.nw), 0, s>>>(A, AdjCoef<T>(A.a));
  return hipGetLastError();
}
template <typename T, bool W1> hipError_t launch_adj_block_form(int shape, const AdjBlockArgs &A, hipStream_t s) {
  if (shape == 0) return go<T, W1, 0>(A, s);
  if (shape == 1) return go<T, W1, 1>(A, s);
  return hipErrorInvalidValue;
}
template hipError_t launch_adj_block_form<ADJ_TYPE, STEP_W1 != 0>(int, const AdjBlockArgs &, hipStream_t);

}  // namespace tflbm
