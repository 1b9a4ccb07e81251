// The block kernels of one storage form and collision stage (STEP_FORM and
// STEP_W1 as in step_form.hip).
#include "block.h"

namespace tflbm {

template <int P, bool W1, int R, int NW>
static hipError_t launch_shape(const BlockArgs &A, hipStream_t s) {
  const dim3 grid(8 * A.per_xcd), block(64 * NW);
  const bool g0 = A.s.g == 0.0;
  const Coef<typename Form<P>::T> C(A.s);
  if (A.kf == kGammaKappa) {
    if (A.s.capture) block_kernel<P, W1, true, false, true, R, NW><<<grid, block, 0, s>>>(A, C);
    else if (g0) block_kernel<P, W1, true, true, false, R, NW><<<grid, block, 0, s>>>(A, C);
    else block_kernel<P, W1, true, false, false, R, NW><<<grid, block, 0, s>>>(A, C);
  } else if (A.s.capture) {
    if (g0) block_kernel<P, W1, false, true, true, R, NW><<<grid, block, 0, s>>>(A, C);
    else block_kernel<P, W1, false, false, true, R, NW><<<grid, block, 0, s>>>(A, C);
  } else {
    if (g0) block_kernel<P, W1, false, true, false, R, NW><<<grid, block, 0, s>>>(A, C);
    else block_kernel<P, W1, false, false, false, R, NW><<<grid, block, 0, s>>>(A, C);
  }
  return hipGetLastError();
}

template <int P, bool W1> hipError_t launch_block_form(int shape, const BlockArgs &A, hipStream_t s) {
  constexpr auto shapes = BlockShapes<P, W1>::list;
  constexpr int n = sizeof(BlockShapes<P, W1>::list) / sizeof(BlockShape);
  if (shape == 0) return launch_shape<P, W1, shapes[0].r, shapes[0].nw>(A, s);
  if (shape == 1) return launch_shape<P, W1, shapes[1].r, shapes[1].nw>(A, s);
  if constexpr (n > 2) {
    if (shape == 2) return launch_shape<P, W1, shapes[2].r, shapes[2].nw>(A, s);
  }
  return hipErrorInvalidValue;
}
template hipError_t launch_block_form<STEP_FORM, STEP_W1 != 0>(int, const BlockArgs &, hipStream_t);

}  // namespace tflbm
