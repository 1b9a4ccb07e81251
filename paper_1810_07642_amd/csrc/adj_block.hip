// Plan and launch of the reverse block kernel (adj_block.h).
#include "adj_block.h"

namespace tflbm {

template <typename T, bool W1> hipError_t launch_adj_block_form(int, const AdjBlockArgs &, hipStream_t);
extern template hipError_t launch_adj_block_form<float, false>(int, const AdjBlockArgs &, hipStream_t);
extern template hipError_t launch_adj_block_form<float, true>(int, const AdjBlockArgs &, hipStream_t);
extern template hipError_t launch_adj_block_form<double, false>(int, const AdjBlockArgs &, hipStream_t);
extern template hipError_t launch_adj_block_form<double, true>(int, const AdjBlockArgs &, hipStream_t);

// Fitted to ten lattices of 37x23 to 1024^2 sites and 1 to 6 steps: within 1 %
// of the fastest measured, on average.  [FP64, FP32][general, omega = 1]
static const TileModel kModel[2][2] = {
    {{0.31, 0.33, 0.445, 0.0263, 0.00, 0.73, 5.3, 1.35e-3, 1.35e-3}, {0.91, 0.29, 0.262, 0.0300, 0.70, 0.80, 5.2, 1.35e-3, 1.35e-3}},
    {{0.72, 1.75, 0.178, 0.0000, 0.83, 1.57, 5.0, 0.85e-3, 0.85e-3}, {0.31, 1.53, 0.156, 0.0277, 0.00, 1.26, 5.0, 0.60e-3, 0.60e-3}}};
constexpr int64_t kAdjBlockMaxSites = 1100000;  // the largest lattice it was fitted to

static const BlockShape *shapes_of(int prec, bool w1) {
  if (prec == kF64) return w1 ? AdjBlockShapes<double, true>::list : AdjBlockShapes<double, false>::list;
  return w1 ? AdjBlockShapes<float, true>::list : AdjBlockShapes<float, false>::list;
}

// False where the marching kernels are faster, or the block kernel does not
// serve the handle: disjoining exponents other than (9, 3) and (3, 9), arrays
// its 32-bit row offsets do not reach.
bool plan_adj_block(const tflbm_sim *s, BlockPlan &best) {
  best = BlockPlan();
  const tflbm_params &p = s->p;
  const bool exps = (p.n_exp == 9 && p.m_exp == 3) || (p.n_exp == 3 && p.m_exp == 9);
  if (!exps || s->kfield == kGammaKappa) return false;
  const size_t row = (size_t)s->adj_nstrips * adj_record_bytes_max(p.prec);
  if (row * p.ny >= (size_t)kDropBytes || s->kf_bytes >= (size_t)kDropBytes || tflbm_capture_bytes(s) >= (size_t)kDropBytes)
    return false;
  if ((int64_t)p.nx * p.ny > kAdjBlockMaxSites && std::getenv("TFLBM_ADJ_BLOCK") == nullptr) return false;
  const TileModel &m = kModel[p.prec == kF64 ? 0 : 1][s->w1 ? 1 : 0];
  const double t = best_plan(m, shapes_of(p.prec, s->w1), 2, p.nx, p.ny, 0, "TFLBM_ADJ_BLOCK",
                             "TFLBM_ADJ_BLOCK_SHAPE", best);
  if (best.ns == 0) return false;
  if (best.always) return true;
  return best.ns >= 2 && t < 0.9 * m.march((double)s->adj_nstrips * p.ny, m.march2);
}

hipError_t launch_adj_block(const tflbm_sim *s, const AdjArgs &B, int64_t cap_stride, int ns, hipStream_t st) {
  const int shape = s->adj_block.shape;
  const bool f64 = s->p.prec == kF64;
  const Tiles t(s->p.nx, s->p.ny, shapes_of(s->p.prec, s->w1)[shape], ns);
  if (!t.fits) return hipErrorInvalidValue;
  AdjBlockArgs A;
  A.a = B;
  A.cap_stride = cap_stride;
  A.ns = ns;
  A.halo = t.halo;
  A.bw = t.bw;
  A.bh = t.bh;
  A.ntx = t.ntx;
  A.ntiles = t.ntiles;
  A.per_xcd = t.per_xcd;
  A.n9 = s->p.n_exp == 9;
  A.inv_ntx = t.inv_ntx;
  A.inv_capB = (unsigned)(((uint64_t)1 << 32) / (unsigned)B.capB);
  if (f64) return s->w1 ? launch_adj_block_form<double, true>(shape, A, st) : launch_adj_block_form<double, false>(shape, A, st);
  return s->w1 ? launch_adj_block_form<float, true>(shape, A, st) : launch_adj_block_form<float, false>(shape, A, st);
}

}  // namespace tflbm
