// Plan and launch of the reverse block kernel (adj_block.h).
#include "adj_block.h"

namespace tflbm {

template <typename T, bool W1> hipError_t launch_adj_block_form(int, const AdjBlockArgs &, hipStream_t);
extern template hipError_t launch_adj_block_form<float, false>(int, const AdjBlockArgs &, hipStream_t);
extern template hipError_t launch_adj_block_form<float, true>(int, const AdjBlockArgs &, hipStream_t);
extern template hipError_t launch_adj_block_form<double, false>(int, const AdjBlockArgs &, hipStream_t);
extern template hipError_t launch_adj_block_form<double, true>(int, const AdjBlockArgs &, hipStream_t);

// [FP64, FP32][general, omega = 1].  FP64 fitted to ten lattices of 37x23 to 1024^2
// sites and 1 to 6 steps; FP32 to 36 of 30,000 to 1.1M sites, both shapes and 2 to 4
// steps: 5 % rms general, 2 % omega = 1, the marching kernel 3 to 4 %.
static const TileModel kModel[2][2] = {
    {{0.31, 0.33, 0.445, 0.0263, 0.00, 0.73, 5.3, 1.35e-3, 1.35e-3}, {0.91, 0.29, 0.262, 0.0300, 0.70, 0.80, 5.2, 1.35e-3, 1.35e-3}},
    {{1.44, 0.00, 0.155, 0.0736, 0.148, 1.0, 5.14, 0.88e-3, 0.79e-3}, {0.00, 0.35, 0.117, 0.0841, 0.00, 0.9, 5.35, 0.64e-3, 0.56e-3}}};
constexpr int64_t kAdjBlockMaxSites = 1100000;  // the largest lattice it was fitted to
// A plan and a call are taken where the model puts their time per step below this
// fraction of the marching kernel's, beyond which its error decides.  With a call's
// own passes (four steps by a plan of three are two passes of two on tiles made for
// three) and these lines, none of 250 calls of 2 to 24 steps on 100 lattices is slower
// than the marching kernel; by the plan alone FP32 calls were, us per step marching /
// block: 675x1181 at tau = 0.9 15.9 / 20.6, 509x1530 at omega = 1 13.7 / 15.2, 606x508
// (calls of 4 and 8 steps) 8.6 / 9.6.
constexpr double kAdjLimit[2][2] = {{0.9, 0.9}, {0.85, 0.9}};

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
  best.limit = kAdjLimit[p.prec == kF64 ? 0 : 1][s->w1 ? 1 : 0] * m.march((double)s->adj_nstrips * p.ny, m.march2);
  return t < best.limit;
}

// Whether a call of nsteps reverse steps takes the plan, in k passes: not where all
// of them are single steps (launch_steps), nor where they are modelled too slow.
bool adj_block_takes(const tflbm_sim *s, int64_t nsteps, int64_t k) {
  const BlockPlan &b = s->adj_block;
  if (b.always || k >= nsteps) return b.always;
  const TileModel &m = kModel[s->p.prec == kF64 ? 0 : 1][s->w1 ? 1 : 0];
  return m.call(s->p.nx, s->p.ny, shapes_of(s->p.prec, s->w1)[b.shape], 0, nsteps, k) < b.limit * (double)nsteps;
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
