// Shapes of the block kernel (block.h), the rule that picks one and the number
// of steps per pass for a lattice, and the dispatch to the translation units
// of the storage forms and stages.
#include <cstdlib>

#include "block.h"
#include "sim.h"

namespace tflbm {

template <int P, bool W1> hipError_t launch_block_form(int, const BlockArgs &, hipStream_t);
extern template hipError_t launch_block_form<kF64, false>(int, const BlockArgs &, hipStream_t);
extern template hipError_t launch_block_form<kF64, true>(int, const BlockArgs &, hipStream_t);
extern template hipError_t launch_block_form<kF32, false>(int, const BlockArgs &, hipStream_t);
extern template hipError_t launch_block_form<kF32, true>(int, const BlockArgs &, hipStream_t);

// Time of a pass of ns steps, in microseconds, as measured over 17 lattices of
// 64^2 to 1200^2 sites, 4 to 13 shapes and 2 to 8 steps (the shape and the
// steps it picks are within 1 % (FP64) to 7 % (FP32, general stages) of the
// fastest measured on average):
//   launch + step ns + load (row_load rows + row_step active row steps),
// with the rows of one workgroup and `load` the workgroups per CU, rounded up
// to whole ones as far as `whole` says (a CU is busy until its last one ends).
// march0..2: time of one step of the marching kernels over n strip rows,
// march0 + march1 min(n, 2500) + march2 max(n - 2500, 0); moments: march2 where
// their passes hand over moments (march.h).
struct BlockModel {
  double launch, step, row_load, row_step, whole, march0, march1, march2, moments;
  int shapes;  // shapes of the form (block_shape)
};
static const BlockModel &block_model(int prec, bool w1) {
  static const BlockModel t[2][2] = {
      {{1.35, 0.00, 0.263, 0.0445, 1.0, 4.0, 1.9e-3, 0.72e-3, 0, 2},
       {1.14, 0.44, 0.107, 0.0682, 1.0, 3.8, 1.8e-3, 0.50e-3, 0.28e-3, 3}},
      {{2.99, 0.21, 0.050, 0.0693, 0.74, 5.0, 1.6e-3, 0.95e-3, 0, 2},
       {2.98, 0.25, 0.034, 0.0562, 0.58, 4.6, 1.8e-3, 0.75e-3, 0.385e-3, 3}}};
  return t[prec == kF64 ? 0 : 1][w1 ? 1 : 0];
}

// Largest lattice the model was fitted to.
constexpr int64_t kBlockMaxSites = 1500000;

// The shape and steps per pass of the least modelled time per step; false where
// the marching kernel is faster, or the block kernel does not serve the handle:
// FP16S, disjoining exponents other than (9, 3) and (3, 9), arrays its 32-bit
// row offsets do not reach.
bool plan_block(const tflbm_sim *s, BlockPlan &best) {
  best = BlockPlan();
  const tflbm_params &p = s->p;
  const bool exps = (p.n_exp == 9 && p.m_exp == 3) || (p.n_exp == 3 && p.m_exp == 9);
  if (p.prec == kF16S || !exps) return false;
  if (s->pop_bytes >= (size_t)kDropBytes || s->kf_bytes >= (size_t)kDropBytes) return false;
  int ns_min = 1, ns_max = 8, only = -1;
  bool forced = false;
  if (const char *e = std::getenv("TFLBM_BLOCK")) {
    const int v = std::atoi(e);
    if (v <= 0) return false;
    ns_min = ns_max = v;
    forced = true;
  }
  if (const char *e = std::getenv("TFLBM_BLOCK_SHAPE")) only = std::atoi(e);
  if (!forced && (int64_t)p.nx * p.ny > kBlockMaxSites) return false;
  const BlockModel &m = block_model(p.prec, s->w1);
  double best_t = 1e30;
  for (int i = 0; i < m.shapes; ++i) {
    const BlockShape sh = block_shape(p.prec, s->w1, i);
    if ((only >= 0 && i != only) || (s->kfield == kGammaKappa && !sh.pairs)) continue;
    for (int ns = ns_min; ns <= ns_max; ++ns) {
      const int bw = 64 - 6 * ns, bh = sh.r * sh.nw - 6 * ns;
      if (bw < 8 || bh < 2) break;
      const double tiles = (double)((p.nx + bw - 1) / bw) * ((p.ny + bh - 1) / bh);
      int row_steps = 0;
      for (int k = 0; k < ns; ++k)
        for (int w = 0; w < sh.nw; ++w)
          if (block_active(w * sh.r, sh.r, sh.r * sh.nw, k)) row_steps += sh.r;
      const double per_cu = tiles / 256.0, whole = (double)(int64_t)(per_cu + 0.999999);
      const double load = per_cu <= 1.0 ? 1.0 : per_cu + m.whole * (whole - per_cu);
      const double t = (m.launch + m.step * ns + load * (m.row_load * sh.r * sh.nw + m.row_step * row_steps)) / ns;
      if (t < best_t) {
        best_t = t;
        best.shape = i;
        best.ns = ns;
      }
    }
  }
  if (best.ns == 0) return false;
  const double n = (double)s->nstrips * p.ny;
  const double march = m.march0 + m.march1 * (n < 2500 ? n : 2500) +
                       (s->march_ns > 0 ? m.moments : m.march2) * (n < 2500 ? 0 : n - 2500);
  return forced || best_t < 0.9 * march;  // (a tie stays with the marching kernel: FP64 1024^2)
}

// Launch shape of a pass of ns steps of a plan.
void shape_block(const tflbm_sim *s, int shape, int ns, BlockArgs &A) {
  const BlockShape sh = block_shape(s->p.prec, s->w1, shape);
  A.ns = ns;
  A.halo = 3 * ns;
  A.bw = 64 - 2 * A.halo;
  A.bh = sh.r * sh.nw - 2 * A.halo;
  A.ntx = (s->p.nx + A.bw - 1) / A.bw;
  A.inv_ntx = A.ntx == 1 ? 0xffffffffu : (unsigned)(((uint64_t)1 << 32) / (unsigned)A.ntx);
  A.ntiles = A.ntx * ((s->p.ny + A.bh - 1) / A.bh);
  A.per_xcd = (A.ntiles + 7) / 8;
  A.kf = s->kfield;
  A.ksign = s->p.n_exp == 9 ? 1.0f : -1.0f;
}

hipError_t launch_block(int prec, bool w1, int shape, const BlockArgs &A, hipStream_t s) {
  switch (prec) {
    case kF64: return w1 ? launch_block_form<kF64, true>(shape, A, s) : launch_block_form<kF64, false>(shape, A, s);
    case kF32: return w1 ? launch_block_form<kF32, true>(shape, A, s) : launch_block_form<kF32, false>(shape, A, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace tflbm
