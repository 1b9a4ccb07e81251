// The rule that picks a shape of the block kernel (block.h) and the number of
// steps per pass for a lattice, and the dispatch to the translation units of
// the storage forms and stages.
#include <cstdlib>

#include "block.h"
#include "sim.h"

namespace tflbm {

template <int P, bool W1> hipError_t launch_block_form(int, const BlockArgs &, hipStream_t);
extern template hipError_t launch_block_form<kF64, false>(int, const BlockArgs &, hipStream_t);
extern template hipError_t launch_block_form<kF64, true>(int, const BlockArgs &, hipStream_t);
extern template hipError_t launch_block_form<kF32, false>(int, const BlockArgs &, hipStream_t);
extern template hipError_t launch_block_form<kF32, true>(int, const BlockArgs &, hipStream_t);
extern template hipError_t launch_block_form<kF16S, false>(int, const BlockArgs &, hipStream_t);
extern template hipError_t launch_block_form<kF16S, true>(int, const BlockArgs &, hipStream_t);

double best_plan(const TileModel &m, const BlockShape *shapes, int n, int nx, int ny, int extra,
                 const char *env, const char *env_shape, BlockPlan &best) {
  best = BlockPlan();
  // A pass of one step is no plan: there are as many launches as of the marching
  // kernel's, and passes whose number cannot be made even or odd with that of its
  // fused ones.  Nor may it stand in the way of two or more steps, which the model
  // puts a few percent behind it at some sizes though they are faster (us per step,
  // marching / one / two or more: FP16S at tau = 0.9 323x925 18.1 / 7.2 / 6.6,
  // 1285x843 32.6 / 18.9 / 15.2) or, where one step is not taken, of the marching
  // kernel (FP64 at tau = 0.9 450^2 9.4 / 8.6, 500^2 10.5 / 9.2; FP16S 212x1089 9.2 /
  // 5.4; reverse, FP64 138x638 8.7 / 6.9).
  int ns_min = 2, ns_max = 9, only = -1;
  if (const char *e = std::getenv(env)) {
    const int v = std::atoi(e);
    if (v <= 0) return 0.0;
    ns_min = ns_max = v;
    best.always = true;
  }
  if (const char *e = std::getenv(env_shape)) only = std::atoi(e);
  double best_t = 1e30;
  for (int i = 0; i < n; ++i) {
    if (only >= 0 && i != only) continue;
    for (int ns = ns_min; ns <= ns_max; ++ns) {
      const Tiles t(nx, ny, shapes[i], ns, extra);
      if (!t.fits) break;
      const double dt = m.pass(t, shapes[i], ns) / ns;
      if (dt < best_t) {
        best_t = dt;
        best.shape = i;
        best.ns = ns;
      }
    }
  }
  return best_t;
}

// Fitted to 17 lattices of 64^2 to 1200^2 sites, 4 to 13 shapes and 2 to 8
// steps: what it picks is within 1 % (FP64) to 6 % (FP16S) of the fastest
// measured, on average.  [FP64, FP32, FP16S][general, omega = 1]
static const TileModel kModel[3][2] = {
    {{1.35, 0.00, 0.263, 0.0445, 0, 1.0, 4.0, 1.9e-3, 0.72e-3}, {1.14, 0.44, 0.107, 0.0682, 0, 1.0, 3.8, 1.8e-3, 0.50e-3}},
    {{1.22, 1.01, 0.158, 0.0048, 0, 0.71, 5.0, 1.6e-3, 0.95e-3}, {2.98, 0.25, 0.034, 0.0562, 0, 0.58, 4.6, 1.8e-3, 0.75e-3}},
    {{1.01, 0.88, 0.099, 0.0564, 0, 0.80, 5.2, 1.6e-3, 0.75e-3}, {0.61, 0.86, 0.074, 0.0599, 0, 0.83, 5.1, 1.5e-3, 0.75e-3}}};
// The marching FP16S kernels on lattices of odd width: their edge strips load
// misaligned column pairs half by half (us per step, 1500 / 1501 columns 21.3 /
// 49.7, 2000 / 2001 32.9 / 73.9), which the block kernel's lanes of one column
// never do (2001^2 46).
constexpr double kOddF16 = 2.3;
// march2 where the marching passes hand over moments (march.h): FP64, FP32.
constexpr double kMarchMoments[3] = {0.28e-3, 0.385e-3, 0};
// Largest lattice the model was fitted to.
constexpr int64_t kBlockMaxSites = 1500000;
// A call is taken where the model puts its own passes below this fraction of the
// marching kernels' time: [FP64, FP32, FP16S][stages][two steps or less; more, which the
// marching kernels step on populations; less than ten by their passes of moments; ten
// and more by those].  What the model leaves out sets the lines, and only where the
// tiles take more than one round of the GPU (FP32 general captures: more than two), or at
// omega = 1 two steps write captures (1 otherwise).  At omega = 1 a call's first and last
// pass move populations (us per step, marching / block: FP32 1165x1007 2 steps 16.6 /
// 22.1, 4 steps 15.9 / 18.6, 24 steps 13.6 / 13.3; FP64 723x817 2 steps 15.1 / 18.1, 24
// steps 10.6 / 10.2), but the marching kernels have slow passes for short odd calls
// (FP64 658x740 3 steps with captures 18.6 / 15.2, FP32 1111x876 9 steps 16.2 / 12.7).
// Captures go out in parts of lines from tiles of 52 columns and less (FP32 general
// 1232x911 without 17.9 / 16.4, with 19.1 / 25.2; 1157x327 with 12.1 / 9.2).  The lines
// are drawn from 5000 calls of 2 to 32 steps on 250 lattices where the model sees between
// 0.55 and the whole of the marching time.
enum CallKind { kGeneral = 0, kGeneralCap = 1, kOmega1 = 2, kOmega1Cap = 3 };
constexpr double kLimit[3][4][4] = {
    {{1.00, 1.00, 1.00, 1.00}, {0.90, 0.90, 0.90, 0.90}, {0.76, 1.20, 0.82, 0.89}, {0.68, 1.20, 0.90, 0.97}},
    {{0.95, 0.95, 0.95, 0.95}, {0.69, 0.69, 0.69, 0.69}, {0.70, 0.95, 0.86, 0.84}, {0.56, 0.90, 0.85, 0.86}},
    {{1.00, 1.00, 1.00, 1.00}, {0.90, 0.90, 0.90, 0.90}, {0.84, 0.89, 0.89, 0.89}, {0.68, 0.88, 0.88, 0.88}}};
// Two or three steps that the number of passes makes single ones, in one round of
// tiles: [form][general, omega = 1].  (FP32 at tau = 0.9 161x1164, two steps: 11.4 / 7.0;
// measured from 0.58 to 1.02 of the marching kernel below these lines.)
constexpr double kSingleLimit[3][2] = {{0.95, 0.70}, {0.97, 0.70}, {0.88, 0.70}};
// And a plan is made where some calls take it.
constexpr double kPlanLimit[3][2] = {{0.90, 0.97}, {0.90, 0.95}, {0.90, 0.89}};  // [form][general, omega = 1]

static const BlockShape *shapes_of(int prec, bool w1, int &n) {
  auto of = [&](const auto &list) {
    n = (int)(sizeof(list) / sizeof(BlockShape));
    return (const BlockShape *)list;
  };
  if (prec == kF64) return w1 ? of(BlockShapes<kF64, true>::list) : of(BlockShapes<kF64, false>::list);
  if (prec == kF16S) return w1 ? of(BlockShapes<kF16S, true>::list) : of(BlockShapes<kF16S, false>::list);
  return w1 ? of(BlockShapes<kF32, true>::list) : of(BlockShapes<kF32, false>::list);
}

// FP16S loses a column per side more: it decodes its populations where they are
// stored and shifts them into place.
static int extra_columns(int prec) { return prec == kF16S ? 1 : 0; }

static int form_of(int prec) { return prec == kF64 ? 0 : (prec == kF32 ? 1 : 2); }

// False where the marching kernels are faster, or the block kernel does not
// serve the handle: disjoining exponents other than (9, 3) and (3, 9), arrays its
// 32-bit row offsets do not reach.
bool plan_block(const tflbm_sim *s, BlockPlan &best) {
  best = BlockPlan();
  const tflbm_params &p = s->p;
  const bool exps = (p.n_exp == 9 && p.m_exp == 3) || (p.n_exp == 3 && p.m_exp == 9);
  if (!exps) return false;
  if (s->pop_bytes >= (size_t)kDropBytes || s->kf_bytes >= (size_t)kDropBytes ||
      tflbm_capture_bytes(s) >= (size_t)kDropBytes)
    return false;
  const int f = form_of(p.prec);
  const TileModel &m = kModel[f][s->w1 ? 1 : 0];
  const bool odd = p.prec == kF16S && (p.nx & 1) != 0;
  if (!odd && (int64_t)p.nx * p.ny > kBlockMaxSites && std::getenv("TFLBM_BLOCK") == nullptr) return false;
  int n = 0;
  const BlockShape *shapes = shapes_of(p.prec, s->w1, n);
  const double t = best_plan(m, shapes, n, p.nx, p.ny, extra_columns(p.prec), "TFLBM_BLOCK", "TFLBM_BLOCK_SHAPE", best);
  if (best.ns == 0) return false;
  if (best.always) {
    best.limit = 1e30;
    return true;
  }
  // a surface tension field, whose second value per site the model leaves out, stays
  // with the marching kernels where that is near (taken from one FP32 lattice, general
  // stages, 808x1306: 25 us per step against 16; the other forms keep the same line)
  const bool gamma = s->kfield == kGammaKappa;
  best.limit = m.march((double)s->nstrips * p.ny, s->march_ns > 0 ? kMarchMoments[f] : m.march2) *
               (odd ? kOddF16 : 1.0) * (gamma ? 0.75 / 0.9 : 1.0);
  best.always = odd;
  return t < kPlanLimit[f][s->w1 && !gamma ? 1 : 0] * best.limit;
}

// Whether a call of nsteps steps takes the plan, in k passes (moments: the marching
// kernels would hand over moments): not where it is modelled too slow, nor (odd widths of
// FP16S excepted) a call of one step, which the marching kernel does for less than a
// tile's load and store (FP64 64^2 4.5 us against 6.3 in a pass of one).
bool block_takes(const tflbm_sim *s, int64_t nsteps, int64_t k, bool capture, bool moments) {
  const BlockPlan &b = s->block;
  if (b.ns == 0 || nsteps == 0 || (nsteps == 1 && !b.always)) return false;
  const tflbm_params &p = s->p;
  const int f = form_of(p.prec), extra = extra_columns(p.prec);
  int n = 0;
  const BlockShape &sh = shapes_of(p.prec, s->w1, n)[b.shape];
  // (a surface tension field's calls hand over no moments by the marching kernels)
  const int kind = capture ? (s->w1 ? kOmega1Cap : kGeneralCap) : (s->w1 && s->kfield != kGammaKappa ? kOmega1 : kGeneral);
  const int length = nsteps <= 2 ? 0 : (!moments ? 1 : (nsteps < 10 ? 2 : 3));
  const int rounds = (Tiles(p.nx, p.ny, sh, (int)((nsteps + k - 1) / k), extra).ntiles + 255) / 256;
  double limit = kLimit[f][kind][length];
  if (moments && (nsteps & 1)) limit += 0.05;  // one of their passes has three steps
  if ((nsteps & 1) == 0 && limit > 1.0) limit = 1.0;
  if (k >= nsteps && !b.always) limit = rounds <= 1 ? kSingleLimit[f][s->w1 ? 1 : 0] : 0.0;
  else if (rounds <= 1 && !(kind == kOmega1Cap && length == 0)) limit = 1.0;
  else if (rounds == 2 && kind == kGeneralCap && p.prec == kF32) limit = kLimit[f][kGeneral][length];
  return kModel[f][s->w1 ? 1 : 0].call(p.nx, p.ny, sh, extra, nsteps, k) < limit * b.limit * (double)nsteps;
}

// Launch shape of a pass of ns steps of a plan.
void shape_block(const tflbm_sim *s, int shape, int ns, BlockArgs &A) {
  int n = 0;
  const Tiles t(s->p.nx, s->p.ny, shapes_of(s->p.prec, s->w1, n)[shape], ns, extra_columns(s->p.prec));
  A.ns = ns;
  A.halo = t.halo;
  A.halo_x = t.halo_x;
  A.bw = t.bw;
  A.bh = t.bh;
  A.ntx = t.ntx;
  A.inv_ntx = t.inv_ntx;
  A.ntiles = t.ntiles;
  A.per_xcd = t.per_xcd;
  A.kf = s->kfield;
  A.ksign = s->p.n_exp == 9 ? 1.0f : -1.0f;
}

hipError_t launch_block(int prec, bool w1, int shape, const BlockArgs &A, hipStream_t s) {
  switch (prec) {
    case kF64: return w1 ? launch_block_form<kF64, true>(shape, A, s) : launch_block_form<kF64, false>(shape, A, s);
    case kF32: return w1 ? launch_block_form<kF32, true>(shape, A, s) : launch_block_form<kF32, false>(shape, A, s);
    default: return w1 ? launch_block_form<kF16S, true>(shape, A, s) : launch_block_form<kF16S, false>(shape, A, s);
  }
}

}  // namespace tflbm
