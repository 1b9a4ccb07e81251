// Passes that hand over moments (march.h): which calls take them, how a call's
// steps are split into passes, and their launch shapes.
#include <cstdlib>

#include "march.h"
#include "sim.h"

namespace tflbm {

template <int P, int KF> hipError_t march_form(int, const StepArgs &, bool, int *, hipStream_t);
extern template hipError_t march_form<kF64, kNoField>(int, const StepArgs &, bool, int *, hipStream_t);
extern template hipError_t march_form<kF64, kKappa>(int, const StepArgs &, bool, int *, hipStream_t);
extern template hipError_t march_form<kF32, kNoField>(int, const StepArgs &, bool, int *, hipStream_t);
extern template hipError_t march_form<kF32, kKappa>(int, const StepArgs &, bool, int *, hipStream_t);

hipError_t launch_march(int prec, int kind, const StepArgs &A, int kf, bool cap, int *occ, hipStream_t s) {
  if (prec == kF64 && kf == kNoField) return march_form<kF64, kNoField>(kind, A, cap, occ, s);
  if (prec == kF64 && kf == kKappa) return march_form<kF64, kKappa>(kind, A, cap, occ, s);
  if (prec == kF32 && kf == kNoField) return march_form<kF32, kNoField>(kind, A, cap, occ, s);
  if (prec == kF32 && kf == kKappa) return march_form<kF32, kKappa>(kind, A, cap, occ, s);
  return hipErrorInvalidValue;
}

static int strip_columns(int prec, int kind) {
  if (kind == kMom2) return prec == kF64 ? march_columns<kF64, 2, true, true>() : march_columns<kF32, 2, true, true>();
  return record_sites(prec);
}

// Three steps per pass from this many sites on, two below: two lose 12 and 16
// columns of a strip's 64 and 128 to their halo and 12 rows of a chunk, three 18
// and 20 columns and 18 rows, for a third fewer bytes.  Measured, us per step,
// two / three: FP32 1536^2 18.5 / 19.4, 2048^2 23.1 / 24.2, 4096^2 74.9 / 68.5;
// FP64 1536^2 26.4 / 26.9, 2048^2 35.7 / 39.4, 4096^2 149.4 / 132.5.
constexpr int64_t kMarch3MinSites = 8000000;
// No such passes on lattices of fewer strip rows: there a tile's time is its chain
// of rows, which passes of two steps make longer than step_kernel's plan of one step
// per pass (api.hip).  (These lattices come here where the block kernel does not
// serve the exponents.)  Measured, us per step of calls of 10 steps, step_kernel /
// moments, exponents (10, 4): FP32 64^2 6.2 / 9.9, 256^2 7.1 / 10.5, 512^2 (2560 strip
// rows) 10.4 / 11.9; FP64 64^2 4.8 / 7.2, 256^2 7.2 / 9.5, 384^2 (3456) 9.2 / 9.4.  From
// 3000 to 5000 strip rows they are 10 % faster to 10 % slower, by the rows of a chunk
// and with captures; in 60 lattices of 5500 to 7000 none is slower (10 steps 2 to 13 %
// faster, 64 steps 4 to 22 %).
constexpr int64_t kMarchMinStripRows = 5400;

void plan_march(tflbm_sim *s) {
  s->march_ns = 0;
  if (!s->w1 || s->p.prec == kF16S || s->kfield == kGammaKappa || s->fuse != 0) return;
  if ((int64_t)s->nstrips * s->p.ny >= kMarchMinStripRows)
    s->march_ns = (int64_t)s->p.nx * s->p.ny >= kMarch3MinSites ? 3 : 2;
  if (const char *e = std::getenv("TFLBM_MARCH")) s->march_ns = std::atoi(e) <= 0 ? 0 : (std::atoi(e) >= 3 ? 3 : 2);
}

// Launch shapes of the passes.
void shape_march(tflbm_sim *s, int cus) {
  if (s->march_ns == 0) return;
  const StepArgs A = make_step_args(s);
  for (int kind = 0; kind < kMarchKinds; ++kind) {
    MarchShape &m = s->march_shape[kind];
    int occ = 0;
    if (launch_march(s->p.prec, kind, A, s->kfield, false, &occ, nullptr) != hipSuccess || occ <= 0) occ = 8;
    m.nstrips = (s->p.nx + strip_columns(s->p.prec, kind) - 1) / strip_columns(s->p.prec, kind);
    m.rows = choose_rows(s->p.ny, m.nstrips, occ * cus, 1, "TFLBM_MARCH_ROWS");
    m.ntiles = m.nstrips * ((s->p.ny + m.rows - 1) / m.rows);
    m.per_xcd = (m.ntiles + 7) / 8;
  }
}

bool split_march(int64_t nsteps, int64_t passes_before, int ns, MarchSplit &sp) {
  // the first pass takes two steps, the others two or three: as few passes as
  // hold the steps (three per pass), or as many (two)
  const int64_t rest = nsteps - 2;
  if (rest < 2) return false;
  int64_t m = ns == 3 ? (rest + 2) / 3 : rest / 2;
  if ((m + 1 - passes_before) & 1) m += ns == 3 ? 1 : -1;
  if (m < 1 || 2 * m > rest || 3 * m < rest) return false;
  sp.passes = m + 1;
  sp.threes = rest - 2 * m;
  return true;
}

}  // namespace tflbm
