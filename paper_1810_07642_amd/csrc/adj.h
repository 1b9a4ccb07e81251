// Reverse mode of the thin-film lattice Boltzmann step: the hand-written
// vector-Jacobian product of one step of eq. "LBE" (arXiv:1810.07642, Sec. II)
// with respect to the pre-collision populations and the kappa field.
//
// Notation.  Forward step t, at every site x (pre-collision state f):
//   h = sum_l f_l, j = sum_l c_l f_l, u = j/h
//   p = -gamma (L h + kappa phi(h)),  phi(h) = (h_*/h)^n - (h_*/h)^m
//   G = grad_s p (isotropic gradient),  F = -h G - nu alpha(h) u + h a
//   f*_l = f_l + omega (feq_l(h, u) - f_l) + 3 w_l c_l . F,   f_l(x + c_l, t + 1) = f*_l(x).
// Adjoint.  lambda^t_l(x) = dLoss/df^t_l(x).  A reverse step at site x reads
// mu_l(x) = lambda^{t+1}_l(x + c_l) = dLoss/df*_l(x) and computes, at every
// site:
//   Lambda_F = 3 sum_l w_l c_l mu_l                       (from the source term)
//   lambda_G = -h Lambda_F                                (from F = -h G)
//   lambda_p = -div_s lambda_G                            (grad_s^T = -div_s)
//   lambda_u = omega sum_l mu_l dfeq_l/du - nu alpha Lambda_F
//   lambda_h = omega sum_l mu_l dfeq_l/dh + Lambda_F.(-G - nu alpha'(h) u + a)
//              - gamma L(lambda_p) - gamma kappa phi'(h) lambda_p - lambda_u.u/h    (L^T = L)
//   lambda_j = lambda_u / h
//   lambda^t_l = (1 - omega) mu_l + lambda_h + c_l . lambda_j
//   g_kappa += -gamma phi(h) lambda_p          (FP64 accumulation)
// and stores lambda^t_l(x) for step t-1 (layout: AdjRec).
// The forward moments h, j of step t come from the capture written by the
// forward step; the film pressure and its gradient are recomputed from h.
#pragma once

#include <algorithm>
#include <cstring>

#include "device.h"
#include "launch.h"
#include "sim.h"

namespace tflbm {

// Adjoint state layout ("push in y, pull in x", as the forward records).
// Records of kAdjW consecutive columns of one row, [ny][nstrips][RB]: the
// nine segments of kAdjW values ordered by c_ly (kSlot), the record padded to
// an odd number of 128-byte lines.  Entry l at (column X, row Y) holds
// nu_l(X, Y) = lambda_l(X, Y + c_ly): a site stores its adjoint populations
// at its own column, in the rows they are read from, so each strip writes
// whole records of its own; the lane of column x takes
// mu_l(x, y) = lambda_l(x + c_l) = nu_l(x + c_lx, y) from column x + c_lx
// of row y.  dLoss/dkappa is FP64 in records of 64 values [ny][nstrips][64]:
// the kAdjW columns and ten padding values, which the strip's halo lanes
// write, so that the record is four whole lines.
constexpr int kAdjW = 54;     // columns per strip and record
constexpr int kAdjHalo = 5;   // halo columns per side: two per reverse step and the shift between two steps
constexpr int kGkRB = 64 * 8;  // bytes of a dLoss/dkappa record
constexpr int kDropOffset = kDropBytes;  // a buffer offset past every row: the access is dropped
static_assert(kAdjW + 2 * kAdjHalo == 64, "a strip and its halo fill one wavefront");
template <typename T> struct AdjRec {
  static constexpr int SEG = kAdjW * (int)sizeof(T);
  static constexpr int LINES = (9 * SEG + 127) / 128;
  static constexpr int RB = (LINES % 2 ? LINES : LINES + 1) * 128;
  __host__ __device__ static constexpr int seg(int l) { return kSlot[l] * SEG; }
};

// With omega = 1 the step's adjoint is lambda^t_l = lambda_h + c_l . lambda_j
// (lam_of): three fields per site carry it between steps instead of nine
// populations.  They are stored at the site itself in records of 64 slots per
// field, [ny][nstrips][3][64] (lambda_h, lambda_jx, lambda_jy): the strip's
// kAdjW columns in slots 0 .. kAdjW-1 and ten padding slots that the halo
// lanes write, so a strip writes whole lines; the reverse step at (x, y)
// forms mu_l(x, y) = lambda_l(x + c_l) from the fields at column x + c_lx of
// row y + c_ly.
template <typename T> struct AdjRec1 {
  static constexpr int SEG = 64 * (int)sizeof(T);
  static constexpr int RB = 3 * SEG;
};

struct AdjArgs {
  const char *src;     // adjoint records at the end of step t (AdjRec; AdjRec1 with omega = 1)
  char *dst;           // adjoint records at the end of step t-1
  const char *cap;     // h, jx, jy of step t: capture records of the forward form
  const char *cap2;    // the same for step t-1 (two-step pass only)
  const void *kfield;  // kappa [ny][ldx] in T or nullptr
  char *gk;            // dLoss/dkappa records [ny][nstrips][64] FP64
  int nx, ny, ldx;
  int cnblk;           // capture records per row (those of the forward step)
  int capB, capRB;     // sites and bytes per capture record (the forward form's)
  int nstrips, H, ntiles, per_xcd;
  int n_exp, m_exp;
  double omega, gamma, nu, hstar, delta, ax, ay, g, kappa0;
};

// ns reverse steps in one launch of the reverse block kernel: the latest step's
// capture is B.cap, an earlier step's cap_stride bytes before the next one's.
hipError_t launch_adj_block(const tflbm_sim *s, const AdjArgs &B, int64_t cap_stride, int ns, hipStream_t st);

// Lambda_F = 3 sum_l w_l c_l mu_l through differences of opposite populations.
template <typename T>
__device__ __forceinline__ void lambda_force(const T (&mu)[9], T cA, T cD, T &LFx, T &LFy) {
  const T d15 = mu[1] - mu[5], d37 = mu[3] - mu[7], d26 = mu[2] - mu[6], d48 = mu[4] - mu[8];
  LFx = madd(cA, d15, cD * (d26 - d48));
  LFy = madd(cA, d37, cD * (d26 + d48));
}

// r^n and r^m; (9, 3) and (3, 9) without loops.
template <typename T> __device__ __forceinline__ void powers(T r, int n, int m, T &rn, T &rm) {
  if ((n == 9 && m == 3) || (n == 3 && m == 9)) {
    const T r3 = r * r * r;
    const T r9 = r3 * r3 * r3;
    rn = n == 9 ? r9 : r3;
    rm = n == 9 ? r3 : r9;
  } else {
    rn = ipow(r, n);
    rm = ipow(r, m);
  }
}

// Scalar coefficients of the reverse step in the working type.
template <typename T> struct AdjCoef {
  T omega, om1, gamma, nu, hstar, delta, three_d2, ax, ay, g, kap0, cA, cD;
  int n_exp, m_exp;
  __host__ __device__ explicit AdjCoef(const AdjArgs &A)
      : omega((T)A.omega), om1(T(1) - (T)A.omega), gamma((T)A.gamma), nu((T)A.nu), hstar((T)A.hstar),
        delta((T)A.delta), three_d2(T(3) * (T)A.delta * (T)A.delta), ax((T)A.ax), ay((T)A.ay), g((T)A.g),
        kap0((T)A.kappa0), cA((T)(3.0 * kW[1])), cD((T)(3.0 * kW[2])), n_exp(A.n_exp), m_exp(A.m_exp) {}
};

// lambda_l = lambda_h + c_l . lambda_j: the part of the step's adjoint that
// does not depend on mu (the whole of it when omega = 1).
template <typename T> __device__ __forceinline__ T lam_of(int l, T lh, T ljx, T ljy) {
  const int cx = kCx[l], cy = kCy[l];
  const T cl = cx == 0 ? (cy == 0 ? T(0) : (cy > 0 ? ljy : -ljy))
                       : (cy == 0 ? (cx > 0 ? ljx : -ljx)
                                  : (cx > 0 ? (cy > 0 ? ljx + ljy : ljx - ljy) : (cy > 0 ? ljy - ljx : -ljx - ljy)));
  return lh + cl;
}

// lambda_h and lambda_j of a site at the start of the step, and its term
// -gamma phi(h) lambda_p of dLoss/dkappa: from mu, the forward h, 1/h, (h_*/h)^n,
// (h_*/h)^m, j and kappa, Lambda_F, the forward pressure gradient G, lambda_p
// (lp) and its Laplacian.
template <typename T>
__device__ __forceinline__ void adj_site(const AdjCoef<T> &C, const T (&mu)[9], T h, T inv_h, T rn, T rm, T jx, T jy, T kap,
                                         T Fx, T Fy, T Gx, T Gy, T lapq, T lp, T &lh_out, T &ljx_out, T &ljy_out,
                                         double &gterm) {
  const T ux = jx * inv_h, uy = jy * inv_h;
  const T invD = recip(madd(T(2) * h, h, madd(T(6) * C.delta, h, C.three_d2)));
  const T alpha = T(6) * h * invD;
  const T dalpha = T(6) * madd(T(-2) * h, h, C.three_d2) * (invD * invD);
  const T phi = rn - rm;
  const T dphi = (T(C.m_exp) * rm - T(C.n_exp) * rn) * inv_h;

  // omega sum_l mu_l dfeq_l/dh and omega sum_l mu_l dfeq_l/du over pairs
  // of opposite populations: S = mu_l + mu_-l takes the parts of the
  // derivatives even in c, D = mu_l - mu_-l the odd ones
  const T usq = madd(ux, ux, uy * uy);
  const T gh = C.g * h;
  const T up = ux + uy, um = uy - ux;
  const T S15 = mu[1] + mu[5], D15 = mu[1] - mu[5];
  const T S37 = mu[3] + mu[7], D37 = mu[3] - mu[7];
  const T S26 = mu[2] + mu[6], D26 = mu[2] - mu[6];
  const T S48 = mu[4] + mu[8], D48 = mu[4] - mu[8];
  // d/dh: rest 1 - 5gh/3 - 2u^2/3; axes gh/3 + cu/3 + cu^2/2 - u^2/6;
  // diagonals gh/12 + cu/12 + cu^2/8 - u^2/24
  T sh = mu[0] * madd(gh, T(-5.0 / 3.0), madd(usq, T(-2.0 / 3.0), T(1)));
  sh = madd(S15 + S37, madd(gh, T(1.0 / 3.0), usq * T(-1.0 / 6.0)), sh);
  sh = madd(T(0.5), madd(S15, ux * ux, S37 * (uy * uy)), sh);
  sh = madd(T(1.0 / 3.0), madd(D15, ux, D37 * uy), sh);
  sh = madd(S26 + S48, madd(gh, T(1.0 / 12.0), usq * T(-1.0 / 24.0)), sh);
  sh = madd(T(0.125), madd(S26, up * up, S48 * (um * um)), sh);
  sh = madd(T(1.0 / 12.0), madd(D26, up, D48 * um), sh);
  // d/du = h (c1 c + c2 (c.u) c - c3 u): rest -4u/3; axes (1/3, 1, 1/3);
  // diagonals (1/12, 1/4, 1/12)
  T sx = mu[0] * ux * T(-4.0 / 3.0);
  sx = madd(D15, T(1.0 / 3.0), sx);
  sx = madd(S15 - T(0.5) * S37, ux * T(2.0 / 3.0), sx);
  sx = madd(D26 - D48, T(1.0 / 12.0), sx);
  sx = madd(S26, madd(up, T(0.25), ux * T(-1.0 / 12.0)), sx);
  sx = madd(S48, madd(um, T(-0.25), ux * T(-1.0 / 12.0)), sx);
  T sy = mu[0] * uy * T(-4.0 / 3.0);
  sy = madd(D37, T(1.0 / 3.0), sy);
  sy = madd(S37 - T(0.5) * S15, uy * T(2.0 / 3.0), sy);
  sy = madd(D26 + D48, T(1.0 / 12.0), sy);
  sy = madd(S26, madd(up, T(0.25), uy * T(-1.0 / 12.0)), sy);
  sy = madd(S48, madd(um, T(0.25), uy * T(-1.0 / 12.0)), sy);
  const T fric = C.nu * alpha;
  const T lux = madd(C.omega * h, sx, -fric * Fx);
  const T luy = madd(C.omega * h, sy, -fric * Fy);
  T lh = C.omega * sh + Fx * (-Gx - C.nu * dalpha * ux + C.ax) + Fy * (-Gy - C.nu * dalpha * uy + C.ay) -
         C.gamma * lapq - C.gamma * kap * dphi * lp;
  lh -= (lux * ux + luy * uy) * inv_h;
  lh_out = lh;
  ljx_out = lux * inv_h;
  ljy_out = luy * inv_h;
  gterm = -(double)C.gamma * (double)phi * (double)lp;
}

}  // namespace tflbm
