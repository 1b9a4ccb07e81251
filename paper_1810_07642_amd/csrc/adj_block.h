// The reverse block kernel: several reverse steps of one tile of the lattice
// per launch, with the tile's adjoint in registers (internal to the library;
// instantiated per working type and collision stage in adj_block_form.hip).
//
// Tiles, halo and exchange are those of the forward block kernel (block.h): a
// workgroup of NW wavefronts holds 64 columns and NW R rows, a reverse step
// reads three sites in each direction (one for mu, one for lambda_p's
// divergence, one for its Laplacian), and the neighbours in y at the edge of a
// wavefront's rows come through LDS in three exchanges: lambda, then the x
// combinations of lambda_G and of the film pressure, then lambda_p.  The
// forward moments of a step are read while the step before it runs, and dLoss/
// dkappa of the tile's own sites is read and written once per pass, receiving
// the steps' terms in the order of single steps.  Measured (us per reverse step,
// marching / block): FP32 at omega = 1 128^2 5.3 / 3.1, 256^2 6.4 / 3.3, 512^2 8.2 /
// 5.7; general 256^2 6.3 / 3.5, 512^2 9.7 / 8.2; FP64 128^2 5.5 / 3.9, 256^2 7.9 /
// 5.7.  Bound by VALU issue: some 210 instructions per row, wavefront and step,
// on tiles of which the halo leaves a quarter to a half.
#pragma once

#include "adj.h"

namespace tflbm {

// Shapes per working type and stage (BlockShapes of block.h; FP64 holds its
// tile's adjoint, mu and the forward moments of two rows per wavefront at most).
template <typename T, bool W1> struct AdjBlockShapes {
  static constexpr BlockShape list[] = {{1, 12}, {2, 8}};
};
template <> struct AdjBlockShapes<float, true> {
  static constexpr BlockShape list[] = {{2, 16}, {3, 12}};
};
template <> struct AdjBlockShapes<float, false> {
  static constexpr BlockShape list[] = {{1, 16}, {2, 16}};
};

struct AdjBlockArgs {
  AdjArgs a;              // a.cap: the capture of the pass's first (latest) step
  int64_t cap_stride;     // bytes from a step's capture to the next (later) step's
  int ns, halo, bw, bh;   // reverse steps, columns and rows lost per side, output columns and rows of a tile
  int ntx, ntiles, per_xcd;
  bool n9;                // the exponents are (9, 3), else (3, 9)
  unsigned inv_ntx, inv_capB;  // 2^32 / ntx and 2^32 / capB rounded down
};

template <typename T, bool W1, int R, int NW>
__global__ __launch_bounds__(64 * NW) void adj_block_kernel(AdjBlockArgs A, AdjCoef<T> C) {
  constexpr int ES = sizeof(T);
  // of a wavefront's first row lambda_2, lambda_3, lambda_4 and of its last
  // lambda_6, lambda_7, lambda_8 (what the rows above and below read); ga, gb,
  // pa, pb of both; lambda_p and the sum of its x neighbours of both
  __shared__ T el[NW][2][3][64], eg[NW][2][4][64], eq[NW][2][2][64];

  const int b = blockIdx.x;  // XCD-aware tile order, as in the marching kernels
  const int tile = (b & 7) * A.per_xcd + (b >> 3);
  if (tile >= A.ntiles) return;
  int ty = (int)__umulhi((unsigned)tile, A.inv_ntx), tx = tile - ty * A.ntx;
  if (tx >= A.ntx) {
    ++ty;
    tx -= A.ntx;
  }
  const int nx = A.a.nx, ny = A.a.ny, halo = A.halo, ns = A.ns;
  const int x0 = tx * A.bw, y0 = ty * A.bh;
  const int xend = min(x0 + A.bw, nx), yend = min(y0 + A.bh, ny);
  const int rows = yend - y0 + 2 * halo;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int r0 = w * R;
  const int wa = w > 0 ? w - 1 : 0, wb = w + 1 < NW ? w + 1 : NW - 1;

  const int a = x0 - halo + lane;
  int col = a, y = y0 - halo + r0;
  while (col < 0) col += nx;
  while (col >= nx) col -= nx;
  while (y < 0) y += ny;
  while (y >= ny) y -= ny;
  const bool out = a >= x0 && a < xend;
  // every array is one buffer resource, its rows scalar offsets (block.h)
  auto ld = [](rsrc_t r, int o, int row) -> T {
    if constexpr (ES == 8) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, o, row, kLoadPolicy));
    else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, o, row, kLoadPolicy));
  };
  auto st = [](rsrc_t r, int o, int row, T v) {
    if constexpr (ES == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, o, row, kStorePolicy);
    else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, o, row, kStorePolicy);
  };
  auto next = [&](int &yr, int &o, int pitch) {
    ++yr;
    o += pitch;
    if (yr == ny) {
      yr = 0;
      o = 0;
    }
  };
  const int strip = col / kAdjW, pos = col - strip * kAdjW;
  const int off = W1 ? strip * AdjRec1<T>::RB + pos * ES : strip * AdjRec<T>::RB + pos * ES;
  const int off_st = out ? off : kDropOffset;
  const int rowA = A.a.nstrips * (W1 ? AdjRec1<T>::RB : AdjRec<T>::RB), lastA = (ny - 1) * rowA;
  const int rowG = A.a.nstrips * kGkRB, off_g = out ? strip * kGkRB + pos * 8 : kDropOffset;
  const int rowC = A.a.cnblk * A.a.capRB, segC = A.a.capB * ES;
  int cb = (int)__umulhi((unsigned)col, A.inv_capB);  // col / capB
  if (col - cb * A.a.capB >= A.a.capB) ++cb;
  const int off_c = cb * A.a.capRB + (col - cb * A.a.capB) * ES;

  // ---- the tile's adjoint lambda_l, kappa and dLoss/dkappa
  T lam[R][9], kap[R];
  T fh[W1 ? R : 1], fx[W1 ? R : 1], fy[W1 ? R : 1];  // omega = 1: lambda_h, lambda_j (lam_of)
  double gk[R];
  {
    const rsrc_t src = make_rsrc(A.a.src, (uint32_t)(ny * rowA)), rg = make_rsrc(A.a.gk, (uint32_t)(ny * rowG));
    int yr = y, o = y * rowA, og = y * rowG;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if constexpr (W1) {
        fh[i] = ld(src, off, o);
        fx[i] = ld(src, off + AdjRec1<T>::SEG, o);
        fy[i] = ld(src, off + 2 * AdjRec1<T>::SEG, o);
      } else {
        // lambda_l(x, y) is entry l of row y - c_ly
        const int rd[3] = {o == lastA ? 0 : o + rowA, o, o == 0 ? lastA : o - rowA};  // by c_ly + 1
#pragma unroll
        for (int l = 0; l < 9; ++l) lam[i][l] = ld(src, off + AdjRec<T>::seg(l), rd[kCy[l] + 1]);
      }
      gk[i] = 0.0;  // (of own sites only: the others' are their tiles')
      if (r0 + i >= halo && r0 + i < rows - halo)
        gk[i] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rg, off_g, og, kLoadPolicy));
      next(yr, o, rowA);
      og = yr == 0 ? 0 : og + rowG;
    }
    if (A.a.kfield != nullptr) {
      const int kpitch = A.a.ldx * ES;
      const rsrc_t rk = make_rsrc(A.a.kfield, (uint32_t)(ny * kpitch));
      yr = y;
      o = y * kpitch;
#pragma unroll
      for (int i = 0; i < R; ++i) {
        kap[i] = ld(rk, col * ES, o);
        next(yr, o, kpitch);
      }
    } else {
#pragma unroll
      for (int i = 0; i < R; ++i) kap[i] = C.kap0;
    }
  }
  auto spread = [&]() {
    if constexpr (W1) {
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int l = 0; l < 9; ++l) lam[i][l] = lam_of(l, fh[i], fx[i], fy[i]);
    }
  };
  spread();
  // forward moments of a step: h of the rows r0 - 1 .. r0 + R, j of the own rows
  T hn[R + 2], jxn[R], jyn[R];
  auto load_step = [&](int s) {
    const rsrc_t rc = make_rsrc(A.a.cap - s * A.cap_stride, (uint32_t)(ny * rowC));
    int yr = y == 0 ? ny - 1 : y - 1, o = yr * rowC;
#pragma unroll
    for (int i = 0; i < R + 2; ++i) {
      hn[i] = ld(rc, off_c, o);
      if (i >= 1 && i <= R) {
        jxn[i >= 1 && i <= R ? i - 1 : 0] = ld(rc, off_c + segC, o);
        jyn[i >= 1 && i <= R ? i - 1 : 0] = ld(rc, off_c + 2 * segC, o);
      }
      next(yr, o, rowC);
    }
  };
  load_step(0);

  for (int s = 0; s < ns; ++s) {
    // the rows whose lambda_p the stored rows still depend on (block_active)
    const bool act = r0 + R > 3 * s + 1 && r0 < rows - 3 * s - 1;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      el[w][0][q][lane] = lam[0][2 + q];
      el[w][1][q][lane] = lam[R - 1][6 + q];
    }
    __syncthreads();
    T mu[R][9], h[R], jx[R], jy[R], ih[R], rn[R], rm[R], Fx[R], Fy[R];
    T ga[R + 2], gb[R + 2], pa[R + 2], pb[R + 2];  // of the rows r0 - 1 .. r0 + R
    if (act) {
      // mu_l(x, y) = lambda_l(x + c_lx, y + c_ly)
      T up[3], dn[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        dn[q] = el[wb][0][q][lane];
        up[q] = el[wa][1][q][lane];
      }
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int l = 0; l < 9; ++l) {
          const int k = i + kCy[l];
          const T v = k >= R ? dn[l >= 2 && l <= 4 ? l - 2 : 0]
                             : (k < 0 ? up[l >= 6 ? l - 6 : 0] : lam[k < 0 || k >= R ? 0 : k][l]);
          mu[i][l] = kCx[l] == 0 ? v : (kCx[l] > 0 ? from_right(v) : from_left(v));
        }
      T hs[R + 2];  // h(x - 1) + h(x + 1)
#pragma unroll
      for (int i = 0; i < R + 2; ++i) hs[i] = from_left(hn[i]) + from_right(hn[i]);
#pragma unroll
      for (int i = 0; i < R; ++i) {
        h[i] = hn[1 + i];
        jx[i] = jxn[i];
        jy[i] = jyn[i];
        lambda_force(mu[i], C.cA, C.cD, Fx[i], Fy[i]);
        // lambda_G = -h Lambda_F, and the forward film pressure
        const T gx = -h[i] * Fx[i], gy = -h[i] * Fy[i];
        ga[1 + i] = from_right(gx) - from_left(gx);
        gb[1 + i] = madd(C.cA, gy, C.cD * (from_left(gy) + from_right(gy)));
        const T lap = (T(4) * ((hs[1 + i] + hn[i + 2]) + hn[i]) + (hs[i + 2] + hs[i]) - T(20) * h[i]) * T(1.0 / 6.0);
        ih[i] = recip(h[i]);
        const T r = C.hstar * ih[i], r3 = r * r * r, r9 = r3 * r3 * r3;
        rn[i] = A.n9 ? r9 : r3;
        rm[i] = A.n9 ? r3 : r9;
        const T p = -C.gamma * (lap + kap[i] * (rn[i] - rm[i]));
        pa[1 + i] = from_right(p) - from_left(p);
        pb[1 + i] = madd(C.cA, p, C.cD * (from_left(p) + from_right(p)));
      }
      const T e[2][4] = {{ga[1], gb[1], pa[1], pb[1]}, {ga[R], gb[R], pa[R], pb[R]}};
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q) eg[w][k][q][lane] = e[k][q];
    }
    if (s + 1 < ns) load_step(s + 1);
    __syncthreads();
    T q[R + 2], qs[R + 2];  // lambda_p and the sum of its x neighbours
    if (act) {
      T *const edge[4] = {ga, gb, pa, pb};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        edge[k][0] = eg[wa][1][k][lane];
        edge[k][R + 1] = eg[wb][0][k][lane];
      }
#pragma unroll
      for (int i = 1; i <= R; ++i) {
        q[i] = -(madd(C.cA, ga[i], C.cD * (ga[i + 1] + ga[i - 1])) + (gb[i + 1] - gb[i - 1]));
        qs[i] = from_left(q[i]) + from_right(q[i]);
      }
      eq[w][0][0][lane] = q[1];
      eq[w][0][1][lane] = qs[1];
      eq[w][1][0][lane] = q[R];
      eq[w][1][1][lane] = qs[R];
    }
    __syncthreads();
    if (act) {
      q[0] = eq[wa][1][0][lane];
      qs[0] = eq[wa][1][1][lane];
      q[R + 1] = eq[wb][0][0][lane];
      qs[R + 1] = eq[wb][0][1][lane];
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const T Gx = madd(C.cA, pa[i + 1], C.cD * (pa[i + 2] + pa[i]));
        const T Gy = pb[i + 2] - pb[i];
        const T lapq = (T(4) * ((qs[i + 1] + q[i + 2]) + q[i]) + (qs[i + 2] + qs[i]) - T(20) * q[i + 1]) * T(1.0 / 6.0);
        T lh, ljx, ljy;
        double gt;
        adj_site(C, mu[i], h[i], ih[i], rn[i], rm[i], jx[i], jy[i], kap[i], Fx[i], Fy[i], Gx, Gy, lapq, q[i + 1], lh, ljx,
                 ljy, gt);
        gk[i] += gt;
        if constexpr (W1) {
          fh[i] = lh;
          fx[i] = ljx;
          fy[i] = ljy;
        } else {
#pragma unroll
          for (int l = 0; l < 9; ++l) lam[i][l] = madd(C.om1, mu[i][l], lam_of(l, lh, ljx, ljy));
        }
      }
      spread();
    }
  }

  // ---- the tile's own rows
  const rsrc_t dst = make_rsrc(A.a.dst, (uint32_t)(ny * rowA)), rg = make_rsrc(A.a.gk, (uint32_t)(ny * rowG));
  int yr = y, o = y * rowA, og = y * rowG;
#pragma unroll
  for (int i = 0; i < R; ++i) {
    if (r0 + i >= halo && r0 + i < rows - halo) {
      if constexpr (W1) {
        st(dst, off_st, o, fh[i]);
        st(dst, off_st + AdjRec1<T>::SEG, o, fx[i]);
        st(dst, off_st + 2 * AdjRec1<T>::SEG, o, fy[i]);
      } else {
        const int rd[3] = {o == lastA ? 0 : o + rowA, o, o == 0 ? lastA : o - rowA};  // by c_ly + 1
#pragma unroll
        for (int l = 0; l < 9; ++l) st(dst, off_st + AdjRec<T>::seg(l), rd[kCy[l] + 1], lam[i][l]);
      }
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, gk[i]), rg, off_g, og, kStorePolicy);
    }
    next(yr, o, rowA);
    og = yr == 0 ? 0 : og + rowG;
  }
}

}  // namespace tflbm
