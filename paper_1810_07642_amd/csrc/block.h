// The block kernel: several time steps of one tile of the lattice per launch,
// with the tile's state in registers (internal to the library; instantiated
// per storage form and collision stage in block_form.hip).
//
// A workgroup of NW wavefronts owns a tile of 64 columns and NW R rows: lane i
// of wavefront w holds column i of the rows w R .. w R + R - 1.  The outermost
// `halo` = 3 ns columns and rows of the tile are re-computed by its neighbours
// (a step reads three sites in each direction); the rest is stored after ns
// steps.  Stencil neighbours in x come from adjacent lanes, in y from the
// lane's own registers and, at the edge of a wavefront's rows, from the
// neighbouring wavefront through LDS: dh, then the film pressure, then the six
// populations that stream across, a barrier each.
//
// With omega = 1 a site's populations are a function of its moments and force,
// so nothing but dh and j has to leave the chip between two passes of a call:
// the first pass reads populations, the last one writes them, and those between
// read and write moments (in the first three segments of the c_ly = 0 group of
// the same records, so that no padding byte changes), a third of the bytes and
// the same bits.
//
// Against the marching kernel (step.h), whose wavefronts walk down a strip one
// row after the other, every row of a tile is in flight at once.  On lattices
// that do not fill the GPU with long strips a marching tile's time is its
// chain of rows; here it is ns times three exchanges.  Measured (us per step,
// marching / block, step graphs on): FP32 at omega = 1 64^2 4.6 / 2.2, 256^2
// 5.3 / 2.5, 512^2 9.1 / 4.1, 1024x512 11.2 / 6.3, 1024^2 14.9 / 10.8; FP32
// general 256^2 5.8 / 2.8, 512^2 9.0 / 4.7; FP16S at omega = 1 128^2 5.2 / 2.6,
// 512^2 9.1 / 4.8, 901x641 (odd width) 24.0 / 7.7; FP64 at omega = 1 64^2 3.8 / 2.7,
// 512^2 10.2 / 5.2; FP64 general 64^2 4.0 / 3.1, 384^2 8.4 / 4.6, 512^2 10.8 /
// 9.4 (its tiles hold two rows per wavefront at most: 2 x 9 FP64 populations).
// What is left of a pass: about 2.5 us of launch, 1.5-2 us until the state is
// in registers, and the steps, bound by VALU issue (3.9 cycles per instruction
// and SIMD at four wavefronts, of which DPP moves and reciprocals take 4 to 16).
#pragma once

#include "step.h"

namespace tflbm {

// Shapes per storage form and stage: rows per wavefront and wavefronts per
// workgroup.  A tile's cost is its region, rows x 64, against the output that
// remains inside the halo, so a lattice that leaves CUs idle wants low tiles and
// many steps, a larger one high tiles; sixteen wavefronts (four per SIMD) issue
// FP32 twice as fast as two per SIMD (2.1-2.6 against 4.2 cycles per
// instruction), and FP64 a little faster than twelve (us per step at omega = 1,
// tiles of 48 rows as 3 x 16 / 4 x 12: 512^2 5.2 / 5.3, 901x641 10.1 / 10.5).  The
// lists hold the fewest shapes within 1-7 % of the best of 14 (FP32, omega = 1),
// 9 and 4 measured.
template <int P, bool W1> struct BlockShapes;
template <> struct BlockShapes<kF32, true> {
  static constexpr BlockShape list[] = {{2, 16}, {3, 16}, {5, 16}};
};
template <> struct BlockShapes<kF32, false> {
  static constexpr BlockShape list[] = {{2, 16}, {3, 8}};
};
template <> struct BlockShapes<kF16S, true> {
  static constexpr BlockShape list[] = {{2, 16}, {3, 16}, {5, 16}};
};
template <> struct BlockShapes<kF16S, false> {
  static constexpr BlockShape list[] = {{2, 16}, {3, 8}};
};
template <> struct BlockShapes<kF64, true> {
  static constexpr BlockShape list[] = {{2, 16}, {3, 16}};
};
template <> struct BlockShapes<kF64, false> {
  static constexpr BlockShape list[] = {{1, 16}, {2, 12}};
};

template <int P, bool W1, bool GF, bool G0, bool CAP, int R, int NW>
__global__ __launch_bounds__(64 * NW) void block_kernel(BlockArgs A, Coef<typename Form<P>::T> C) {
  using T = typename Form<P>::T;
  constexpr bool F16 = P == kF16S;
  constexpr int B = Form<P>::B, RB = Form<P>::RB, ES = sizeof(T), SEG = B * ES, CRB = cap_record_bytes<P>();
  // dh and p of a wavefront's first and last row; of the populations, those
  // that leave it downwards (2, 3, 4 of its last row) and upwards (6, 7, 8 of
  // its first row)
  __shared__ T eh[NW][2][64], ep[NW][2][64], ef[NW][6][64];

  // XCD-aware tile order, as in step_kernel
  const int b = blockIdx.x;
  const int tile = (b & 7) * A.per_xcd + (b >> 3);
  if (tile >= A.ntiles) return;
  // tile / ntx by its reciprocal (rounded down: at most one too small)
  int ty = (int)__umulhi((unsigned)tile, A.inv_ntx), tx = tile - ty * A.ntx;
  if (tx >= A.ntx) {
    ++ty;
    tx -= A.ntx;
  }
  const int nx = A.s.nx, ny = A.s.ny, halo = A.halo, ns = A.ns;
  const int x0 = tx * A.bw, y0 = ty * A.bh;
  const int xend = min(x0 + A.bw, nx), yend = min(y0 + A.bh, ny);
  const int rows = yend - y0 + 2 * halo;  // rows of the tile that are in use
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int r0 = w * R;  // tile row of the wavefront's first row
  const int wa = w > 0 ? w - 1 : 0, wb = w + 1 < NW ? w + 1 : NW - 1;  // (the ends: rows nothing stored depends on)
  const int rowB = A.s.nblk * RB;

  // Lattice columns a - 1, a, a + 1 of the lane and lattice row of the
  // wavefront's first row.  A tile reaches less than one lattice beyond it
  // unless the lattice is smaller than a tile: loops of no or one turn, where a
  // division would cost every launch some twenty instructions per wavefront.
  const int a = x0 - A.halo_x + lane;
  int col[3], y = y0 - halo + r0;
  col[0] = a - 1;
  while (col[0] < 0) col[0] += nx;
  while (col[0] >= nx) col[0] -= nx;
#pragma unroll
  for (int j = 1; j < 3; ++j) col[j] = col[j - 1] + 1 == nx ? 0 : col[j - 1] + 1;
  while (y < 0) y += ny;
  while (y >= ny) y -= ny;
  int off[3];  // byte offsets of the three columns in a row of records
#pragma unroll
  for (int j = 0; j < 3; ++j) off[j] = col[j] / B * RB + col[j] % B * ES;
  const int off16 = col[1] / B * RB + col[1] % B * 2;  // FP16S: of column a in an FP16 segment
  const bool out = a >= x0 && a < xend;  // a column of the tile's own
  const int off_st = out ? off[1] : kStoreDrop, off_st16 = out ? off16 : kStoreDrop;
  // Every array is one buffer resource, its rows scalar byte offsets (the
  // library runs this kernel on arrays under 2 GiB only): building a resource
  // per row costs each wavefront some twenty scalar instructions a row (8 % of
  // the time per step on lattices of 64^2 to 640^2 sites).
  auto ld = [](rsrc_t r, int o, int row) -> T {
    if constexpr (P == kF64) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, o, row, kLoadPolicy));
    else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, o, row, kLoadPolicy));
  };
  auto st = [](rsrc_t r, int o, int row, T v) {
    if constexpr (P == kF64) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, o, row, kStorePolicy);
    else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, o, row, kStorePolicy);
  };
  auto ld16 = [](rsrc_t r, int o, int row) -> unsigned short {
    return __builtin_amdgcn_raw_buffer_load_b16(r, o, row, kLoadPolicy);
  };
  auto st16 = [](rsrc_t r, int o, int row, unsigned int v) {
    __builtin_amdgcn_raw_buffer_store_b16((unsigned short)v, r, o, row, kStorePolicy);
  };
  // FP16S keeps j in the two halves of four FP16 segments
  constexpr int kHalf[2][2] = {{1, 5}, {2, 3}};
  // the next row and its offset in an array of `pitch` bytes per row
  auto next = [&](int &yr, int &o, int pitch) {
    ++yr;
    o += pitch;
    if (yr == ny) {
      yr = 0;
      o = 0;
    }
  };

  // ---- the tile's state: populations, or with omega = 1 dh and j; and per
  // site kr = -gamma kappa (with ksign) and, with a surface tension field, ar =
  // -gamma/6, rounded as the marching kernel rounds them
  T f[R][9], dh[R], jx[W1 ? R : 1], jy[W1 ? R : 1], kr[R], ar[GF ? R : 1];
  const bool in_mom = W1 && A.in_mom;
  {
    const rsrc_t src = make_rsrc(A.s.src, (uint32_t)(ny * rowB));
    int yr = y, o = y * rowB;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if (in_mom) {
        const int k = W1 ? i : 0;
        dh[i] = ld(src, off[1], o);
        if constexpr (F16) {
          T *const j[2] = {&jx[k], &jy[k]};
#pragma unroll
          for (int d = 0; d < 2; ++d) {
            const unsigned int hi = ld16(src, off16 + seg_offset<P>(kHalf[d][0]), o),
                               lo = ld16(src, off16 + seg_offset<P>(kHalf[d][1]), o);
            *j[d] = __uint_as_float(hi << 16 | lo);
          }
        } else {
          jx[k] = ld(src, off[1] + SEG, o);
          jy[k] = ld(src, off[1] + 2 * SEG, o);
        }
      } else if constexpr (!F16) {
#pragma unroll
        for (int l = 0; l < 9; ++l) f[i][l] = ld(src, off[1 - kCx[l]] + seg_offset<P>(l), o);
      }
      next(yr, o, rowB);
    }
    if constexpr (F16) {
      if (!in_mom) {
        // decode as fp16s_decode does: the moving populations of a row with the
        // rest equilibrium of their source rows, the implied rest population from
        // those the row emitted into the rows around it; then the x shift
        const int last = (ny - 1) * rowB;
        T sh[R + 2], q[R + 2][9];
        o = y == 0 ? last : (y - 1) * rowB;
        yr = y == 0 ? ny - 1 : y - 1;
#pragma unroll
        for (int i = 0; i < R + 2; ++i) {
          sh[i] = ld(src, off[1], o);
#pragma unroll
          for (int l = 1; l < 9; ++l)
            if ((i >= 1 && i <= R) || (i == 0 && l >= 6) || (i == R + 1 && l >= 2 && l <= 4))
              q[i][l] = dec16(__ushort_as_half(ld16(src, off16 + seg_offset<P>(l), o)), A.s.qinv);
          next(yr, o, rowB);
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
          T t[9], d[9];
          t[0] = 0.0f;
          if constexpr (G0) {
#pragma unroll
            for (int l = 1; l < 9; ++l) {
              d[l] = q[1 + i][l];
              t[l] = q[1 + i + kCy[l]][l];
            }
          } else {
            const float h2 = 2.0f * C.href;
            const Rest16 e[3] = {rest16(sh[i], C.g, h2), rest16(sh[1 + i], C.g, h2), rest16(sh[2 + i], C.g, h2)};
#pragma unroll
            for (int l = 1; l < 9; ++l) {
              d[l] = rest16_l(e[1 - kCy[l]], l) + q[1 + i][l];
              t[l] = rest16_l(e[1], l) + q[1 + i + kCy[l]][l];
            }
          }
          d[0] = rest16_d0(sh[1 + i], t);
#pragma unroll
          for (int l = 0; l < 9; ++l) shift_x<T, 1>(l, &d[l], &f[i][l]);
        }
      }
    }
    const T sg = (T)A.ksign;
    if (GF || A.kf == kKappa) {
      const int kpitch = A.s.ldx * ES * (GF ? 2 : 1), c = col[1] * (GF ? 2 * ES : ES);
      const rsrc_t kap = make_rsrc(A.s.kfield, (uint32_t)(ny * kpitch));
      yr = y;
      o = y * kpitch;
#pragma unroll
      for (int i = 0; i < R; ++i) {
        if constexpr (GF) {
          ar[i] = ld(kap, c, o);
          kr[i] = sg * ld(kap, c + ES, o);
        } else {
          kr[i] = sg * (C.mgam * ld(kap, c, o));
        }
        next(yr, o, kpitch);
      }
    } else {
#pragma unroll
      for (int i = 0; i < R; ++i) kr[i] = sg * (C.mgam * C.kap0);
    }
  }
  // dh (and with omega = 1 j) of the populations
  auto moments = [&]() {
#pragma unroll
    for (int i = 0; i < R; ++i) {
      T hs = f[i][0];
#pragma unroll
      for (int l = 1; l < 9; ++l) hs += f[i][l];
      dh[i] = hs;
      if constexpr (W1) momentum(f[i], jx[i], jy[i]);
    }
  };
  if (!in_mom) moments();

  unsigned long long bad = 0;  // lanes that met a height that is not positive and finite
  const unsigned long long own = __ballot(out);
  const int rowc = A.s.nblk * CRB;
  const size_t capblk = (size_t)ny * rowc;
  for (int s = 0; s < ns; ++s) {
    const bool act = block_active(r0, R, rows, s);
    eh[w][0][lane] = dh[0];
    eh[w][1][lane] = dh[R - 1];
    __syncthreads();
    T pr[R], ih[R];
    if (act) {
      // film pressure of the wavefront's rows (hx: dh of the rows r0 - 1 .. r0 + R)
      T hx[R + 2][3];
      hx[0][1] = eh[wa][1][lane];
      hx[R + 1][1] = eh[wb][0][lane];
#pragma unroll
      for (int i = 0; i < R; ++i) hx[1 + i][1] = dh[i];
#pragma unroll
      for (int i = 0; i < R + 2; ++i) row_sums<1>(hx[i]);
#pragma unroll
      for (int i = 0; i < R; ++i) {
        ih[i] = recip(C.href + dh[i]);
        const T lap6 = laplacian6(hx[i + 2], hx[i + 1], hx[i]);
        const T r = C.hstar * ih[i], r3 = r * r * r, phi = r3 * r3 * r3 - r3;
        if constexpr (GF) pr[i] = madd(ar[i], lap6, kr[i] * phi);
        else pr[i] = madd(C.mgam6, lap6, kr[i] * phi);
      }
      ep[w][0][lane] = pr[0];
      ep[w][1][lane] = pr[R - 1];
    }
    __syncthreads();
    if (act) {
      // x difference and x-smoothed pressure of the rows r0 - 1 .. r0 + R
      T dx[R + 2], sm[R + 2];
#pragma unroll
      for (int i = 0; i < R + 2; ++i) {
        const T p = i == 0 ? ep[wa][1][lane] : (i == R + 1 ? ep[wb][0][lane] : pr[i == 0 || i == R + 1 ? 0 : i - 1]);
        const T pl = from_left(p), pq = from_right(p);
        dx[i] = pq - pl;
        sm[i] = madd(C.cA, p, C.cD * (pl + pq));
      }
      int yr = y, o = y * rowc;
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const bool mine = r0 + i >= halo && r0 + i < rows - halo;
        const T gx = madd(C.cA, dx[i + 1], C.cD * (dx[i + 2] + dx[i]));
        const T gy = sm[i + 2] - sm[i];
        const T h = C.href + dh[i];
        T jxv, jyv;
        if constexpr (W1) {
          jxv = jx[i];
          jyv = jy[i];
        } else {
          momentum(f[i], jxv, jyv);
        }
        T pv[9];
        collide<T, W1, G0>(C, h, ih[i], gx, gy, dh[i], jxv, jyv, f[i], pv);
#pragma unroll
        for (int l = 0; l < 9; ++l) f[i][l] = pv[l];
        if (mine) bad |= own & __ballot(!(h > T(0) && h < T(INFINITY)));
        if constexpr (CAP) {
          if (mine) {
            const rsrc_t cap = make_rsrc(A.s.capture + s * capblk, (uint32_t)capblk);
            const int c = out ? col[1] / B * CRB + col[1] % B * ES : kStoreDrop;
            st(cap, c, o, C.href + dh[i]);
            st(cap, c + SEG, o, jxv);
            st(cap, c + 2 * SEG, o, jyv);
          }
          next(yr, o, rowc);
        }
      }
    }
    if (s + 1 == ns && !(W1 && A.out_mom)) break;
    if constexpr (F16) {
      if (act) {
#pragma unroll
        for (int i = 0; i < R; ++i) {  // as if stored and loaded again
          T pv[9][1];
          const T hv[1] = {dh[i]};
#pragma unroll
          for (int l = 0; l < 9; ++l) pv[l][0] = f[i][l];
          fp16s_roundtrip<1, G0>(pv, hv, A.s);
#pragma unroll
          for (int l = 0; l < 9; ++l) f[i][l] = pv[l][0];
        }
      }
    }
    if (act) {
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        ef[w][q][lane] = f[R - 1][2 + q];
        ef[w][3 + q][lane] = f[0][6 + q];
      }
    }
    __syncthreads();
    if (act) {
      // streaming: the value at (x, y) comes from (x - c_lx, y - c_ly)
      T up[3], dn[3];  // populations 2, 3, 4 of the row above and 6, 7, 8 of the row below
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        up[q] = ef[wa][q][lane];
        dn[q] = ef[wb][3 + q][lane];
      }
#pragma unroll
      for (int l = 0; l < 9; ++l) {
        T t[R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
          const int k = i - kCy[l];
          const T v = k < 0 ? up[l >= 2 && l <= 4 ? l - 2 : 0] : (k >= R ? dn[l >= 6 ? l - 6 : 0] : f[k < 0 || k >= R ? 0 : k][l]);
          shift_x<T, 1>(l, &v, &t[i]);
        }
#pragma unroll
        for (int i = 0; i < R; ++i) f[i][l] = t[i];
      }
      moments();
    }
  }

  // ---- the tile's own rows: the populations after the collision of the last
  // step, at their columns in rows y + c_ly, or the moments
  {
    const rsrc_t dst = make_rsrc(A.s.dst, (uint32_t)(ny * rowB));
    const int last = (ny - 1) * rowB;
    int yr = y, o = y * rowB;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if (r0 + i >= halo && r0 + i < rows - halo) {
        if (W1 && A.out_mom) {
          const int k = W1 ? i : 0;
          st(dst, off_st, o, dh[i]);
          if constexpr (F16) {
            const T j[2] = {jx[k], jy[k]};
#pragma unroll
            for (int d = 0; d < 2; ++d) {
              const unsigned int u = __float_as_uint(j[d]);
              st16(dst, off_st16 + seg_offset<P>(kHalf[d][0]), o, u >> 16);
              st16(dst, off_st16 + seg_offset<P>(kHalf[d][1]), o, u & 0xffffu);
            }
          } else {
            st(dst, off_st + SEG, o, jx[k]);
            st(dst, off_st + 2 * SEG, o, jy[k]);
          }
        } else {
          const int rd[3] = {o == 0 ? last : o - rowB, o, o == last ? 0 : o + rowB};  // by c_ly + 1
          if constexpr (F16) {
            st(dst, off_st, o, dh[i]);
            const Rest16 e = rest16(dh[i], C.g, 2.0f * C.href);
#pragma unroll
            for (int l = 1; l < 9; ++l) {
              const float d = G0 ? f[i][l] : f[i][l] - rest16_l(e, l);
              st16(dst, off_st16 + seg_offset<P>(l), rd[kCy[l] + 1],
                   __builtin_bit_cast(unsigned short, (_Float16)(d * A.s.qscale)));
            }
          } else {
#pragma unroll
            for (int l = 0; l < 9; ++l) st(dst, off_st + seg_offset<P>(l), rd[kCy[l] + 1], f[i][l]);
          }
        }
      }
      next(yr, o, rowB);
    }
  }
  if (bad != 0 && lane == __ffsll(bad) - 1) atomicOr(A.s.flag, 1);
}

}  // namespace tflbm
