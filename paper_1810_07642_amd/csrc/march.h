// Marching kernels that hand the moments from pass to pass (omega = 1; internal
// to the library, instantiated per storage form in march_form.hip).
//
// With omega = 1 the populations that leave a step are a function of the
// moments (dh, j) and the force of the site, and the next step reads nothing of
// them but their sums dh and j after streaming.  The passes of a call of several
// passes therefore need not store nine populations in between: the first
// reads populations and writes moments, those between read and write
// moments, the last one writes populations, so that the state a call leaves, its
// readout and its checkpoints are those of step_kernel bit for bit.  The last
// stage of a pass that writes moments streams its rows in registers like the
// stages before it (Handoff) and adds them up.  The moments lie in the records
// of the population buffers (moment_offset): no memory is added.
//
// Structure, tile walk and stages are those of step_kernel (step.h).  A pass
// between two others moves 12 + 12 B per site in FP32 (24 + 24 in FP64) where
// step_kernel moves 36 + 36 (72 + 72).  Measured, us per step, step_kernel /
// these passes: FP32 2048^2 33.6 / 23.1, 4096^2 104 / 68.5; FP64 1024^2 19.8 /
// 13.7, 2048^2 57.0 / 35.7, 4096^2 198 / 132.5.  They are bound by VALU issue
// now: the FP64 pass of three steps at 4096^2 issues 157k instructions per SIMD
// in 0.86 M busy cycles (4.2-4.4 cycles each at FP64 rate, its two hardware
// reciprocals per site 16), moves 1.03 GB at 2.5 TB/s, and computes 1.53 sites
// (18 halo columns of 64, 18 halo rows of a 187-row chunk) per site it stores.
#pragma once

#include "step.h"

namespace tflbm {

// Byte offset of dh of a column in a row of moments.  The moments of the three
// records 3 j .. 3 j + 2 lie in the three c_ly groups of record j (dh, j_x and
// j_y in a group's three segments), so that a row's moments are contiguous
// but for the groups' padding, which keeps its zeros, and no byte past the last
// column is written.
template <int P> __device__ __forceinline__ int moment_offset(int col) {
  using F = Form<P>;
  const int blk = col / F::B;
  return blk / 3 * F::RB + blk % 3 * F::GRP + (col - blk * F::B) * (int)sizeof(typename F::T);
}

// Output columns of a strip: one record where populations are read or
// written, else all that the halo of the fused steps leaves (an even halo for
// two columns per lane).
template <int P, int NS, bool MI, bool MO> __host__ __device__ constexpr int march_columns() {
  constexpr int V = Form<P>::V, halo = V == 2 ? (3 * NS + 1) / 2 * 2 : 3 * NS;
  return MI && MO ? 64 * V - 2 * halo : Form<P>::B;
}

// The stages of a pass and what happens to the rows they emit.
template <int P, int KF, bool CAP, int NS, bool MO, bool G0, bool PAD> struct March {
  using T = typename Form<P>::T;
  static constexpr int V = Form<P>::V, B = Form<P>::B, RB = Form<P>::RB, SEG = Form<P>::SEG;
  static constexpr int HALO = MO ? 3 * NS : 3 * NS - 1;
  // first row iteration whose last stage's row is stored: each stage emits from
  // its fifth row on, stage s starts six rows after stage s - 1, and moments
  // come two rows after the populations they are made of
  static constexpr int KST = 4 + 6 * (NS - 1) + (MO ? 2 : 0);
  static constexpr int KQ = 3 * (NS - 1);  // rows between the first stage and the last
  Stage<P, KF, true, G0, true> st[NS];
  Handoff<T, V> ho[NS];
  T (*kring)[64 * V];      // kappa of stage 0's last KQ rows, for the later stages (a ring in LDS)
  int kslot = 0;           // the slot of the current row
  int bad = 0;
  int y0, yend, x0, xend, lane;
  int om[V];               // byte offsets of the lane's columns in a row of moments
  int opad;                // the lane's word of the padding after the strip's group of moments, or kStoreDrop
  size_t capblk;

  // Moments of row y into its records; UNI: on every path, lanes without
  // output dropped.
  template <bool UNI>
  __device__ __forceinline__ void store_moments(const StepArgs &A, int y, const T (&g)[9][V], const Lane<P> &L) {
    const size_t rowB = (size_t)A.nblk * RB;
    const rsrc_t row = make_rsrc(A.dst + y * rowB, (uint32_t)rowB);
    T m[3][V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      T fv[9], hs = g[0][v];
#pragma unroll
      for (int l = 1; l < 9; ++l) hs += g[l][v];
#pragma unroll
      for (int l = 0; l < 9; ++l) fv[l] = g[l][v];
      m[0][v] = hs;
      momentum(fv, m[1][v], m[2][v]);
    }
    if constexpr (V == 1) {
      const int o = L.out[0] ? om[0] : kStoreDrop;
#pragma unroll
      for (int i = 0; i < 3; ++i) st_t(row, o + i * SEG, m[i][0]);
    } else if constexpr (UNI) {
      const int o = L.pair ? om[0] : kStoreDrop;
#pragma unroll
      for (int i = 0; i < 3; ++i) st_f32x2(row, o + i * SEG, m[i][0], m[i][1]);
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const int o = L.out[v] ? om[v] : kStoreDrop;
#pragma unroll
        for (int i = 0; i < 3; ++i) st_t(row, o + i * SEG, m[i][v]);
      }
    }
    // the padding, so that the group's last line is written whole
    if constexpr (PAD) st_f32(row, opad, 0.f);
  }

  // Stage S emitted its row q at its own iteration k.
  template <int S, bool UNI>
  __device__ __forceinline__ void emitted(const StepArgs &A, const Coef<T> &C, const Lane<P> &L, int k, int q,
                                          T (&post)[9][V], const T (&hv)[V], const T (&jx)[V], const T (&jy)[V]) {
    if constexpr (CAP) {
      const bool valid = q >= y0 && q < yend;
      if constexpr (UNI) capture_row<P, true>(A, A.capture + S * capblk, q, hv, jx, jy, L, C.href, x0, xend, lane, valid);
      else if (valid) capture_row<P>(A, A.capture + S * capblk, q, hv, jx, jy, L, C.href, x0, xend, lane);
    }
    if constexpr (S + 1 == NS && !MO) {
      store_row<P, G0, UNI>(A, q, post, hv, L, x0, xend, lane);
    } else {
      T g[9][V];
      ho[S].feed(post, g);  // row q - 1 of the next step
      if (k >= 6) {
        if constexpr (S + 1 == NS) {
          store_moments<UNI>(A, q - 1, g, L);
        } else {
          T unused[9][V];
          T kap[V] = {}, none[V] = {};
          if constexpr (KF != kNoField) {
            // the row's kappa came in 3 (S + 1) rows ago
            int slot = kslot - 3 * (S + 1);
            slot = slot < 0 ? slot + KQ : slot;
#pragma unroll
            for (int v = 0; v < V; ++v) kap[v] = kring[slot][V * lane + v];
          }
          st[S + 1].ingest(k - 6, g, kap, none, unused, lane);
          T post2[9][V], hv2[V], jx2[V], jy2[V];
          if (st[S + 1].finish(k - 6, unused, post2, hv2, jx2, jy2, C, L, bad))
            emitted<S + 1, UNI>(A, C, L, k - 6, q - 3, post2, hv2, jx2, jy2);
        }
      }
    }
  }
};

// NS steps; MI / MO: moments in / out (else populations); PF: rows are loaded
// that many rows ahead of their use; U: rows per turn of the row loop.
template <int P, int KF, bool CAP, int NS, bool MI, bool MO, bool G0, int PF, int U>
__global__ __launch_bounds__(64, 2) void march_kernel(StepArgs A) {
  using T = typename Form<P>::T;
  static_assert(P == kF64 || P == kF32, "storage forms with one element type");
  constexpr int V = Form<P>::V, B = Form<P>::B, RB = Form<P>::RB, SEG = Form<P>::SEG;
  constexpr int SW = march_columns<P, NS, MI, MO>(), HX = (64 * V - SW) / 2;
  constexpr bool PAD = MO && SW == B;  // a strip writes one record's moments
  using M = March<P, KF, CAP, NS, MO, G0, PAD>;
  constexpr int HALO = M::HALO, KST = M::KST, KQ = M::KQ;
  // columns a pass loses per side: three per step, one where populations are
  // shifted into place, less one where the last stage's rows are not streamed
  static_assert(HX >= 3 * NS + (MI ? 0 : 1) - (MO ? 0 : 1), "halo columns too narrow for the fused steps");
  __shared__ T jhist[NS][2][2][64 * V], kring[KF == kNoField ? 1 : KQ][64 * V];

  const int b = blockIdx.x;  // XCD-aware tile order, as in step_kernel
  const int tile = (b & 7) * A.per_xcd + (b >> 3);
  if (tile >= A.ntiles) return;
  const int strip = tile % A.nstrips, chunk = tile / A.nstrips;
  M m;
  m.lane = threadIdx.x;
  m.x0 = strip * SW;
  m.y0 = chunk * A.H;
  m.yend = min(m.y0 + A.H, A.ny);
  m.xend = min(m.x0 + SW, A.nx);
  m.capblk = (size_t)A.ny * A.nblk * cap_record_bytes<P>();
#pragma unroll
  for (int s = 0; s < NS; ++s) m.st[s].jhist = jhist[s];
  m.kring = kring;
  const int ny = A.ny;
  const size_t rowB = (size_t)A.nblk * RB;
  const Lane<P> L(m.x0 - HX + V * m.lane, m.x0, m.xend, A.nx);
#pragma unroll
  for (int v = 0; v < V; ++v) m.om[v] = moment_offset<P>(L.col[v]);
  m.opad = PAD && m.xend - m.x0 == B && 4 * m.lane < pad_bytes<P>(0) ? moment_offset<P>(m.x0) + 3 * SEG + 4 * m.lane : kStoreDrop;
  const Coef<T> C(A);

  const int K = (m.yend - m.y0) + 2 * HALO;
  auto rsrc_src = [&](int row) { return make_rsrc(A.src + row * rowB, (uint32_t)rowB); };
  constexpr int NL = MI ? 3 : 9;  // segments of a row
  int ry = wrap(m.y0 - HALO, ny), rpre = (ry + PF) % ny;
  const uint32_t kpitch = (uint32_t)(A.ldx * sizeof(T));
  auto rsrc_kap = [&](int row) { return make_rsrc((const char *)A.kfield + (size_t)row * kpitch, kpitch); };
  using Word = std::conditional_t<P == kF32, unsigned long long, double>;
  auto run = [&](auto av) {
    constexpr bool AV = decltype(av)::value;
    constexpr bool UNI = P == kF64 || AV;
    Word fa[NL], fb[NL], fc[NL];  // values of rows r (being consumed), r + 1 and r + 2
    KapBuf<P, KF> ka, kb, kc;
    auto load_buf = [&](rsrc_t row, Word (&out)[NL]) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int seg = MI ? i * SEG : seg_offset<P>(i);
        const int o0 = MI ? m.om[0] : L.oe[0], o1 = MI ? m.om[V - 1] : L.oe[V - 1];
        if constexpr (P == kF64) {
          out[i] = ld_f64(row, o0 + seg);
        } else if (AV || L.allvec) {
          out[i] = __builtin_bit_cast(Word, __builtin_amdgcn_raw_buffer_load_b64(row, o0 + seg, 0, kLoadPolicy));
        } else {
          const u32x2 w = {__builtin_amdgcn_raw_buffer_load_b32(row, o0 + seg, 0, kLoadPolicy),
                           __builtin_amdgcn_raw_buffer_load_b32(row, o1 + seg, 0, kLoadPolicy)};
          out[i] = __builtin_bit_cast(Word, w);
        }
      }
    };
    auto columns = [](const Word &w, T (&c)[V]) {
      if constexpr (P == kF64) {
        c[0] = w;
      } else {
        const u32x2 u = __builtin_bit_cast(u32x2, w);
        c[0] = __uint_as_float(u.x);
        c[V - 1] = __uint_as_float(u.y);
      }
    };
    auto load_first = [&](int i, Word (&f)[NL], KapBuf<P, KF> &kap) {
      const int r = (ry + i) % ny;
      load_buf(rsrc_src(r), f);
      if constexpr (KF != kNoField) load_kappa<P, KF>(rsrc_kap(r), L, kap);
    };
    load_first(0, fa, ka);
    if constexpr (PF >= 2) load_first(1, fb, kb);  // (K > 2 HALO >= 10)
    if constexpr (PF >= 3) load_first(2, fc, kc);
    if constexpr (UNI) drop_row_stores<P, MO ? 3 + PAD : 12>(A);

    auto iteration = [&](int k, Word (&cur)[NL], KapBuf<P, KF> &kcur) {
      T k0[V] = {}, a0[V] = {}, f2[9][V];
      if constexpr (KF != kNoField) kappa_cols<P, KF>(kcur, k0, a0);
      if constexpr (MI) {
        T dh[V], jx[V], jy[V];
        columns(cur[0], dh);
        columns(cur[1], jx);
        columns(cur[2], jy);
        m.st[0].ingest(k, dh, jx, jy, k0, a0, m.lane);
      } else {
        T f[9][V];
#pragma unroll
        for (int l = 0; l < 9; ++l) {
          T c[V];
          columns(cur[l], c);
          shift_x<T, V>(l, c, f[l]);
        }
        m.st[0].ingest(k, f, k0, a0, f2, m.lane);
      }
      // prefetch row r + PF (past the tile's last row an empty range, as in step_kernel)
      load_buf(k + PF < K ? rsrc_src(rpre) : make_rsrc(A.src, 0), cur);
      if constexpr (KF != kNoField) load_kappa<P, KF>(k + PF < K ? rsrc_kap(rpre) : make_rsrc(A.kfield, 0), L, kcur);
      if constexpr (UNI) {
        if (k < KST) drop_row_stores<P, MO ? 3 + PAD : 12>(A);
      }
      T post[9][V], hv[V], jx[V], jy[V];
      if (m.st[0].finish(k, f2, post, hv, jx, jy, C, L, m.bad))
        m.template emitted<0, UNI>(A, C, L, k, m.y0 - HALO + k - 2, post, hv, jx, jy);
      if constexpr (KF != kNoField) {
#pragma unroll
        for (int v = 0; v < V; ++v) m.kring[m.kslot][V * m.lane + v] = k0[v];
        m.kslot = m.kslot + 1 == KQ ? 0 : m.kslot + 1;
      }
      ry = ry + 1 == ny ? 0 : ry + 1;
      rpre = rpre + 1 == ny ? 0 : rpre + 1;
    };
    // groups of U rows, a multiple of PF, so that each buffer keeps its
    // registers around the loop; of three or six (a whole number of turns of the
    // stages' three-row histories), so that those do too.  After KST the
    // compiler is told that every row stores (uniform stores, store_row)
    auto group = [&](auto n, int k) {
#pragma unroll
      for (int i = 0; i < decltype(n)::value; ++i) {
        if (i % PF == 0) iteration(k + i, fa, ka);
        else if (i % PF == 1) iteration(k + i, fb, kb);
        else iteration(k + i, fc, kc);
      }
    };
    using std::integral_constant;
    constexpr int UU = P == kF64 || AV || U < 3 ? U : 3;  // (the general FP32 loop would spill)
    int k = 0;
    for (; k + PF <= K && k < KST; k += PF) group(integral_constant<int, PF>(), k);
    if constexpr (UU > PF && UU % PF == 0) {
      for (; k + UU <= K; k += UU) {
        __builtin_assume(k >= KST);
        group(integral_constant<int, UU>(), k);
      }
    }
    for (; k + PF <= K; k += PF) {
      __builtin_assume(k >= KST);
      group(integral_constant<int, PF>(), k);
    }
    if (PF >= 2 && k < K) iteration(k, fa, ka);
    if (PF == 3 && k + 1 < K) iteration(k + 1, fb, kb);
  };
  if constexpr (P == kF32) {
    if (L.allvec && L.fast_store) run(std::true_type{});
    else run(std::false_type{});
  } else {
    run(std::false_type{});
  }

  const unsigned long long bm = __ballot(m.bad);
  if (bm != 0ull && m.lane == __ffsll((unsigned long long)bm) - 1) atomicOr(A.flag, 1);
}

}  // namespace tflbm
