// Host-side geometry and cost model of the block kernels' tiles (block.h,
// adj_block.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tflbm {

struct BlockShape {
  int r, nw;  // rows per wavefront, wavefronts per workgroup
};

// Whether the n tile rows from r0 on, of `rows` in use, hold a row whose
// pressure (reverse: lambda_p) the stored rows still depend on in step s of a pass.
__host__ __device__ __forceinline__ bool block_active(int r0, int n, int rows, int s) {
  return r0 + n > 3 * s + 1 && r0 < rows - 3 * s - 1;
}

// Tiles of a pass of ns steps: 64 columns and r nw rows less three of each per
// step and side, and `extra` columns per side.
struct Tiles {
  int halo, halo_x, bw, bh, ntx, ntiles, per_xcd;
  unsigned inv_ntx;  // 2^32 / ntx rounded down, at most 2^32 - 1
  bool fits;         // the tile has an output worth launching for
  Tiles(int nx, int ny, const BlockShape &sh, int ns, int extra = 0) {
    halo = 3 * ns;
    halo_x = halo + extra;
    bw = 64 - 2 * halo_x;
    bh = sh.r * sh.nw - 2 * halo;
    fits = bw >= 8 && bh >= 2;
    if (!fits) return;
    ntx = (nx + bw - 1) / bw;
    const int64_t n = (int64_t)ntx * ((ny + bh - 1) / bh);
    fits = n < (1 << 30);
    ntiles = (int)n;
    per_xcd = (ntiles + 7) / 8;
    inv_ntx = ntx == 1 ? 0xffffffffu : (unsigned)(((uint64_t)1 << 32) / (unsigned)ntx);
  }
};

// Time of a pass of ns steps, in microseconds:
//   launch + step ns + load (row_load rows + row_step active row steps + step_load ns),
// with the rows of one workgroup and `load` the workgroups per CU (256 CUs),
// rounded up to whole ones as far as `whole` says (a CU is busy until its last
// one ends).  march0..2: time of one step of the marching kernels over n strip
// rows, march0 + march1 min(n, 2500) + march2 max(n - 2500, 0).
struct TileModel {
  double launch, step, row_load, row_step, step_load, whole, march0, march1, march2;
  double pass(const Tiles &t, const BlockShape &sh, int ns) const {
    int row_steps = 0;
    for (int k = 0; k < ns; ++k) row_steps += sh.r * (sh.nw - 2 * ((3 * k + 1) / sh.r));  // wavefronts with block_active
    const double per_cu = t.ntiles / 256.0, up = (double)(int64_t)(per_cu + 0.999999);
    const double load = per_cu <= 1.0 ? 1.0 : per_cu + whole * (up - per_cu);
    return launch + step * ns + load * (row_load * sh.r * sh.nw + row_step * row_steps + step_load * ns);
  }
  // k passes of nearly equal length over n steps, the longer ones first
  double call(int nx, int ny, const BlockShape &sh, int extra, int64_t n, int64_t k) const {
    const int q = (int)(n / k);
    const int64_t longer = n % k;
    const Tiles t(nx, ny, sh, q, extra);
    double us = (double)(k - longer) * pass(t, sh, q);
    if (longer > 0) us += (double)longer * pass(Tiles(nx, ny, sh, q + 1, extra), sh, q + 1);
    return us;
  }
  double march(double n, double slope) const { return march0 + march1 * (n < 2500 ? n : 2500) + slope * (n < 2500 ? 0 : n - 2500); }
};

// A block plan: index of the shape and most steps per pass (0: no plan).
struct BlockPlan {
  int shape = 0, ns = 0;
  bool always = false;  // also for calls whose passes are single steps
  double limit = 0.0;   // modelled time per step from which on a call stays with the marching kernels
};

// The shape and steps per pass (two or more) of the least modelled time per step, of n
// shapes, and that time; TFLBM_<name> and TFLBM_<name>_SHAPE (`env`, `env_shape`) force
// both, one step too.
// best.ns = 0 where no shape serves or TFLBM_<name>=0.
double best_plan(const TileModel &m, const BlockShape *shapes, int n, int nx, int ny, int extra,
                 const char *env, const char *env_shape, BlockPlan &best);

}  // namespace tflbm
