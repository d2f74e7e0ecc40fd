// density_kernel.h -- one step with two densities in one pass over memory.
#pragma once

#include "pair_kernel.h"

namespace lbe {

// With two densities the pressure of Eq. 9 needs u, hence the force, at every
// site of its stencil.  As two launches (the pressure into a plane, then the
// step) every site is read twice; here the pressure of a row follows its
// moments by one row and the collision follows by another, all in LDS.  As in
// pair_step_kernel a wave marches a strip by itself, here with three columns
// (kDensityHalo) on each side that only feed the others, and stores only its
// own sites.  At row r it loads row r + 2, forms the moments of row r + 1, the
// pressure of row r and the collision of row r - 1; the loads come before the
// collision's stores, which they would otherwise wait for.  Four rows stay in
// registers, so a CU holds four waves.  The arithmetic is that of the two
// launches (site_moments, site_collide with kPress and with kStore), so the
// states are bitwise the same.
using host::kDensityHalo;

template <typename R>
struct DensityLds {
  static constexpr int W = 66;
  double c[4][W];
  R t[4][W], p[4][W];   // row r in slot r mod 4; p is the pressure of Eq. 9
  R sf[W];              // sum f of the row whose pressure is formed
};

template <typename R>
struct PressureSink {
  R &p;
  template <typename V>
  __device__ __forceinline__ void operator()(int, int, V) const {}
  __device__ __forceinline__ void rest(double, double) const {}
  __device__ __forceinline__ void pressure(double v) const { p = R(v); }
};

template <typename S, typename R, bool DEV, int MODE, int NW>
__global__ void __launch_bounds__(64 * NW)
__attribute__((amdgpu_waves_per_eu(1, 1)))
density_step_kernel(const StepArgs a) {
  static_assert((MODE & ~(kCurv | kDiag)) == (kStore | kVarRho), "steps with two densities");
  __shared__ DensityLds<R> lds[NW];
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  DensityLds<R> &l = lds[wave];
  const int nx = a.nx, ny = a.ny;
  const bool walls = a.walls_y != 0;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int ngroups = (a.nstrips + NW - 1) / NW;
  const int strip = (tile % ngroups) * NW + wave, chunk = tile / ngroups;
  if (strip >= a.nstrips) return;
  const int wx = (nx + a.nstrips - 1) / a.nstrips;
  const int x0 = strip * wx, w = min(wx, nx - x0);
  const int y0 = chunk * a.rows_per_chunk, y1 = min(y0 + a.rows_per_chunk, ny);
  const int lane = threadIdx.x & 63, k = lane + 1;
  int x = (x0 - kDensityHalo + lane) % nx;
  x = x < 0 ? x + nx : x;
  const bool owned = lane >= kDensityHalo && lane < kDensityHalo + w;
  const size_t n = (size_t)nx * (size_t)ny;
  const __amdgpu_buffer_rsrc_t rsrc = plane_rsrc(a.src, state_bytes_for<S>(n));
  const uint32_t pb = (uint32_t)(nx * sizeof(S));
  const uint32_t RB = (uint32_t)row_bytes<S>(nx);
  const uint32_t rb0 = (uint32_t)rest_base<S>(0, nx), rb1 = (uint32_t)rest_base<S>(1, nx);
  using T0 = typename RestRaw<rest_fmt<S>(0)>::T;
  using T1 = typename RestRaw<rest_fmt<S>(1)>::T;
  const uint32_t vx = (uint32_t)x * (uint32_t)sizeof(S);
  const uint32_t vx0 = (uint32_t)x * (uint32_t)sizeof(T0), vx1 = (uint32_t)x * (uint32_t)sizeof(T1);
  auto wrap_row = [&](int r) { return r < 0 ? r + ny : (r >= ny ? r - ny : r); };
  auto load_row = [&](int row, RowVals<R> &v) {
    const uint32_t step = opaque(pb);
    uint32_t so = (uint32_t)wrap_row(row) * RB;
#pragma unroll
    for (int q = 0; q < 27; ++q)
      if (q != 9 && q != 18) {
        v.v[q] = R(buf_load<S>(rsrc, vx, so));
        so += step;
      }
    v.g0r = buf_load<T0>(rsrc, vx0, so);   // the rest populations follow the 25 planes
    v.h0r = buf_load<T1>(rsrc, vx1, so + (uint32_t)(sizeof(T0) / sizeof(S)) * step);
  };
  // rows of the cones: collisions d0..d1, pressures p0..p1, moments one beyond
  const int d0 = walls ? max(y0 - 1, 0) : y0 - 1, d1 = walls ? min(y1, ny - 1) : y1;
  const int p0 = walls ? max(d0 - 1, 0) : d0 - 1, p1 = walls ? min(d1 + 1, ny - 1) : d1 + 1;
  auto slot = [](int r) { return r & 3; };
  auto put = [&](int r, const RowVals<R> &v) {
    const double tref = DEV ? a.Ts + a.Tg * (double(wrap_row(r)) + 0.5) : 0.0;
    double c, T;
    R p;
    site_moments<R, true>(v, a.inv_rcv, &c, &T, &p, a.rho, a.drho, a.cv, tref);
    l.c[slot(r)][k] = c;
    l.t[slot(r)][k] = R(T);
  };
  // the row beyond a wall: c and p mirrored, T_ghost = 2 T_wall - T
  auto put_ghost = [&](int r, int from) {
    const bool bottom = r < 0;
    const double twref = DEV ? a.Ts + (bottom ? 0.0 : a.Tg * double(ny)) : 0.0;
    const R twv = R((bottom ? a.twb : a.twt)[x] - twref);
    l.c[slot(r)][k] = l.c[slot(from)][k];
    l.t[slot(r)][k] = R(2) * twv - l.t[slot(from)][k];
  };
  uint32_t xs[3];
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    const int o = lane - kDensityHalo + e - 1;
    int xx = x + e - 1;
    xx = xx < 0 ? xx + nx : (xx >= nx ? xx - nx : xx);
    xs[e] = o >= 0 && o < w ? (uint32_t)xx * (uint32_t)sizeof(S) : kDropped;
  }
  double acc[kNumPartials], own_acc[kNumPartials];
#pragma unroll
  for (int m = 0; m < kNumPartials; ++m) acc[m] = own_acc[m] = 0.0;

  RowVals<R> ra, rb, rc, rd;
  if (!(walls && p0 == 0)) {
    load_row(p0 - 1, rd);
    load_row(p0, rb);
    load_row(p0 + 1, rc);
    put(p0 - 1, rd);
    put(p0, rb);
  } else {
    load_row(0, rb);
    load_row(1, rc);
    put(0, rb);
    put_ghost(-1, 0);
  }
  // A = row r - 1, B = row r, C = row r + 1 (in flight), D: row r + 2
  auto iteration = [&](int r, RowVals<R> &A, RowVals<R> &B, RowVals<R> &C,
                       RowVals<R> &D) __attribute__((always_inline)) {
    if (NW > 1) __builtin_amdgcn_s_barrier();   // neighbouring strips in step
    if (r + 2 <= p1 + 1 && !(walls && r + 2 >= ny)) load_row(r + 2, D);
    if (r <= p1) {
      if (walls && r + 1 == ny) put_ghost(ny, ny - 1);
      else put(r + 1, C);
      R f = 0;
#pragma unroll
      for (int q = 0; q < 9; ++q) f += B.v[q];
      l.sf[k] = f;
      wave_lds_fence();
      const int sS = slot(r - 1), sC = slot(r), sN = slot(r + 1);
      R p = 0;
      site_collide<R, DEV, kVarRho | kPress | (MODE & kCurv), false>(
          a, wrap_row(r), x, false, false, &l.c[sS][lane], &l.c[sC][lane], &l.c[sN][lane],
          &l.t[sS][lane], &l.t[sC][lane], &l.t[sN][lane], &l.sf[lane], &l.sf[lane], &l.sf[lane], B,
          acc, PressureSink<R>{p});
      l.p[sC][k] = p;
      if (walls && r == 0) l.p[sS][k] = p;
      if (walls && r == ny - 1) l.p[sN][k] = p;
    }
    __builtin_amdgcn_sched_barrier(0);
    const int j = r - 1;
    if (j >= d0 && j <= d1) {
      wave_lds_fence();
      const int sS = slot(j - 1), sC = slot(j), sN = slot(j + 1);
      const bool bot = walls && j == 0, top = walls && j == ny - 1;
      const int jw = wrap_row(j);
      const bool okO = j >= y0 && j < y1, okU = j + 1 >= y0 && j + 1 < y1,
                 okD = j - 1 >= y0 && j - 1 < y1;
      PairOut out;
      out.rd = plane_rsrc(a.dst, state_bytes_for<S>(n));
      out.pb = opaque(pb);
      out.own = (uint32_t)jw * RB;
      out.up = top ? 0u : (uint32_t)wrap_row(j + 1) * RB;   // top, bot: not addressed
      out.down = bot ? 0u : (uint32_t)wrap_row(j - 1) * RB;
#pragma unroll
      for (int e = 0; e < 3; ++e) {
        out.xo[e] = okO ? xs[e] : kDropped;
        out.xu[e] = okU ? xs[e] : kDropped;
        out.xd[e] = okD ? xs[e] : kDropped;
      }
      out.x0 = okO && owned ? vx0 : kDropped;
      out.x1 = okO && owned ? vx1 : kDropped;
      out.rb0 = rb0;
      out.rb1 = rb1;
      out.bot = bot;
      out.top = top;
      site_collide<R, DEV, MODE, true>(
          a, jw, x, bot, top, &l.c[sS][lane], &l.c[sC][lane], &l.c[sN][lane], &l.t[sS][lane],
          &l.t[sC][lane], &l.t[sN][lane], &l.p[sS][lane], &l.p[sC][lane], &l.p[sN][lane], A, acc,
          PairOutSink<S, false, true, true>{out, nullptr});
      if constexpr ((MODE & kDiag) != 0) {
#pragma unroll
        for (int m = 0; m < kNumPartials; ++m) {
          if (owned && okO) own_acc[m] += acc[m];
          acc[m] = 0.0;
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // four rows per turn, so that the rows in registers change roles by name
#pragma nounroll
  for (int r = p0; r <= d1 + 1; r += 4) {
    iteration(r, ra, rb, rc, rd);
    iteration(r + 1, rb, rc, rd, ra);
    iteration(r + 2, rc, rd, ra, rb);
    iteration(r + 3, rd, ra, rb, rc);
  }
  if constexpr ((MODE & kDiag) != 0) {
    double *out = a.partials + (size_t)(chunk * a.nstrips + strip) * kNumPartials;
#pragma unroll
    for (int m = 0; m < kNumPartials; ++m) {
      double v = own_acc[m];
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
      if (lane == 0) out[m] = v;
    }
  }
}

}  // namespace lbe
