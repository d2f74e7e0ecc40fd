// pair_kernel.h -- two steps of the flow per launch, for grids whose state
// does not stay in the caches.
#pragma once

#include <type_traits>

#include "step_kernel.h"

namespace lbe {

// Two plain steps in one pass over memory.  One step reads and writes the 27
// values of every site once and is bound by HBM; this kernel reads F_n, keeps
// F_{n+1} on the chip and writes F_{n+2}, so the two steps move the bytes of
// one.
//
// A wave owns kPairCols columns (one lane each, of which the outer four on
// each side only feed the others: a step's cone is two sites wide) and
// marches up a chunk of rows.  It shares no data with other waves: the exchange
// between its lanes goes through its own piece of LDS.  Where a block has more
// than one wave (neighbouring strips) they meet at a barrier once a row, only to
// keep the strips in step.  At row r a wave
//   - forms the moments of row r + 1 of F_n (loaded one iteration earlier),
//   - collides row r of F_n and streams it into LDS,
//   - loads row r + 2,
//   - collects row r - 1 of F_{n+1}, complete now, and its moments,
//   - collides row r - 2 of F_{n+1} and streams it to the other state.
// A chunk works its first and last rows' cones beyond its own rows and stores
// only its own sites.  The site arithmetic is site_moments and site_collide
// of the one-step kernels, and the values kept in LDS are those they store,
// so the states are bitwise the same as after two single steps.
//
// LDS of a wave: the moments of three rows at both times, and of F_{n+1} the
// populations that a later row collects: those moving up of three rows, those
// moving along x of two, those moving down and sideways of one, and those that
// stay in their column (at rest, straight down) of one and of three.  20,008
// bytes in the FP32 form (eight waves a CU, with under 4 KB of its 160 KB
// left), 36,336 in FP64 (four).
using host::kPairHalo;

template <typename S, typename R>
struct PairLds {
  static constexpr int W = 66;   // a column beyond each end, read by lanes whose result is not used
  double c[2][3][W];
  R t[2][3][W], p[2][3][W];
  S up[3][9][W];     // directions 2, 5, 6 of f, g, hbar; row r in slot r mod 3
  S mid[2][6][W];    // directions 1, 3
  S down[6][W];      // directions 7, 8
  // populations that stay in their column: kept here for want of registers
  double g0[64];
  typename RestRaw<rest_fmt<S>(1)>::T h0[64];
  S f0[64], south[3][64];
};
static_assert(8 * sizeof(PairLds<float, float>) <= 160 * 1024);
static_assert(4 * sizeof(PairLds<double, double>) <= 160 * 1024);

// A scalar that the compiler recomputes from: multiples of the plane stride
// kept for a whole loop would take all scalar registers and spill to lanes of
// vector registers, one vector instruction for each use.
__device__ __forceinline__ uint32_t opaque(uint32_t v) {
  asm volatile("" : "+s"(v));
  return v;
}

// orders this wave's LDS accesses (a wave's LDS operations complete in order)
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// A lane or row that has nothing to store carries an offset past the end of
// the buffer, whose stores the hardware drops (the host keeps states below
// host::kPairMaxBytes, so the offset is past the end of any of them).
constexpr uint32_t kDropped = 0xfffffff0u;
static_assert(host::kPairMaxBytes <= kDropped);

// The moment tape of a wave's row (kTape): only its own sites are written.
template <typename R>
struct PairTape {
  __amdgpu_buffer_rsrc_t rd;
  uint32_t n, row, vc, vr;   // sites; first site of the row; lane offsets in the c and R planes
  __device__ __forceinline__ PairTape(void *tape, uint32_t n_, uint32_t row_, int x, bool own)
      : n(n_), row(row_) {
    rd = plane_rsrc(tape, (size_t)n_ * (8 + 4 * sizeof(R)));
    vc = own ? (uint32_t)x * 8u : kDropped;
    vr = own ? (uint32_t)x * (uint32_t)sizeof(R) : kDropped;
  }
  __device__ __forceinline__ void write(double c, R T, R p, R jx, R jy) const {
    constexpr uint32_t E = sizeof(R);
    buf_store<double>(c, rd, vc, row * 8u);
    buf_store<R>(T, rd, vr, n * 8u + row * E);
    buf_store<R>(p, rd, vr, n * (8u + E) + row * E);
    buf_store<R>(jx, rd, vr, n * (8u + 2u * E) + row * E);
    buf_store<R>(jy, rd, vr, n * (8u + 3u * E) + row * E);
  }
};

// F_{n+1} of one row into LDS and registers
template <typename S, typename R, bool EDGE>
struct PairMidSink {
  PairLds<S, R> &l;
  int lane;              // index of the lane's own column in the LDS rows
  int su, sprev, sm;     // slots of this row's and (bottom wall) the row before's up values, of mid
  bool bot, top;
  const PairTape<R> *tp;
  __device__ __forceinline__ void tape(double c, R T, R p, R jx, R jy) const { tp->write(c, T, p, jx, jy); }
  __device__ __forceinline__ static constexpr int up_of(int i) { return i == 2 ? 0 : (i == 5 ? 1 : 2); }
  template <typename V>
  __device__ __forceinline__ void operator()(int i, int lat, V v) const {
    const S s = S(v);
    if (i == 0) {
      l.f0[lane - 1] = s;
    } else if (kEy[i] == 0) {
      l.mid[sm][2 * lat + (i == 1 ? 0 : 1)][lane] = s;
    } else if (kEy[i] > 0) {
      // at the top wall the reflected values take the place of this row's up
      // values, which no row collects
      l.up[su][3 * lat + up_of(i)][lane] = s;
    } else {
      if (EDGE && bot) {
        // reflected: row 0 collects them as if they came up from below
        const int o = kOpp[i];
        l.up[sprev][3 * lat + up_of(o)][lane - kEx[o]] = s;
      } else if (i == 4) {
        l.south[lat][lane - 1] = s;
      } else {
        l.down[2 * lat + (i == 7 ? 0 : 1)][lane] = s;
      }
    }
  }
  __device__ __forceinline__ void rest(double g, double h) const {
    l.g0[lane - 1] = g;
    l.h0[lane - 1] = typename RestRaw<rest_fmt<S>(1)>::T(h);
  }
};

// F_{n+2}: only the wave's own columns and the chunk's own rows are stored.
struct PairOut {
  __amdgpu_buffer_rsrc_t rd;
  uint32_t pb, own, up, down, rb0, rb1;
  uint32_t xo[3], xu[3], xd[3];   // columns x - 1, x, x + 1 in rows j, j + 1, j - 1 (without
                                  // EDGE xo serves all three)
  uint32_t x0, x1;                // rest populations
  bool bot, top;
};
template <typename S, bool STREAM, bool EDGE, bool WALL>
struct PairOutSink {
  const PairOut &o;
  const PairTape<S> *tp;
  __device__ __forceinline__ void tape(double c, S T, S p, S jx, S jy) const { tp->write(c, T, p, jx, jy); }
  template <typename V>
  __device__ __forceinline__ void operator()(int i, int lat, V v) const {
    const bool out = WALL && ((kEy[i] > 0 && o.top) || (kEy[i] < 0 && o.bot));
    const uint32_t row = kEy[i] == 0 ? o.own : (kEy[i] > 0 ? o.up : o.down);
    // planes of direction i: i, 8 + i, 16 + i
    const uint32_t so = (out ? o.own + (uint32_t)kOpp[i] * o.pb : row + (uint32_t)i * o.pb) +
                        (uint32_t)(8 * lat) * o.pb;
    const uint32_t *xs = !EDGE || kEy[i] == 0 ? o.xo : (kEy[i] > 0 ? o.xu : o.xd);
    const uint32_t vo = out ? o.xo[1] : xs[1 + kEx[i]];
    if (STREAM && kEx[i] == 0) buf_store_stream<S>(S(v), o.rd, vo, so);
    else buf_store<S>(S(v), o.rd, vo, so);
  }
  __device__ __forceinline__ void rest(double g, double h) const {
    using T0 = typename RestRaw<rest_fmt<S>(0)>::T;
    using T1 = typename RestRaw<rest_fmt<S>(1)>::T;
    if constexpr (STREAM) {
      buf_store_stream<T0>(T0(g), o.rd, o.x0, o.own + o.rb0);
      buf_store_stream<T1>(T1(h), o.rd, o.x1, o.own + o.rb1);
    } else {
      buf_store<T0>(T0(g), o.rd, o.x0, o.own + o.rb0);
      buf_store<T1>(T1(h), o.rd, o.x1, o.own + o.rb1);
    }
  }
};

template <typename S, typename R, bool DEV, int MODE, int NW>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(sizeof(S) == 8 ? 1 : 2, sizeof(S) == 8 ? 1 : 2)))
pair_step_kernel(const StepArgs a) {
  static_assert((MODE & ~(kStream | kCurv | kDiag | kTape)) == kStore, "pairs of steps");
  constexpr bool STREAM = (MODE & kStream) != 0;
  constexpr int kMode = MODE & ~(kStream | kDiag), kMode1 = MODE & ~kStream;
  __shared__ PairLds<S, R> lds[NW];
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  PairLds<S, R> &l = lds[wave];
  const int nx = a.nx, ny = a.ny;
  const bool walls = a.walls_y != 0;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int ngroups = (a.nstrips + NW - 1) / NW;
  const int strip = (tile % ngroups) * NW + wave, chunk = tile / ngroups;
  if (strip >= a.nstrips) return;
  // strips of equal width, so that no strip is left nearly empty
  const int wx = (nx + a.nstrips - 1) / a.nstrips;
  const int x0 = strip * wx, w = min(wx, nx - x0);
  const int y0 = chunk * a.rows_per_chunk, y1 = min(y0 + a.rows_per_chunk, ny);
  const int lane = threadIdx.x & 63;
  int x = (x0 - kPairHalo + lane) % nx;
  x = x < 0 ? x + nx : x;
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
  // rows of the cones: collisions of F_n in c0..c1, of F_{n+1} in d0..d1,
  // rows of F_{n+1} collected in q0..q1
  const int c0 = walls ? max(y0 - 3, 0) : y0 - 3, c1 = walls ? min(y1 + 2, ny - 1) : y1 + 2;
  const int d0 = walls ? max(y0 - 1, 0) : y0 - 1, d1 = walls ? min(y1, ny - 1) : y1;
  const int q0 = walls && d0 == 0 ? 0 : d0 - 1, q1 = walls && d1 == ny - 1 ? ny - 1 : d1 + 1;
  const int k = lane + 1;   // own column in the LDS rows
  // slots of the rings: row r in slot r mod 3 (rows from c0 - 1 >= -4)
  auto slot = [&](int r) { return (int)((unsigned)(r + 6) % 3u); };
  auto put = [&](int lev, int r, const RowVals<R> &v) {
    double c, T;
    R p;
    site_moments<R, false>(v, a.inv_rcv, &c, &T, &p);
    const int s = slot(r);
    l.c[lev][s][k] = c;
    l.t[lev][s][k] = R(T);
    l.p[lev][s][k] = p;
  };
  // the row beyond a wall: c and p mirrored, T_ghost = 2 T_wall - T
  // (deviations against the reference at the wall)
  auto put_ghost = [&](int lev, int r, int from) {
    const bool bottom = r < 0;
    const double twref = DEV ? a.Ts + (bottom ? 0.0 : a.Tg * double(ny)) : 0.0;
    const R twv = R((bottom ? a.twb : a.twt)[x] - twref);
    const int s = slot(r), f = slot(from);
    l.c[lev][s][k] = l.c[lev][f][k];
    l.p[lev][s][k] = l.p[lev][f][k];
    l.t[lev][s][k] = R(2) * twv - l.t[lev][f][k];
  };
  // the columns that a lane's pushes reach: x - 1, x, x + 1 where they are the
  // strip's own
  uint32_t xs[3];
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    const int o = lane - kPairHalo + e - 1;
    int xx = x + e - 1;
    xx = xx < 0 ? xx + nx : (xx >= nx ? xx - nx : xx);
    xs[e] = o >= 0 && o < w ? (uint32_t)xx * (uint32_t)sizeof(S) : kDropped;
  }
  const bool owned = lane >= kPairHalo && lane < kPairHalo + w;
  // diagnostics (of F_n): of the wave's own sites
  double acc[kNumPartials], own_acc[kNumPartials];
#pragma unroll
  for (int m = 0; m < kNumPartials; ++m) acc[m] = own_acc[m] = 0.0;

  RowVals<R> ra, rb, fa, fb;
  if (!(walls && c0 == 0)) {
    load_row(c0 - 1, rb);
    load_row(c0, ra);
    put(0, c0 - 1, rb);
  } else {
    load_row(c0, ra);
  }
  load_row(c0 + 1, rb);
  put(0, c0, ra);
  if (walls && c0 == 0) put_ghost(0, -1, 0);

  // row r: cur = row r of F_n, nxt = row r + 1 (in flight), f1 = row r - 2 of
  // F_{n+1}, f1n: row r - 1 of it.  Without EDGE every row involved exists, no
  // wall is touched and the three rows stored to are the chunk's own.
  auto iteration = [&](auto edge, int r, RowVals<R> &cur, RowVals<R> &nxt, RowVals<R> &f1,
                       RowVals<R> &f1n) __attribute__((always_inline)) {
    constexpr bool EDGE = decltype(edge)::value;
    if (NW > 1) __builtin_amdgcn_s_barrier();
    // row r - 1's values of F_{n+1} that row r's take the place of
    f1n.v[0] = R(l.f0[lane]);
    f1n.g0r = l.g0[lane];
    f1n.h0r = l.h0[lane];
    if (!EDGE || r <= c1) {
      if (EDGE && walls && r + 1 == ny) put_ghost(0, ny, ny - 1);
      else put(0, r + 1, nxt);
      wave_lds_fence();
      const int sS = slot(r - 1), sC = slot(r), sN = slot(r + 1);
      const PairTape<R> tape(a.tape, (uint32_t)n, (uint32_t)(wrap_row(r) * nx), x,
                             owned && r >= y0 && r < y1);
      const bool bot = EDGE && walls && r == 0, top = EDGE && walls && r == ny - 1;
      site_collide<R, DEV, kMode1, EDGE>(
          a, wrap_row(r), x, bot, top, &l.c[0][sS][lane], &l.c[0][sC][lane], &l.c[0][sN][lane],
          &l.t[0][sS][lane], &l.t[0][sC][lane], &l.t[0][sN][lane], &l.p[0][sS][lane],
          &l.p[0][sC][lane], &l.p[0][sN][lane], cur, acc,
          PairMidSink<S, R, EDGE>{l, k, sC, sS, r & 1, bot, top, &tape});
      if constexpr ((MODE & kDiag) != 0) {
#pragma unroll
        for (int m = 0; m < kNumPartials; ++m) {
          if (owned && r >= y0 && r < y1) own_acc[m] += acc[m];
          acc[m] = 0.0;
        }
      }
      if (!EDGE || (r + 2 <= c1 + 1 && !(walls && r + 2 >= ny))) load_row(r + 2, cur);
    }
    __builtin_amdgcn_sched_barrier(0);
    const int q = r - 1;
    if (!EDGE || (q >= q0 && q <= q1)) {
      wave_lds_fence();
      const int su = slot(q - 1), sm = q & 1;
      const bool refl = EDGE && walls && q == ny - 1;   // the top wall's reflected values
      const int sr = slot(q);
#pragma unroll
      for (int lat = 0; lat < 3; ++lat) {
        const int o = 9 * lat;
        f1n.v[o + 2] = R(l.up[su][3 * lat][k]);
        f1n.v[o + 5] = R(l.up[su][3 * lat + 1][k - 1]);
        f1n.v[o + 6] = R(l.up[su][3 * lat + 2][k + 1]);
        f1n.v[o + 1] = R(l.mid[sm][2 * lat][k - 1]);
        f1n.v[o + 3] = R(l.mid[sm][2 * lat + 1][k + 1]);
        if (refl) {
          f1n.v[o + 4] = R(l.up[sr][3 * lat][k]);
          f1n.v[o + 7] = R(l.up[sr][3 * lat + 1][k]);
          f1n.v[o + 8] = R(l.up[sr][3 * lat + 2][k]);
        } else {
          f1n.v[o + 4] = R(l.south[lat][lane]);
          f1n.v[o + 7] = R(l.down[2 * lat][k + 1]);
          f1n.v[o + 8] = R(l.down[2 * lat + 1][k - 1]);
        }
      }
      put(1, q, f1n);
      if (EDGE && walls && q == 0) put_ghost(1, -1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    const int j = r - 2;
    if (!EDGE || (j >= d0 && j <= d1)) {
      if (EDGE && walls && j == ny - 1) put_ghost(1, ny, ny - 1);
      wave_lds_fence();
      const int sS = slot(j - 1), sC = slot(j), sN = slot(j + 1);
      const bool bot = EDGE && walls && j == 0, top = EDGE && walls && j == ny - 1;
      const int jw = EDGE ? wrap_row(j) : j;
      const PairTape<R> tape(a.tape2, (uint32_t)n, (uint32_t)(jw * nx), x,
                             owned && j >= y0 && j < y1);
      PairOut out;
      out.rd = plane_rsrc(a.dst, state_bytes_for<S>(n));
      out.pb = opaque(pb);
      out.own = (uint32_t)jw * RB;
      if constexpr (EDGE) {
        const bool okO = j >= y0 && j < y1, okU = j + 1 >= y0 && j + 1 < y1,
                   okD = j - 1 >= y0 && j - 1 < y1;
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
      } else {
        out.up = out.own + RB;
        out.down = out.own - RB;
#pragma unroll
        for (int e = 0; e < 3; ++e) out.xo[e] = xs[e];
        out.x0 = owned ? vx0 : kDropped;
        out.x1 = owned ? vx1 : kDropped;
      }
      out.rb0 = rb0;
      out.rb1 = rb1;
      out.bot = bot;
      out.top = top;
      site_collide<R, DEV, kMode, EDGE>(
          a, jw, x, bot, top, &l.c[1][sS][lane], &l.c[1][sC][lane], &l.c[1][sN][lane],
          &l.t[1][sS][lane], &l.t[1][sC][lane], &l.t[1][sN][lane], &l.p[1][sS][lane],
          &l.p[1][sC][lane], &l.p[1][sN][lane], f1, acc,
          PairOutSink<S, STREAM, EDGE, EDGE>{out, &tape});
    }
  };
  // two rows per turn, so that the rows in registers change roles by name;
  // the turns that stay clear of walls and of the chunk's ends take the short
  // form
  const int last = d1 + 2, i0 = y0 + 3, i1 = min(y1, ny - 3);
  int r = c0;
#pragma nounroll
  for (int part = 0; part < 2; ++part) {
    const int end = part == 0 ? min(i0 - 1, last) : last;
#pragma nounroll
    for (; r <= end; ++r) {
      iteration(std::true_type{}, r, ra, rb, fa, fb);
      const RowVals<R> t0 = ra, t1 = fa;
      ra = rb;
      rb = t0;
      fa = fb;
      fb = t1;
    }
#pragma nounroll
    for (; r >= i0 && r + 1 <= i1; r += 2) {
      iteration(std::false_type{}, r, ra, rb, fa, fb);
      iteration(std::false_type{}, r + 1, rb, ra, fb, fa);
    }
  }
  if constexpr ((MODE & kDiag) != 0) {
    // one partial per wave, a fixed butterfly over its lanes
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

// ---------------------------------------------------------------------------
// Two plain steps in one launch on latency-bound grids.  A step of such a grid
// is one pass of latency (launch, loads, moments, collision, stores: 5-6 us)
// whatever its size, and most of the chip idles; here one pass takes two
// steps, at the price of colliding the margin of each tile again.  A block
// holds the rows of a tile and four more on each side, one wave a row: as in
// pair_step_kernel a wave's outer four columns on each side only feed the
// others.  Moments, collision of F_n into LDS, moments of F_{n+1}, collision
// into the other state, with a block barrier in between.  Diagnostics (of
// F_n) may come along.  The states are bitwise those of two single steps.
template <typename S, typename R, int TY>
struct PairTileLds {
  static constexpr int H = TY + 2 * kPairHalo, W = 66;
  double c[H][W];
  R t[H][W], p[H][W];
  S f[24][TY + 6][W];   // moving populations of F_{n+1}, rows 2 .. H - 3 of the block (from 1 on), and
                        // one row on each side for pushes that no row collects
  double red[H][kNumPartials];
};

// F_{n+1} of the tile: pushes into LDS; the rest populations stay with the wave
template <typename S, typename R, int TY, bool WALL>
struct PairTileSink {
  PairTileLds<S, R, TY> &l;
  int k, row;            // own column in the LDS rows, row of the block
  bool bot, top;
  RowVals<R> &f1;        // receives the rest populations
  const PairTape<R> *tp;
  __device__ __forceinline__ void tape(double c, R T, R p, R jx, R jy) const { tp->write(c, T, p, jx, jy); }
  template <typename V>
  __device__ __forceinline__ void operator()(int i, int lat, V v) const {
    if (i == 0) {
      f1.v[0] = R(S(v));
      return;
    }
    const bool out = WALL && ((kEy[i] > 0 && top) || (kEy[i] < 0 && bot));
    const int to = max(0, min(TY + 5, row - 1 + (out ? 0 : kEy[i])));
    const int d = out ? kOpp[i] : i;
    l.f[8 * lat + d - 1][to][out ? k : k + kEx[i]] = S(v);
  }
  __device__ __forceinline__ void rest(double g, double h) const {
    f1.g0r = g;
    f1.h0r = typename RestRaw<rest_fmt<S>(1)>::T(h);
  }
};

template <typename S, typename R, bool DEV, int MODE, int TY>
__global__ void __launch_bounds__(64 * (TY + 2 * kPairHalo))
pair_tile_kernel(const StepArgs a) {
  static_assert((MODE & ~(kCurv | kDiag | kTape)) == kStore, "pairs of steps");
  constexpr int H = TY + 2 * kPairHalo;
  constexpr int kMode = MODE & ~kDiag;
  __shared__ PairTileLds<S, R, TY> l;
  const int nx = a.nx, ny = a.ny;
  const bool walls = a.walls_y != 0;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int wx = (nx + a.nstrips - 1) / a.nstrips;
  const int x0 = (tile % a.nstrips) * wx, w = min(wx, nx - x0);
  const int y0 = (tile / a.nstrips) * TY, y1 = min(y0 + TY, ny);
  const int lane = threadIdx.x & 63, k = lane + 1;
  const int row = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  int x = (x0 - kPairHalo + lane) % nx;
  x = x < 0 ? x + nx : x;
  const int r = y0 - kPairHalo + row;   // this wave's row, beyond y0 - 1 and y1 a cone's
  const bool live = r < y1 + kPairHalo && !(walls && (r < 0 || r >= ny));
  int jr = r % ny;
  jr = jr < 0 ? jr + ny : jr;
  const bool bot = walls && r == 0, top = walls && r == ny - 1;
  const bool owned = lane >= kPairHalo && lane < kPairHalo + w && r >= y0 && r < y1;
  const size_t n = (size_t)nx * (size_t)ny;
  const uint32_t pb = (uint32_t)(nx * sizeof(S));
  const uint32_t RB = (uint32_t)row_bytes<S>(nx);
  const uint32_t rb0 = (uint32_t)rest_base<S>(0, nx), rb1 = (uint32_t)rest_base<S>(1, nx);
  using T0 = typename RestRaw<rest_fmt<S>(0)>::T;
  using T1 = typename RestRaw<rest_fmt<S>(1)>::T;
  // moments of the wave's row, and of the row beyond a wall (c and p mirrored,
  // T_ghost = 2 T_wall - T, deviations against the reference at the wall)
  auto put = [&](const RowVals<R> &v) {
    double c, T;
    R p;
    site_moments<R, false>(v, a.inv_rcv, &c, &T, &p);
    l.c[row][k] = c;
    l.t[row][k] = R(T);
    l.p[row][k] = p;
    if (bot || top) {
      const int g = bot ? row - 1 : row + 1;
      if (g >= 0 && g < H) {
        const double twref = DEV ? a.Ts + (bot ? 0.0 : a.Tg * double(ny)) : 0.0;
        const R twv = R((bot ? a.twb : a.twt)[x] - twref);
        l.c[g][k] = c;
        l.t[g][k] = R(2) * twv - R(T);
        l.p[g][k] = p;
      }
    }
  };
  RowVals<R> cur;
  double acc[kNumPartials];
#pragma unroll
  for (int m = 0; m < kNumPartials; ++m) acc[m] = 0.0;
  if (live) {
    const __amdgpu_buffer_rsrc_t rsrc = plane_rsrc(a.src, state_bytes_for<S>(n));
    const uint32_t vx = (uint32_t)x * (uint32_t)sizeof(S), ro = (uint32_t)jr * RB;
#pragma unroll
    for (int q = 0; q < 27; ++q)
      if (q != 9 && q != 18) cur.v[q] = R(buf_load<S>(rsrc, vx, ro + (uint32_t)plane_of(q) * pb));
    cur.g0r = buf_load<T0>(rsrc, (uint32_t)x * (uint32_t)sizeof(T0), ro + rb0);
    cur.h0r = buf_load<T1>(rsrc, (uint32_t)x * (uint32_t)sizeof(T1), ro + rb1);
    if (sizeof(S) == 4) touch_args(a);   // FP32 3.78 -> 3.53 us a step on 40 x 100; FP64 no gain
    put(cur);
  }
  // FP32: a wave takes the form with walls only where its own row touches one
  // (in FP64 the two forms together spill registers)
  auto collide = [&](auto mode, auto wall, auto &&sink) __attribute__((always_inline)) {
    site_collide<R, DEV, decltype(mode)::value, decltype(wall)::value>(
        a, jr, x, bot, top, &l.c[row - 1][lane], &l.c[row][lane], &l.c[row + 1][lane],
        &l.t[row - 1][lane], &l.t[row][lane], &l.t[row + 1][lane], &l.p[row - 1][lane],
        &l.p[row][lane], &l.p[row + 1][lane], cur, acc, sink);
  };
  __syncthreads();
  if (live && row >= 1 && row < H - 1) {
    RowVals<R> f1;
    const PairTape<R> tape(a.tape, (uint32_t)n, (uint32_t)(jr * nx), x, owned);
    constexpr std::integral_constant<int, MODE> mode{};
    if (sizeof(S) == 8 || bot || top)
      collide(mode, std::true_type{}, PairTileSink<S, R, TY, true>{l, k, row, bot, top, f1, &tape});
    else
      collide(mode, std::false_type{}, PairTileSink<S, R, TY, false>{l, k, row, bot, top, f1, &tape});
    cur.v[0] = f1.v[0];
    cur.g0r = f1.g0r;
    cur.h0r = f1.h0r;
  }
  if constexpr ((MODE & kDiag) != 0) {
#pragma unroll
    for (int m = 0; m < kNumPartials; ++m)
      if (!owned) acc[m] = 0.0;
    block_partials<H>(acc, l.red, threadIdx.x, a.partials + (size_t)blockIdx.x * kNumPartials);
  }
  __syncthreads();
  if (live && row >= 2 && row < H - 2) {
#pragma unroll
    for (int q = 1; q < 27; ++q)
      if (q % 9 != 0) cur.v[q] = R(l.f[8 * (q / 9) + q % 9 - 1][row - 1][k]);
    put(cur);
  }
  __syncthreads();
  if (live && row >= 3 && row < H - 3) {
    PairOut out;
    out.rd = plane_rsrc(a.dst, state_bytes_for<S>(n));
    out.pb = pb;
    out.own = (uint32_t)jr * RB;
    out.up = jr + 1 == ny ? 0u : out.own + RB;
    out.down = (jr == 0 ? (uint32_t)ny : (uint32_t)jr) * RB - RB;
    out.rb0 = rb0;
    out.rb1 = rb1;
    out.bot = bot;
    out.top = top;
    const bool okO = r >= y0 && r < y1, okU = r + 1 >= y0 && r + 1 < y1,
               okD = r - 1 >= y0 && r - 1 < y1;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      const int o = lane - kPairHalo + e - 1;
      int xx = x + e - 1;
      xx = xx < 0 ? xx + nx : (xx >= nx ? xx - nx : xx);
      const uint32_t xs = o >= 0 && o < w ? (uint32_t)xx * (uint32_t)sizeof(S) : kDropped;
      out.xo[e] = okO ? xs : kDropped;
      out.xu[e] = okU ? xs : kDropped;
      out.xd[e] = okD ? xs : kDropped;
    }
    out.x0 = owned ? (uint32_t)x * (uint32_t)sizeof(T0) : kDropped;
    out.x1 = owned ? (uint32_t)x * (uint32_t)sizeof(T1) : kDropped;
    const PairTape<R> tape(a.tape2, (uint32_t)n, (uint32_t)(jr * nx), x, owned);
    constexpr std::integral_constant<int, kMode> mode{};
    if (sizeof(S) == 8 || bot || top)
      collide(mode, std::true_type{}, PairOutSink<S, false, true, true>{out, &tape});
    else
      collide(mode, std::false_type{}, PairOutSink<S, false, true, false>{out, &tape});
  }
}

}  // namespace lbe
