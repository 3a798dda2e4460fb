// D2Q9 sweeps of large grids without temperature: waves that march along y.
//
// The tile kernels spend 183 vector instructions per node and step (half of
// them on the halo, on addresses and on LDS) and wait at three barriers per
// tile. Here every wave owns a strip of 64 columns, one per lane, and a chunk
// of rows, and walks up its rows one at a time: a row's neighbours below and
// above are in registers, its neighbours left and right one lane away (DPP
// moves), so there is no LDS and no barrier, and 86 instructions remain (92 in
// the adjoint). K steps are taken in one walk, each step two rows behind the
// one before, which divides the traffic by K; the 2K outer lanes of a strip and
// 2K rows at the ends of a chunk are the redundant work. Bound by the length
// of a wave's walk (one or two waves per SIMD): 2048 x 2048, us per step
// (forward, adjoint): FP32 31.5, 31.1 -> 16.9, 19.2; FP64 52.5, 64 -> 30.5, 37.
//
// The per-node functions are those of the tile kernels (lks_node.h), with the
// same operands in the same order, so the results have the same bits.
#include <algorithm>
#include <type_traits>

#include "lks_node.h"

namespace lks {
namespace {

// value of the lane to the right or left (0 at the end of the wave)
constexpr int RIGHT = 0x130, LEFT = 0x138;  // DPP wave_shl:1, wave_shr:1
template <int C>
__device__ inline float lane(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), C, 0xf, 0xf, true));
}
template <int C>
__device__ inline double lane(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), C, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), C, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// strip and chunk of a wave
struct Strip {
  int i, ic;       // column of this lane, clamped to the grid
  int y0, y1, Y0;  // rows stored, first row read
  int nx, ny;
  int ex;          // end kind of the column
  bool xe;         // the strip holds an end column (wave-uniform)
  bool own;        // the lane stores its column
};

// element `col` of a row that starts at `row` (uniform base, 32-bit byte offset)
template <typename T>
__device__ inline T& at(T* p, size_t row, int col) {
  using C = std::conditional_t<std::is_const_v<T>, const char, char>;
  return *reinterpret_cast<T*>(reinterpret_cast<C*>(p + row) + unsigned(col) * unsigned(sizeof(T)));
}

// The waves of a launch of up to k steps: ntx strips, consecutive ones
// overlapping by the 4k lanes that only feed others, cut into nty chunks of rows,
// the strips at the ends of x into nte; the chunks at the ends of y are `pad`
// rows shorter. The strips at the ends of x form more values and choose among
// them, and the chunks at the ends of y push some rows one by one: with the same
// rows as the others they end a launch late (2048 x 2048 FP32 adjoint: 31 us per
// step instead of 19), so they get a third of the rows and 24 rows less.
struct MarchShape {
  int k, ntx, nty, nte, pad;
  __host__ __device__ int waves() const { return max(ntx - 2, 0) * nty + min(ntx, 2) * nte; }
};
__host__ __device__ inline MarchShape march_shape(int nx, int ny, int k, int nty) {
  const int most = max(ny / 8, 1), w = 64 - 4 * k;
  MarchShape ms;
  ms.k = k;
  ms.ntx = nx <= 64 ? 1 : (nx - 4 * k + w - 1) / w;
  ms.nty = max(1, min(nty, most));
  ms.nte = min(3 * ms.nty, most);
  ms.pad = max(0, min(24, ny / ms.nte - 8));
  return ms;
}

template <int K>
__device__ inline Strip strip_of(const Geo& g, int t, const MarchShape& ms) {
  Strip c;
  const int mid = max(ms.ntx - 2, 0), nin = mid * ms.nty, nend = min(ms.ntx, 2);
  const bool in = t < nin;
  const int q = in ? t : t - nin, per = in ? mid : nend, n = in ? ms.nty : ms.nte;
  const int by = q / per, bx = in ? 1 + q % per : (q % per) * (ms.ntx - 1);
  const int l = int(threadIdx.x) & 63, h = 2 * ms.k;
  auto row = [&](int b) {
    const int y = int((long long)b * (g.ny + 2 * ms.pad) / n) - ms.pad;
    return b == n ? g.ny : min(max(y, 0), g.ny);
  };
  c.nx = g.nx;
  c.ny = g.ny;
  c.i = bx * (64 - 2 * h) + l;
  c.ic = min(c.i, g.nx - 1);
  c.y0 = row(by);
  c.y1 = row(by + 1);
  c.Y0 = max(c.y0 - 2 * K, 0);
  c.ex = end_of(c.i, g.nx, 0);
  c.xe = bx == 0 || bx == ms.ntx - 1;
  c.own = c.i < g.nx && (bx == 0 || l >= h) && (bx == ms.ntx - 1 || l < 64 - h);
  return c;
}
// index of this wave among `total`, or -1
__device__ inline int march_wave(int total) {
  const int b = xcd_tile((total + 3) / 4);
  if (b < 0) return -1;
  const int t = __builtin_amdgcn_readfirstlane(4 * b + (int(threadIdx.x) >> 6));
  return t < total ? t : -1;
}

// How much of the boundary a push has to handle: nothing, the columns at the
// ends of x, or also the first and last rows (with the rows' bookkeeping as
// loops and branches, after which a wave waits for all its loads and stores:
// 1.5 us a row instead of 0.5)
enum { INNER = 0, XENDS = 1, ANY = 2 };

// x difference of a value held by the lanes
template <int MODE, typename R>
__device__ inline R lane_dx(const Strip& c, R f0) {
  const R r = lane<RIGHT>(f0), l = lane<LEFT>(f0);
  if constexpr (MODE == INNER) return R(0.5) * (r - l);
  const R r2 = lane<RIGHT>(r), l2 = lane<LEFT>(l);
  return end_f(f0, c.ex < 0 ? l : r, c.ex == 0 ? l : (c.ex > 0 ? r2 : l2), c.ex);
}
// y difference from three rows in ascending order, the node's own among them:
// the middle one (e = 0), the lowest (1) or the highest (-1)
template <int MODE, typename R>
__device__ inline R row_dy(R x0, R x1, R x2, int e) {
  if constexpr (MODE != ANY) return R(0.5) * (x2 - x0);
  return end_f(e == 0 ? x1 : (e > 0 ? x0 : x2), e == 0 ? x2 : x1, e > 0 ? x2 : x0, e);
}

// ---------------------------------------------------------------------------
// LKS steps
// ---------------------------------------------------------------------------
// A step's rows: state of the last three rows pushed (2 the newest), the
// populations that have arrived at the row to be put out and those on their
// way to the row above it, and the coefficients of the row to be put out.
template <typename R>
struct FwdLevel {
  R d[3], u[3], v[3];
  R f0, f1, f3, f2, f5, f6, n2, n5, n6;
  R s, bx, by, last;
  int m;
};
template <typename R, int K>
struct FwdMarch {
  const FwdArgs<R>& a;
  const Geo& g;
  Strip c;
  R A;
  double fac[K];  // inflow factor of the level each step writes
};

// coefficients of row y
template <int MODE, typename R, int K>
__device__ inline void fwd_fetch(const FwdMarch<R, K>& w, FwdLevel<R>& l, int y) {
  const size_t row = size_t(max(min(y, w.c.ny - 1), 0)) * w.c.nx;
  l.s = at(w.a.inv1pa, row, w.c.ic);
  if constexpr (MODE != INNER) {
    l.m = at(w.a.mask, row, w.c.ic);
    l.bx = at(w.a.ubx, row, w.c.ic);
    l.by = at(w.a.uby, row, w.c.ic);
  }
}

// Row j of the level before step LV arrives (j >= ny: nothing arrives, but
// the step goes on with the rows it holds). Then the post-collision values of
// row j - 1 are formed and row j - 2 of the new level is put out. A chunk at
// the bottom forms row 0 together with row 1 (its differences need row 2). The
// first rows put out by a chunk that starts higher up are formed from rows
// that were not read; they reach none that is stored.
template <int MODE, typename R, int K, int LV>
__device__ __forceinline__ void fwd_push(const FwdMarch<R, K>& w, FwdLevel<R>* L, int j, R d, R u,
                                         R v) {
  const Strip& c = w.c;
  FwdLevel<R>& l = L[LV];
  if (MODE != ANY || j < c.ny) {
    l.d[0] = l.d[1];
    l.u[0] = l.u[1];
    l.v[0] = l.v[1];
    l.d[1] = l.d[2];
    l.u[1] = l.u[2];
    l.v[1] = l.v[2];
    l.d[2] = d;
    l.u[2] = u;
    l.v[2] = v;
  }
  auto row = [&](int r) {  // post-collision values of row r, row r - 1 out
    R f[9], s4 = R(0), s7 = R(0), s8 = R(0);
    const bool there = MODE != ANY || r < c.ny;
    if (there) {
      R d0 = l.d[1], u0 = l.u[1], v0 = l.v[1];
      int e = 0;
      if (MODE == ANY && r == 0) {
        e = 1;
        // a corner has the density of its y-neighbour
        d0 = LV && c.ex ? l.d[1] : l.d[0];
        u0 = l.u[0];
        v0 = l.v[0];
      } else if (MODE == ANY && r == c.ny - 1) {
        e = -1;
        d0 = l.d[2];
        u0 = l.u[2];
        v0 = l.v[2];
      }
      fwd_post(w.A, d0, u0, v0, lane_dx<MODE>(c, u0), row_dy<MODE>(l.u[0], l.u[1], l.u[2], e),
               lane_dx<MODE>(c, v0), row_dy<MODE>(l.v[0], l.v[1], l.v[2], e),
               [&](int q, R x) { f[q] = x; });
      s4 = f[4];
      s7 = lane<RIGHT>(f[7]);
      s8 = lane<LEFT>(f[8]);
    }
    const int y = r - 1;
    if (MODE != ANY || y >= 0) {
      const R q[9] = {l.f0, l.f1, l.f2, l.f3, s4, l.f5, l.f6, s7, s8};
      const R z[9] = {};
      const bool ye = MODE == ANY && (y == 0 || y == c.ny - 1);
      R dn, un, vn, Tn;
      fwd_interior<R, false>(w.g, q, z, l.s, false, R(0), dn, un, vn, Tn);
      if constexpr (MODE != INNER) {
        if (ye || c.ex) {
          const int o = c.ex ? (c.ex > 0 ? 0 : 1) : (y == 0 ? 2 : 3);
          const R S0 = q[0] + (o < 2 ? q[2] : q[1]) + (o < 2 ? q[4] : q[3]);
          const R p2 = o == 0 ? q[3] : (o == 1 ? q[1] : (o == 2 ? q[4] : q[2]));
          const R p3 = o == 0 ? q[6] : (o == 2 ? q[7] : q[5]);
          const R p4 = o == 0 ? q[7] : (o == 3 ? q[6] : q[8]);
          const R Sp = p2 + p3 + p4;
          const double fac = (l.m & 3) == FLOW_VELOCITY ? w.fac[LV] : 0.0;
          fwd_ring<R, false>(
              w.g, S0, Sp, R(0), R(0), o, l.m, [&](int x) { return x ? l.by : l.bx; },
              [&]() { return fac; }, [&]() { return R(0); }, dn, un, vn, Tn);
          if (ye && c.ex) {
            un = vn = R(0);
            dn = l.last;  // (of row 0: taken from row 1 later)
          }
        }
        l.last = dn;
      }
      fwd_fetch<MODE>(w, l, y + 1);
      if constexpr (LV < K - 1) {
        fwd_push<MODE, R, K, LV + 1>(w, L, y, dn, un, vn);
      } else if (y >= c.y0 && y < c.y1 && c.own) {
        const size_t o = size_t(y) * c.nx;
        at(w.a.d1, o, c.i) = dn;
        at(w.a.ux1, o, c.i) = un;
        at(w.a.uy1, o, c.i) = vn;
        if (MODE == ANY && y == 1 && c.ex) w.a.d1[c.i] = dn;  // the corner below
      }
    }
    l.f2 = l.n2;
    l.f5 = l.n5;
    l.f6 = l.n6;
    if (there) {
      l.f0 = f[0];
      l.f1 = lane<LEFT>(f[1]);
      l.f3 = lane<RIGHT>(f[3]);
      l.n2 = f[2];
      l.n5 = lane<LEFT>(f[5]);
      l.n6 = lane<RIGHT>(f[6]);
    }
  };
  if constexpr (MODE != ANY) {
    row(j - 1);
  } else {
    if (j < 2) return;
    for (int r = j == 2 ? 0 : j - 1; r < j; ++r) row(r);
  }
}

// The rows of a wave: those whose pushes meet the first or last row of the grid
// apart from the others. read(x, j) reads row j into slot x, push(mode, x, j)
// pushes it, next() renames slots 1, 2 to 0, 1. Rows are read two ahead, and
// three are pushed per turn of the loop, after which every value is back in its
// register: a move of a value in flight would wait for it.
template <int K, typename F, typename P, typename N>
__device__ __forceinline__ void march_chunk(const Strip& c, F&& read, P&& push, N&& next) {
  const int end = c.y1 + 2 * K;
  read(0, c.Y0);
  read(1, c.Y0 + 1);
  int j = c.Y0;
  auto any = [&](int to) {
#pragma nounroll
    for (; j < to; ++j) {
      read(2, j + 2);
      push(std::integral_constant<int, ANY>(), 0, j);
      next();
    }
  };
  // (a turn may go past the end of a chunk: what it puts out is not stored)
  auto turns = [&](auto mode) {
    const bool top = end > c.ny;
    const int n = (top ? c.ny - j : end - j + 2) / 3;
#pragma nounroll
    for (int t = 0; t < n; ++t, j += 3) {
      read(2, j + 2);
      push(mode, 0, j);
      read(0, j + 3);
      push(mode, 1, j + 1);
      read(1, j + 4);
      push(mode, 2, j + 2);
    }
  };
  if (j == 0) any(min(2 * K + 3, end));
  if (c.xe) turns(std::integral_constant<int, XENDS>());
  else turns(std::integral_constant<int, INNER>());
  any(end);
}

template <typename R, int K>
__device__ __forceinline__ void march_fwd(const Geo& g, const FwdArgs<R>& a, int t,
                                          const MarchShape& ms) {
  FwdMarch<R, K> w{a, g, strip_of<K>(g, t, ms), R(g.A)};
  const Strip& c = w.c;
  FwdLevel<R> L[K] = {};
#pragma unroll
  for (int s = 0; s < K; ++s) {
    w.fac[s] = a.ufac[min(a.level_mid + s, a.level_out)];
    fwd_fetch<ANY>(w, L[s], c.Y0 - 2 * s - 1);
  }
  R d[3], u[3], v[3];
  auto read = [&](int x, int j) {
    const size_t row = size_t(min(j, c.ny - 1)) * c.nx;
    d[x] = at(a.d0, row, c.ic);
    u[x] = at(a.ux0, row, c.ic);
    v[x] = at(a.uy0, row, c.ic);
  };
  march_chunk<K>(
      c, read,
      [&](auto mode, int x, int j) {
        fwd_push<decltype(mode)::value, R, K, 0>(w, L, j, d[x], u[x], v[x]);
      },
      [&]() {
        for (int x = 0; x < 2; ++x) {
          d[x] = d[x + 1];
          u[x] = u[x + 1];
          v[x] = v[x + 1];
        }
      });
}

// ---------------------------------------------------------------------------
// ALKS steps
// ---------------------------------------------------------------------------
// A step's rows: what the next two rows of moments pull from the rows below
// (a: the row under the next one, b: the next one itself), the moments rho~,
// U~, s~ of the last three rows (2 the newest), and the coefficients of the
// row to be put out.
template <typename R>
struct AdjLevel {
  R e0, e1, e3, a4, a7, a8, b4, b7, b8;
  R M[3][6];
  R s, ux, uy;
  int m;  // class of the next row of moments
};
template <typename R>
struct AdjMarch {
  const AdjArgs<R>& a;
  const Geo& g;
  Strip c;
};

template <typename R>
__device__ inline void adj_fetch(const AdjMarch<R>& w, AdjLevel<R>& l, int y) {
  const size_t row = size_t(max(min(y, w.c.ny - 1), 0)) * w.c.nx;
  l.s = at(w.a.inv1pa, row, w.c.ic);
  l.ux = at(w.a.ux, row, w.c.ic);
  l.uy = at(w.a.uy, row, w.c.ic);
}
template <int MODE, typename R>
__device__ inline void adj_fetch_class(const AdjMarch<R>& w, AdjLevel<R>& l, int y) {
  if constexpr (MODE != INNER)
    l.m = at(w.a.mask, size_t(max(min(y, w.c.ny - 1), 0)) * w.c.nx, w.c.ic);
}

// Row j of the level after the step arrives; the moments of row j - 1 are
// formed and row j - 2 of the new level is put out. A chunk at the bottom puts
// out row 0 together with row 1.
template <int MODE, typename R, int K, int LV>
__device__ __forceinline__ void adj_push(const AdjMarch<R>& w, AdjLevel<R>* L, int j, R r_, R vx,
                                         R vy) {
  const Strip& c = w.c;
  AdjLevel<R>& l = L[LV];
  const R xp = r_ + vx, xm = r_ - vx;
  const R s5 = lane<RIGHT>(xp + vy), s6 = lane<LEFT>(xm + vy);
  const int r = j - 1;  // row of moments
  if (MODE != ANY || (r >= 0 && r < c.ny)) {
    const R E[9] = {l.e0, l.e1, r_ + vy, l.e3, l.a4, s5, s6, l.a7, l.a8};
    const R z[9] = {};
    R mom[9];
    adj_mom<R, false>(E, z, mom);
    if constexpr (MODE != INNER) {
      const bool ye = MODE == ANY && (r == 0 || r == c.ny - 1);
      if (ye) adj_fetch_class<MODE>(w, l, r);  // (INNER pushes fetch none)
      if (ye || c.ex) {
        const int o = c.ex ? (c.ex > 0 ? 0 : 1) : (r == 0 ? 2 : 3);
        const R f[6] = {E[0],
                        o == 0 ? E[4] : (o == 1 ? E[2] : (o == 2 ? E[1] : E[3])),
                        o == 0 ? E[2] : (o == 1 ? E[4] : (o == 2 ? E[3] : E[1])),
                        o == 0 ? E[1] : (o == 1 ? E[3] : (o == 2 ? E[2] : E[4])),
                        o == 0 ? E[8] : (o == 1 ? E[6] : (o == 2 ? E[5] : E[7])),
                        o == 0 ? E[5] : (o == 1 ? E[7] : (o == 2 ? E[6] : E[8]))};
        ring_fill<R, false>(w.a, o, l.m, R(0), R(0), R(0), f, z, mom);
      }
      if constexpr (MODE == ANY) {
        // corners take the moments of their y-neighbour
#pragma unroll
        for (int x = 0; x < 6; ++x) {
          if (r == 1 && c.ex) l.M[2][x] = mom[x];
          if (r == c.ny - 1 && c.ex) mom[x] = l.M[2][x];
        }
      }
    }
#pragma unroll
    for (int x = 0; x < 6; ++x) {
      l.M[0][x] = l.M[1][x];
      l.M[1][x] = l.M[2][x];
      l.M[2][x] = mom[x];
    }
    adj_fetch_class<MODE>(w, l, r + 1);
  }
  l.a4 = l.b4;
  l.a7 = l.b7;
  l.a8 = l.b8;
  l.b4 = r_ - vy;
  l.b7 = lane<LEFT>(xm - vy);
  l.b8 = lane<RIGHT>(xp - vy);
  l.e0 = r_;
  l.e1 = lane<RIGHT>(xp);
  l.e3 = lane<LEFT>(xm);
  auto row = [&](int y) {
    R mom[9] = {l.M[1][0], l.M[1][1], l.M[1][2], l.M[1][3], l.M[1][4],
                l.M[1][5], R(0),      R(0),      R(0)};
    int e = 0;
    if (MODE == ANY && y == 0) {
      e = 1;
#pragma unroll
      for (int x = 0; x < 6; ++x) mom[x] = l.M[0][x];
    } else if (MODE == ANY && y == c.ny - 1) {
      e = -1;
#pragma unroll
      for (int x = 0; x < 6; ++x) mom[x] = l.M[2][x];
    }
    AdjNode<R> nd = {};
    nd.s = l.s;
    nd.ux = l.ux;
    nd.uy = l.uy;
    const R dsx =
        add2(lane_dx<MODE>(c, mom[3]), row_dy<MODE>(l.M[0][4], l.M[1][4], l.M[2][4], e));
    const R dsy =
        add2(lane_dx<MODE>(c, mom[4]), row_dy<MODE>(l.M[0][5], l.M[1][5], l.M[2][5], e));
    R rn, vxn, vyn, th;
    double pair, adj_T;
    adj_node<R, false>(w.g, w.a, nd, mom, dsx, dsy, R(0), rn, vxn, vyn, th, pair, adj_T);
    adj_fetch(w, l, y + 1);
    if constexpr (LV < K - 1) {
      adj_push<MODE, R, K, LV + 1>(w, L, y, rn, vxn, vyn);
    } else if (y >= c.y0 && y < c.y1 && c.own) {
      const size_t o = size_t(y) * c.nx;
      at(w.a.r1, o, c.i) = rn;
      at(w.a.vx1, o, c.i) = vxn;
      at(w.a.vy1, o, c.i) = vyn;
      if (w.a.sens_mode) {  // the last launch of a sweep
        const bool ring = y == 0 || y == c.ny - 1 || c.ex;
        const R dA3 = at(w.a.dA3, o, c.i);
        at(w.a.sens, o, c.i) =
            ring ? 0.0
                 : adj_sens<R, false>(w.a, pair, adj_T, dA3, R(0), R(0), R(0), R(0), R(0), R(0),
                                      R(0));
      }
    }
  };
  if constexpr (MODE != ANY) {
    row(j - 2);
  } else {
    if (j < 3) return;
    for (int y = j == 3 ? 0 : j - 2; y < j - 1; ++y) row(y);
  }
}

template <typename R, int K>
__device__ __forceinline__ void march_adj(const Geo& g, const AdjArgs<R>& a, int t,
                                          const MarchShape& ms) {
  AdjMarch<R> w{a, g, strip_of<K>(g, t, ms)};
  const Strip& c = w.c;
  AdjLevel<R> L[K] = {};
#pragma unroll
  for (int s = 0; s < K; ++s) {
    adj_fetch(w, L[s], c.Y0 - 2 * s - 2);
    adj_fetch_class<ANY>(w, L[s], c.Y0 - 2 * s - 1);
  }
  R r[3], vx[3], vy[3];
  auto read = [&](int x, int j) {
    const size_t row = size_t(min(j, c.ny - 1)) * c.nx;
    r[x] = at(a.r0, row, c.ic);
    vx[x] = at(a.vx0, row, c.ic);
    vy[x] = at(a.vy0, row, c.ic);
  };
  march_chunk<K>(
      c, read,
      [&](auto mode, int x, int j) {
        adj_push<decltype(mode)::value, R, K, 0>(w, L, j, r[x], vx[x], vy[x]);
      },
      [&]() {
        for (int x = 0; x < 2; ++x) {
          r[x] = r[x + 1];
          vx[x] = vx[x + 1];
          vy[x] = vy[x + 1];
        }
      });
}

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------
template <typename R, int K>
__global__ __launch_bounds__(256) void lks_march_kernel(Geo g, FwdArgs<R> a, MarchShape ms) {
  const int t = march_wave(ms.waves());
  if (t < 0) return;
  march_fwd<R, K>(g, a, t, ms);
}
template <typename R, int K>
__global__ __launch_bounds__(256) void alks_march_kernel(Geo g, AdjArgs<R> a, MarchShape ms) {
  const int t = march_wave(ms.waves());
  if (t < 0) return;
  march_adj<R, K>(g, a, t, ms);
}

// chunks of about `rows` rows of a design of a batch
__host__ __device__ inline MarchShape batch_shape(const Geo& g, int k, int rows) {
  return march_shape(g.nx, g.ny, k, (g.ny + rows - 1) / rows);
}
// batches: tmap holds the design and the wave within it; k is the step count of
// the plan, whose waves a launch of K <= k steps takes
template <typename R, int K>
__global__ __launch_bounds__(256) void lks_march_batch_kernel(const BatchFwd<R>* __restrict__ d,
                                                              const int* __restrict__ tmap,
                                                              int total, int k, int rows,
                                                              int parity) {
  const int t = march_wave(total);
  if (t < 0) return;
  const int di = tmap[2 * t];
  const Geo g = d[di].g;
  FwdArgs<R> a = d[di].a[parity];
  a.level_mid = a.level_out;
  march_fwd<R, K>(g, a, tmap[2 * t + 1], batch_shape(g, k, rows));
}
template <typename R, int K>
__global__ __launch_bounds__(256) void alks_march_batch_kernel(const BatchAdj<R>* __restrict__ d,
                                                               const int* __restrict__ tmap,
                                                               int total, int k, int rows,
                                                               int parity, int last) {
  const int t = march_wave(total);
  if (t < 0) return;
  const int di = tmap[2 * t];
  const Geo g = d[di].g;
  AdjArgs<R> a = d[di].a[parity];
  a.sens_mode = last ? 2 : 0;
  march_adj<R, K>(g, a, tmap[2 * t + 1], batch_shape(g, k, rows));
}

// Waves of a launch: one per SIMD (of 1024) in FP64 and two in FP32, what the registers of
// three and two steps allow. A second round of waves costs more than it hides
// (2048 x 2048 FP32 adjoint, 8 % over one round: 31 instead of 19 us).
constexpr int round_waves(int rsz) { return (rsz == 8 ? 1024 : 2048) - 8; }

// f(K) for the launch of `steps` steps
template <int RSZ, typename F>
void with_steps(int steps, F&& f) {
  if (steps == 1) f(std::integral_constant<int, 1>());
  else if (steps == 2) f(std::integral_constant<int, 2>());
  else if constexpr (RSZ == 8) f(std::integral_constant<int, 3>());
}
template <int RSZ>
MarchShape shape_for(const Geo& g, int k) {
  const int ntx = march_shape(g.nx, g.ny, k, 1).ntx;
  return march_shape(g.nx, g.ny, k,
                     round_waves(RSZ) / (std::max(ntx - 2, 0) + 3 * std::min(ntx, 2)));
}
unsigned blocks_of(int waves) { return unsigned(xcd_blocks((waves + 3) / 4)); }

}  // namespace

// The march needs one round of waves whose chunks are well over 4K rows tall.
// us per step, tile or several-steps kernels -> march (forward, adjoint): FP32
// 1024 x 1024 10.4, 11.6 -> 10.2, 12.4; 1500 x 1400 18.3, 19.2 -> 12.3, 14.2; 3001 x
// 2003 41.8, 42.3 -> 21.8, 24.2; FP64 1024 x 768 11.1, 13.4 -> 10.2, 14.9; 1024 x 1024
// 14.3, 17.3 -> 11.6, 15.1; 3001 x 2003 83, 90 -> 45, 49. Three steps where the fields
// of an FP64 sweep outgrow the 256 MB of the last cache (2048 x 2048 36.6, 43.1 with
// two, 30.5, 37.6 with three; 1500 x 1400 16.3, 20.1 and 17.3, 22.8); FP32 2048 x 2048
// 16.9, 19.2 with two, 17.0, 31.8 with three, whose rows take all registers.
MultiPlan march_plan(const Geo& g, int rsz) {
  MultiPlan p;
  if (g.thermal || g.periodic || std::min(g.nx, g.ny) < 128) return p;
  if (g.N < (rsz == 8 ? 1 << 20 : 1250000)) return p;
  p.k = rsz == 8 && g.N >= 3000000 ? 3 : 2;
  p.variant = MARCH;
  return p;
}

int march_waves(const Geo& g, int k, int rows) { return batch_shape(g, k, rows).waves(); }

// Batches: the same lines on the nodes of all designs, in the shortest chunks
// of which all waves fit one round. us per step of all designs, several-steps
// kernels -> march (forward, adjoint): FP32 32 designs of 128 to 512, 3.2M nodes, 43.9,
// 38.3 -> 27.8, 25.1; 256 of 128 x 128 89.8, 56.3 -> 75.8, 55.9; 10 of 380 x 380 21.0,
// 18.5 -> 14.8, 16.0. In FP64 half the waves share the work and the rows at the
// ends of a small design outweigh the others: 64 of 256 x 256 75, 64 -> 108, 111, 16 of
// 512 x 512 68, 62 -> 62, 65, 2 of 900 x 900 26.4, 23.5 -> 17.8, 19.4, so only large
// designs march.
BatchPlan march_batch_plan(const Geo* const* g, int n, int rsz) {
  BatchPlan p;
  long long N = 0;
  for (int d = 0; d < n; ++d) {
    if (g[d]->thermal || g[d]->periodic) return p;
    N += g[d]->N;
  }
  if (N < (rsz == 8 ? std::max(1LL << 20, 750000LL * n) : 1250000)) return p;
  const int k = rsz == 8 && N >= 3000000 ? 3 : 2;
  for (int rows = 8; rows <= (1 << 14); rows += std::max(1, rows / 32)) {
    long long waves = 0;
    for (int d = 0; d < n; ++d) waves += march_waves(*g[d], k, rows);
    if (waves > round_waves(rsz)) continue;
    p.tile = rows;
    p.kf = p.ka = k;
    p.vf = p.va = MARCH;
    break;
  }
  return p;
}

template <typename R>
void launch_lks_march(const Geo& g, int steps, const FwdArgs<R>& a, hipStream_t s) {
  with_steps<sizeof(R)>(steps, [&](auto k) {
    const MarchShape ms = shape_for<sizeof(R)>(g, k.value);
    lks_march_kernel<R, decltype(k)::value><<<blocks_of(ms.waves()), 256, 0, s>>>(g, a, ms);
  });
}
template <typename R>
void launch_alks_march(const Geo& g, int steps, const AdjArgs<R>& a, hipStream_t s) {
  with_steps<sizeof(R)>(steps, [&](auto k) {
    const MarchShape ms = shape_for<sizeof(R)>(g, k.value);
    alks_march_kernel<R, decltype(k)::value><<<blocks_of(ms.waves()), 256, 0, s>>>(g, a, ms);
  });
}
template <typename R>
void launch_lks_march_batch(const BatchFwd<R>* d, const int* tmap, int total, const BatchPlan& p,
                            int steps, int parity, hipStream_t s) {
  with_steps<sizeof(R)>(steps, [&](auto k) {
    lks_march_batch_kernel<R, decltype(k)::value>
        <<<blocks_of(total), 256, 0, s>>>(d, tmap, total, p.kf, p.tile, parity);
  });
}
template <typename R>
void launch_alks_march_batch(const BatchAdj<R>* d, const int* tmap, int total, const BatchPlan& p,
                             int steps, int parity, int last, hipStream_t s) {
  with_steps<sizeof(R)>(steps, [&](auto k) {
    alks_march_batch_kernel<R, decltype(k)::value>
        <<<blocks_of(total), 256, 0, s>>>(d, tmap, total, p.ka, p.tile, parity, last);
  });
}

#define LKS_MARCH_INSTANTIATE(R)                                                              \
  template void launch_lks_march<R>(const Geo&, int, const FwdArgs<R>&, hipStream_t);         \
  template void launch_alks_march<R>(const Geo&, int, const AdjArgs<R>&, hipStream_t);        \
  template void launch_lks_march_batch<R>(const BatchFwd<R>*, const int*, int,                \
                                          const BatchPlan&, int, int, hipStream_t);           \
  template void launch_alks_march_batch<R>(const BatchAdj<R>*, const int*, int,               \
                                           const BatchPlan&, int, int, int, hipStream_t);
LKS_MARCH_INSTANTIATE(float)
LKS_MARCH_INSTANTIATE(double)

}  // namespace lks
