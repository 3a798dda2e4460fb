// D2Q9 sweeps of small grids: several LKS or ALKS steps per kernel launch.
//
// A dependent chain of launches costs about 2.7 us per launch on an MI355X
// however little each does, and on a grid that does not fill the 256 CUs the
// rest of a step is the length of one block's chain (load, LDS stages,
// store), not work. These kernels cut the grid into about one tile per CU, of
// any width and height, load a tile with a halo of two nodes per step, and
// run k steps on the shrinking region: two LDS stages per step and no global
// round trip between them. Every thread owns the same one or two nodes of
// the region through the launch, so a node's own values stay in registers,
// its LDS positions are formed once, and only what neighbours read goes
// through LDS. The off-ring part of a region is a rectangle and is dealt to
// the first waves; its ring nodes get waves of their own, so that no wave runs
// both rules. The redundant work of the halo is the price: MultiPlan weighs
// it against the launches saved.
//
// The per-node functions are those of the tile kernels (lks_node.h), so k
// steps here give the bits of k one-step launches.
#include <algorithm>
#include <type_traits>

#include "lks_node.h"

namespace lks {
namespace {

// the nodes of this thread in the region of its tile
struct MultiTile {
  int x0, x1, y0, y1;  // tile
  int X0, Y0, W, H;    // region: tile + 2k, clipped to a bounded domain
  int tile;
};

__device__ inline void multi_tile(const Geo& g, const MultiShape& ms, int tile, MultiTile& t) {
  t.tile = tile;
  const int bx = t.tile % ms.ntx, by = t.tile / ms.ntx;
  t.x0 = int((long long)bx * g.nx / ms.ntx);
  t.x1 = int((long long)(bx + 1) * g.nx / ms.ntx);
  t.y0 = int((long long)by * g.ny / ms.nty);
  t.y1 = int((long long)(by + 1) * g.ny / ms.nty);
  const int h = 2 * ms.k;
  t.X0 = t.x0 - h;
  t.Y0 = t.y0 - h;
  int X1 = t.x1 + h, Y1 = t.y1 + h;
  if (!g.periodic) {
    t.X0 = max(t.X0, 0);
    t.Y0 = max(t.Y0, 0);
    X1 = min(X1, g.nx);
    Y1 = min(Y1, g.ny);
  }
  t.W = X1 - t.X0;
  t.H = Y1 - t.Y0;
}

// A register value the compiler takes as new here: what is derived from it (LDS
// and field addresses of a node) is formed where it is used, instead of being
// kept in registers through all steps (which spilled 60 to 80 of them).
// Only where registers are short: with two nodes per thread of 1024.
template <int NT, int NPT>
__device__ inline int here(int p) {
  if constexpr (NT * NPT > 1024) asm volatile("" : "+v"(p));
  return p;
}

// one node of a thread: its index k, its position p in the region (pitch W)
// and its packed description c, three registers in all
struct MultiNode {
  int k, p, c;
  // how far outside the tile the node lies (0: in the tile)
  __device__ int ext() const { return c & 255; }
  __device__ bool ring() const { return c & 0x100; }
  __device__ bool corner() const { return c & 0x200; }
  __device__ int side() const { return (c >> 10) & 3; }
  __device__ int ex() const { return ((c >> 12) & 3) - 1; }  // end kinds (ring nodes)
  __device__ int ey() const { return ((c >> 14) & 3) - 1; }
  // index of the corner this node is, or (feeds) is the y-neighbour of
  __device__ bool feeds(int top) const { return (c >> (16 + top)) & 1; }
  __device__ int corner_at(int top) const { return (side() & 1) + 2 * top; }
  __device__ int corner_of() const { return (ex() < 0 ? 1 : 0) + (ey() < 0 ? 2 : 0); }
};
constexpr int NO_NODE = 255;  // ext of a slot without a node

// node of slot e of this thread: the off-ring rectangle row by row over the
// slots, then, from a wave of its own and in the last slot of the threads, the
// ring nodes
template <int NT, int NPT>
__device__ inline MultiNode multi_node(const Geo& g, const MultiTile& t, int e) {
  const int q = int(threadIdx.x) + e * NT;
  int rx0 = t.X0, ry0 = t.Y0, wi = t.W, hi = t.H;
  if (!g.periodic) {
    rx0 = max(t.X0, 1);
    ry0 = max(t.Y0, 1);
    wi = min(t.X0 + t.W, g.nx - 1) - rx0;
    hi = min(t.Y0 + t.H, g.ny - 1) - ry0;
  }
  const int nint = wi * hi;
  int i = 0, j = 0, c = NO_NODE;
  if (q < nint) {
    const int ly = q / wi;
    i = rx0 + q - ly * wi;
    j = ry0 + ly;
    c = 0;
  } else if (!g.periodic && e == NPT - 1) {
    RingSet s;
    const int nr = ring_set(g, t.X0, t.Y0, t.W, t.H, s);
    const int r = q - max((nint + 63) & ~63, NT * (NPT - 1));
    if (r >= 0 && r < nr) {
      ring_at(g, s, r, &i, &j);
      const bool xe = i == 0 || i == g.nx - 1, ye = j == 0 || j == g.ny - 1;
      c = 0x100 | (xe && ye ? 0x200 : 0) | (ring_side(g, i, j) << 10) |
          ((end_of(i, g.nx, 0) + 1) << 12) | ((end_of(j, g.ny, 0) + 1) << 14);
      if (xe && j == 1) c |= 1 << 16;
      if (xe && j == g.ny - 2) c |= 1 << 17;
    }
  }
  MultiNode n;
  n.p = 0;
  if (c != NO_NODE) {
    c |= max(max(max(t.x0 - i, i - t.x1 + 1), max(t.y0 - j, j - t.y1 + 1)), 0);
    n.p = (j - t.Y0) * t.W + i - t.X0;
  }
  if (g.periodic) {
    i %= g.nx;
    j %= g.ny;
    i = i < 0 ? i + g.nx : i;
    j = j < 0 ? j + g.ny : j;
  }
  n.k = j * g.nx + i;
  n.c = c;
  return n;
}

// ---------------------------------------------------------------------------
// LKS steps
// ---------------------------------------------------------------------------
// LDS per node: u (, T) for the differences and the eight moving values f'_q
// (, g_q) for the pull. Levels a launch passes through go to lv.f[s] where
// wanted (the last one always); their objective terms are summed per wave and
// level and added to the tile's accumulator in level order, so the sum does
// not depend on how a sweep is cut into launches.
// (lv(st, out) gives the pointers of step st)
template <typename R, bool TH, int NT, int NPT, int NMAX, typename Out>
__device__ __forceinline__ void multi_fwd(const Geo& g, const FwdArgs<R>& a, const MultiShape& ms,
                                          int tile, Out&& lv) {
  constexpr int LU = 0, LV = 1, LT = 2, LF = TH ? 3 : 2, LG = LF + 8, NA = TH ? 19 : 10;
  __shared__ R L[NA][NMAX];
  __shared__ double red[MULTI_STEPS][NT / 64];
  __shared__ R cd[4];  // new density of the corners (by their y-neighbours)
  MultiTile t;
  multi_tile(g, ms, tile, t);
  const int W = t.W, tid = int(threadIdx.x);
  const R A = R(g.A);
  MultiNode n[NPT];
  R d[NPT], u[NPT], v[NPT], T[NPT], s[NPT], B[NPT], be[NPT], f0[NPT], g0[NPT];
  R ubx[NPT], uby[NPT], Tb[NPT];
  int m[NPT];
#pragma unroll
  for (int e = 0; e < NPT; ++e) {
    n[e] = multi_node<NT, NPT>(g, t, e);
    d[e] = u[e] = v[e] = T[e] = s[e] = B[e] = be[e] = f0[e] = g0[e] = R(0);
    ubx[e] = uby[e] = Tb[e] = R(0);
    m[e] = 0;
    if (n[e].ext() == NO_NODE) continue;
    const int k = here<NT, NPT>(n[e].k);
    d[e] = a.d0[k];
    u[e] = a.ux0[k];
    v[e] = a.uy0[k];
    s[e] = a.inv1pa[k];
    m[e] = a.mask[k];
    if constexpr (TH) {
      T[e] = a.T0[k];
      B[e] = a.B[k];
      if (a.beta) be[e] = a.beta[k];
      if (n[e].ring()) Tb[e] = a.Tb[k];
    }
    if (n[e].ring()) {
      ubx[e] = a.ubx[k];
      uby[e] = a.uby[k];
    }
  }
#pragma unroll
  for (int e = 0; e < NPT; ++e) {
    if (n[e].ext() == NO_NODE) continue;
    L[LU][n[e].p] = u[e];
    L[LV][n[e].p] = v[e];
    if constexpr (TH) L[LT][n[e].p] = T[e];
  }
  for (int st = 0; st < ms.k; ++st) {
    const int reach = 2 * (ms.k - st) - 1;  // the post-collision values are needed this far out
    const int level = min(a.level_mid + st, a.level_out);
    // (scalar loads share their wait with LDS reads: fetched before the stages)
    R* out[4];
    lv(st, out);
    lds_barrier();
#pragma unroll
    for (int e = 0; e < NPT; ++e) {
      if (n[e].ext() > reach) continue;
      const bool RING_SLOT = e == NPT - 1;  // (known once the loop is unrolled)
      const int p = here<NT, NPT>(n[e].p);
      if (RING_SLOT && n[e].corner() && st) {  // the y-neighbour completed the corner's last step
        d[e] = cd[n[e].corner_of()];
        u[e] = v[e] = R(0);
        if constexpr (TH) T[e] = L[TH ? LT : 0][p];
      }
      auto collide = [&](auto ring) {
        constexpr bool RING = decltype(ring)::value;
        auto dx = [&](int f) { return end_d(L[f], p, 1, RING ? n[e].ex() : 0); };
        auto dy = [&](int f) { return end_d(L[f], p, W, RING ? n[e].ey() : 0); };
        R f[9];
        fwd_post(A, d[e], u[e], v[e], dx(LU), dy(LU), dx(LV), dy(LV),
                 [&](int q, R x) { f[q] = x; });
        f0[e] = f[0];
#pragma unroll
        for (int q = 1; q < 9; ++q) L[LF + q - 1][p] = f[q];
        if constexpr (TH) {
          R Wx, Wy;
          fwd_flux(T[e], B[e], u[e], v[e], dx(TH ? LT : 0), dy(TH ? LT : 0), Wx, Wy);
          g0[e] = g_eq<R>(0, T[e], Wx, Wy);
#pragma unroll
          for (int q = 1; q < 9; ++q) L[TH ? LG + q - 1 : 0][p] = g_eq<R>(q, T[e], Wx, Wy);
        }
      };
      if (RING_SLOT && n[e].ring()) collide(std::true_type());
      else collide(std::false_type());
    }
    lds_barrier();
    double part = 0.0;
    const bool keep = out[1] != nullptr;
#pragma unroll
    for (int e = 0; e < NPT; ++e) {
      const bool RING_SLOT = e == NPT - 1;
      if (n[e].ext() > reach - 1 || (RING_SLOT && n[e].corner())) continue;
      const int p = here<NT, NPT>(n[e].p), k = here<NT, NPT>(n[e].k);
      R f[9], gg[9], dn, un, vn, Tn = R(0);
      f[0] = f0[e];
      gg[0] = g0[e];
      if (!(RING_SLOT && n[e].ring())) {
#pragma unroll
        for (int q = 1; q < 9; ++q) {
          const int o = p - CX[q] - CY[q] * W;
          f[q] = L[LF + q - 1][o];
          if constexpr (TH) gg[q] = L[TH ? LG + q - 1 : 0][o];
        }
        fwd_interior<R, TH>(g, f, gg, s[e], TH && a.beta, be[e], dn, un, vn, Tn);
      } else {
        const int o = n[e].side();
        R x[5], y[5] = {R(0), R(0), R(0), R(0), R(0)};
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          const int q = ring_in(o, c);
          const int z = p - dir_x(q) - dir_y(q) * W;
          x[c] = L[LF + q - 1][z];
          if constexpr (TH) y[c] = L[TH ? LG + q - 1 : 0][z];
        }
        const R S0 = f[0] + x[0] + x[1], Sp = x[2] + x[3] + x[4];
        const R S0g = gg[0] + y[0] + y[1], Spg = y[2] + y[3] + y[4];
        const bool vel = (m[e] & 3) == FLOW_VELOCITY;
        const double fac = vel ? a.ufac[level] : 0.0;
        fwd_ring<R, TH>(
            g, S0, Sp, S0g, Spg, o, m[e], [&](int c) { return c ? uby[e] : ubx[e]; },
            [&]() { return fac; }, [&]() { return Tb[e]; }, dn, un, vn, Tn);
        for (int top = 0; top < 2; ++top) {
          if (!n[e].feeds(top)) continue;
          const int pc = p + (top ? W : -W), kc = k + (top ? g.nx : -g.nx);
          cd[n[e].corner_at(top)] = dn;
          L[LU][pc] = L[LV][pc] = R(0);
          if constexpr (TH) L[LT][pc] = Tn;
          if (keep && n[e].ext() == 0) {
            if (out[0]) out[0][kc] = dn;
            out[1][kc] = out[2][kc] = R(0);
            if constexpr (TH) out[3][kc] = Tn;
          }
        }
      }
      d[e] = dn;
      u[e] = un;
      v[e] = vn;
      L[LU][p] = un;
      L[LV][p] = vn;
      if constexpr (TH) {
        T[e] = Tn;
        L[LT][p] = Tn;
      }
      if (n[e].ext() == 0) {
        if (keep) {
          if (out[0]) out[0][k] = dn;
          out[1][k] = un;
          out[2][k] = vn;
          if constexpr (TH) out[3][k] = Tn;
        }
        if (a.acc) obj_add<R, TH>(a.objective, m[e], be[e], dn, un, Tn, part);
      }
    }
    if (a.acc) {
      if (__any(part != 0.0)) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off, 64);
      }
      if ((tid & 63) == 0) red[st][tid >> 6] = part;
    }
  }
  if (a.acc) {
    lds_barrier();
    if (tid == 0) {
      double acc = a.acc[t.tile];
      for (int st = 0; st < ms.k; ++st) {
        double x = 0.0;
        for (int w = 0; w < NT / 64; ++w) x += red[st][w];
        acc += x;
      }
      a.acc[t.tile] = acc;
    }
  }
}

// ---------------------------------------------------------------------------
// ALKS steps
// ---------------------------------------------------------------------------
// position of direction (cx, cy) among the eight stored ones
__device__ inline int dir_of(int cx, int cy) {
  // directions 7 4 8 / 3 0 1 / 6 2 5 by row cy = -1, 0, 1
  return int((0x526103847ull >> (4 * (3 * (cy + 1) + cx + 1))) & 15) - 1;
}

// LDS per node: the eight moving values rho~ + c_q.V (and Theta) for the pull,
// s~ (and q~, or B q~ in exact mode) for the divergences, T for its gradient.
// The state of step st is st.u[st] ...; a steady sweep gives one state
// (frozen). The sensitivity of the tile's nodes is summed in registers over
// the launch, in the order of single steps.
// (sv(st, f) gives field f of the state of step st: 1, 2 velocity, 3 T)
template <typename R, bool TH, int NT, int NPT, int NMAX, typename In>
__device__ __forceinline__ void multi_adj(const Geo& g, const AdjArgs<R>& a0, const MultiShape& ms,
                                          int tile, bool frozen, int unseeded, In&& sv) {
  constexpr int LE = 0, LS = 8, LQ = 11, LTH = 13, LT = 14, LBQ = 15, NA = TH ? 17 : 11;
  __shared__ R L[NA][NMAX];
  __shared__ R cm[4][4];  // r, U~, T~ of the corners (by their y-neighbours)
  MultiTile t;
  multi_tile(g, ms, tile, t);
  const int W = t.W;
  AdjArgs<R> a = a0;
  // corners take the moments of their y-neighbour and its local terms
  auto local_of = [&](const MultiNode& x) {
    return x.corner() ? x.k + (x.ey() > 0 ? g.nx : -g.nx) : x.k;
  };
  // the values the neighbours pull
  auto send = [&](int p, R r_, R vx_, R vy_, R th_) {
    const R xp = r_ + vx_, xm = r_ - vx_;
    L[LE + 0][p] = xp;
    L[LE + 1][p] = r_ + vy_;
    L[LE + 2][p] = xm;
    L[LE + 3][p] = r_ - vy_;
    L[LE + 4][p] = xp + vy_;
    L[LE + 5][p] = xm + vy_;
    L[LE + 6][p] = xm - vy_;
    L[LE + 7][p] = xp - vy_;
    if constexpr (TH) L[TH ? LTH : 0][p] = th_;
  };
  MultiNode n[NPT];
  // a node's own rho~, velocity, T and coefficients, and its moments rho~, U~,
  // T~ between the stages; the others wait in LDS, where its neighbours read them
  R r[NPT], ux[NPT], uy[NPT], T[NPT];
  R s[NPT], B[NPT], dBx[NPT], dBy[NPT], be[NPT];
  R Ux[NPT], Uy[NPT], Tt[NPT];
  double sens[NPT];
  int m[NPT];
#pragma unroll
  for (int e = 0; e < NPT; ++e) {
    n[e] = multi_node<NT, NPT>(g, t, e);
    r[e] = ux[e] = uy[e] = T[e] = R(0);
    s[e] = B[e] = dBx[e] = dBy[e] = be[e] = R(0);
    Ux[e] = Uy[e] = Tt[e] = R(0);
    sens[e] = 0.0;
    m[e] = 0;
    if (n[e].ext() == NO_NODE) continue;
    const int k = here<NT, NPT>(n[e].k);
    const int kl = local_of(n[e]);
    r[e] = a.r0[k];
    const R vx = a.vx0[k], vy = a.vy0[k];
    R th = R(0);
    s[e] = a.inv1pa[k];
    m[e] = a.mask[kl];
    ux[e] = sv(0, 1)[k];
    uy[e] = sv(0, 2)[k];
    if constexpr (TH) {
      th = a.th0[k];
      T[e] = sv(0, 3)[kl];
      B[e] = a.B[k];
      if (a.beta) be[e] = a.beta[k];
    }
    if (a.sens_mode == 1 && n[e].ext() == 0) sens[e] = a.sens[k];
    send(n[e].p, r[e], vx, vy, th);
    if constexpr (TH) L[LS][n[e].p] = B[e];
  }
  if constexpr (TH) {
    lds_barrier();
    if (!a.exact)
#pragma unroll
      for (int e = 0; e < NPT; ++e)
        if (n[e].ext() <= 2 * ms.k - 2) {
          dBx[e] = end_d(L[LS], n[e].p, 1, n[e].ring() ? n[e].ex() : 0);
          dBy[e] = end_d(L[LS], n[e].p, W, n[e].ring() ? n[e].ey() : 0);
        }
  }
  // the moments whose differences the second stage takes
  auto keep = [&](int p, const R mom[9], R B_) {
#pragma unroll
    for (int x = 0; x < 3; ++x) L[LS + x][p] = mom[3 + x];
    if constexpr (TH) {
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        L[TH ? LQ + x : 0][p] = mom[7 + x];
        if (a.exact) L[TH ? LBQ + x : 0][p] = B_ * mom[7 + x];
      }
    }
  };
  for (int st = 0; st < ms.k; ++st) {
    const int reach = 2 * (ms.k - st) - 1;  // moments are needed this far out
    const bool want = a0.sens_mode == 1 || (a0.sens_mode == 2 && st == ms.k - 1);
    if (st == unseeded) {  // level 0 carries no seed
      a.seed_dp = a.seed_heat = a.seed_src = a.seed_bt = 0.0;
      a.sens_b_only = a0.exact;
    }
    lds_barrier();
#pragma unroll
    for (int e = 0; e < NPT; ++e) {
      if (n[e].ext() > reach) continue;
      const int p = here<NT, NPT>(n[e].p);
      if constexpr (TH)
        if (want && (st == 0 || !frozen || a0.sens_mode == 2)) {
          // (a corner's own T enters no gradient that is used)
          L[TH ? LT : 0][p] = T[e];
        }
      const bool RING_SLOT = e == NPT - 1;  // (known once the loop is unrolled)
      if (RING_SLOT && n[e].corner()) continue;
      R mom[9];
      if (!(RING_SLOT && n[e].ring())) {
        R E[9], G[9];
        E[0] = r[e];
        G[0] = TH ? L[TH ? LTH : 0][p] : R(0);
#pragma unroll
        for (int q = 1; q < 9; ++q) {
          const int o = p + CX[q] + CY[q] * W;
          E[q] = L[LE + q - 1][o];
          G[q] = TH ? L[TH ? LTH : 0][o] : R(0);
        }
        adj_mom<R, TH>(E, G, mom);
      } else {
        const int o = n[e].side();
        int cx[6], cy[6];
        ring_dirs(o, cx, cy);
        R f[6], gq[6];
        f[0] = r[e];
        gq[0] = TH ? L[TH ? LTH : 0][p] : R(0);
#pragma unroll
        for (int q = 1; q < 6; ++q) {
          const int x = p + cx[q] + cy[q] * W;
          f[q] = L[LE + dir_of(cx[q], cy[q])][x];
          gq[q] = TH ? L[TH ? LTH : 0][x] : R(0);
        }
        ring_fill<R, TH>(a, o, m[e], ux[e], uy[e], T[e], f, gq, mom);
        for (int top = 0; top < 2; ++top) {
          if (!n[e].feeds(top)) continue;
          const int pc = p + (top ? W : -W), c = n[e].corner_at(top);
          cm[c][0] = mom[0];
          cm[c][1] = mom[1];
          cm[c][2] = mom[2];
          if constexpr (TH) cm[c][3] = mom[6];
          keep(pc, mom, B[e]);  // (B is that of the fluid on the whole ring)
        }
      }
      keep(p, mom, B[e]);
      r[e] = mom[0];
      Ux[e] = mom[1];
      Uy[e] = mom[2];
      if constexpr (TH) Tt[e] = mom[6];
    }
    // the next step's state, in flight during the second stage
    R nux[NPT], nuy[NPT], nT[NPT];
    const bool next = !frozen && st + 1 < ms.k;
#pragma unroll
    for (int e = 0; e < NPT; ++e) {
      nux[e] = nuy[e] = nT[e] = R(0);
      if (!next || n[e].ext() > reach - 2) continue;
      const int k = here<NT, NPT>(n[e].k);
      nux[e] = sv(st + 1, 1)[k];
      nuy[e] = sv(st + 1, 2)[k];
      if constexpr (TH) nT[e] = sv(st + 1, 3)[local_of(n[e])];
    }
    lds_barrier();
#pragma unroll
    for (int e = 0; e < NPT; ++e) {
      if (n[e].ext() > reach - 1) continue;
      const bool RING_SLOT = e == NPT - 1;
      const int p = here<NT, NPT>(n[e].p), k = here<NT, NPT>(n[e].k);
      R mom[9] = {r[e], Ux[e], Uy[e], L[LS][p], L[LS + 1][p], L[LS + 2][p], Tt[e], R(0), R(0)};
      if (RING_SLOT && n[e].corner()) {
        const int c = n[e].corner_of();
        mom[0] = cm[c][0];
        mom[1] = cm[c][1];
        mom[2] = cm[c][2];
        if constexpr (TH) mom[6] = cm[c][3];
      }
      if constexpr (TH) {
        mom[7] = L[TH ? LQ : 0][p];
        mom[8] = L[TH ? LQ + 1 : 0][p];
      }
      R rn, vxn, vyn, thn = R(0);
      auto local = [&](auto rc) {
        constexpr bool RING = decltype(rc)::value;
        auto dx = [&](int f) { return end_d(L[f], p, 1, RING ? n[e].ex() : 0); };
        auto dy = [&](int f) { return end_d(L[f], p, W, RING ? n[e].ey() : 0); };
        AdjNode<R> nd;
        nd.s = s[e];
        nd.ux = ux[e];
        nd.uy = uy[e];
        nd.ring = RING;
        R dq = R(0);
        if constexpr (TH) {
          nd.Tl = T[e];
          nd.probe = a.seed_heat != 0.0 && (m[e] & TAG_PROBE);
          nd.uxl = ux[e];
          if (RING && nd.probe && n[e].corner()) nd.uxl = sv(frozen ? 0 : st, 1)[local_of(n[e])];
          nd.beta = be[e];
          nd.B = B[e];
          nd.dBx = dBx[e];
          nd.dBy = dBy[e];
          dq = a.exact ? add2(dx(TH ? LBQ : 0), dy(TH ? LBQ + 1 : 0))
                       : add2(dx(TH ? LQ : 0), dy(TH ? LQ + 1 : 0));
        }
        double pair, adj_T;
        adj_node<R, TH>(g, a, nd, mom, add2(dx(LS), dy(LS + 1)),
                        add2(dx(LS + 1), dy(LS + 2)), dq, rn, vxn, vyn, thn, pair,
                        adj_T);
        if (!RING && want && n[e].ext() == 0) {
          R dTx = R(0), dTy = R(0);
          if constexpr (TH) {
            dTx = dx(TH ? LT : 0);
            dTy = dy(TH ? LT : 0);
          }
          sens[e] += adj_sens<R, TH>(a, pair, adj_T, a.dA3[k], TH ? a.dB[k] : R(0),
                                     TH && a.beta ? a.dbeta[k] : R(0), T[e], dTx, dTy,
                                     mom[7], mom[8]);
        }
      };
      if (RING_SLOT && n[e].ring()) local(std::true_type());
      else local(std::false_type());
      if (st + 1 < ms.k) {
        r[e] = rn;
        send(p, rn, vxn, vyn, thn);
        if (next) {
          ux[e] = nux[e];
          uy[e] = nuy[e];
          T[e] = nT[e];
        }
      } else {  // (only the tile's nodes reach this far in the last step)
        a.r1[k] = rn;
        a.vx1[k] = vxn;
        a.vy1[k] = vyn;
        if constexpr (TH) a.th1[k] = thn;
        if (a0.sens_mode) a.sens[k] = sens[e];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// kernels: one design
// ---------------------------------------------------------------------------
template <typename R, bool TH, int NT, int NPT, int NMAX>
__global__ __launch_bounds__(NT) void lks_multi_kernel(Geo g, FwdArgs<R> a, MultiShape ms,
                                                       MultiLevels<R> lv) {
  const int tile = xcd_tile(ms.ntx * ms.nty);
  if (tile < 0) return;
  multi_fwd<R, TH, NT, NPT, NMAX>(g, a, ms, tile, [&](int st, R* out[4]) {
#pragma unroll
    for (int f = 0; f < 4; ++f) out[f] = lv.f[st][f];
  });
}
template <typename R, bool TH, int NT, int NPT, int NMAX>
__global__ __launch_bounds__(NT) void alks_multi_kernel(Geo g, AdjArgs<R> a, MultiShape ms,
                                                        MultiStates<R> sv) {
  const int tile = xcd_tile(ms.ntx * ms.nty);
  if (tile < 0) return;
  multi_adj<R, TH, NT, NPT, NMAX>(g, a, ms, tile, sv.frozen, sv.unseeded,
                                  [&](int st, int f) {
                                    return f == 1 ? sv.u[st] : (f == 2 ? sv.v[st] : sv.T[st]);
                                  });
}

// ---------------------------------------------------------------------------
// kernels: batches
// ---------------------------------------------------------------------------
// The table tmap holds the design and the tile within it of every global
// tile; a design's tile counts are those of its descriptor's geometry.
template <typename R, bool TH, int NT, int NPT, int NMAX>
__global__ __launch_bounds__(NT) void lks_multi_batch_kernel(const BatchFwd<R>* __restrict__ d,
                                                             const int* __restrict__ tmap,
                                                             int total, int k, int parity) {
  const int t = xcd_tile(total);
  if (t < 0) return;
  const int di = tmap[2 * t];
  const Geo g = d[di].g;
  FwdArgs<R> a = d[di].a[parity];
  a.level_mid = a.level_out;
  multi_fwd<R, TH, NT, NPT, NMAX>(g, a, {g.ntx, g.nty, k}, tmap[2 * t + 1],
                                  [&](int st, R* out[4]) {
                                    const bool last = st == k - 1;
                                    out[0] = last ? a.d1 : nullptr;
                                    out[1] = last ? a.ux1 : nullptr;
                                    out[2] = last ? a.uy1 : nullptr;
                                    out[3] = last ? a.T1 : nullptr;
                                  });
}
template <typename R, bool TH, int NT, int NPT, int NMAX>
__global__ __launch_bounds__(NT) void alks_multi_batch_kernel(const BatchAdj<R>* __restrict__ d,
                                                              const int* __restrict__ tmap,
                                                              int total, int k, int parity,
                                                              int last) {
  const int t = xcd_tile(total);
  if (t < 0) return;
  const int di = tmap[2 * t];
  const Geo g = d[di].g;
  AdjArgs<R> a = d[di].a[parity];
  a.sens_mode = last ? 2 : 0;
  multi_adj<R, TH, NT, NPT, NMAX>(g, a, {g.ntx, g.nty, k}, tmap[2 * t + 1], true, -1,
                                  [&](int, int f) {
                                    return f == 1 ? a.ux : (f == 2 ? a.uy : a.T);
                                  });
}

// unsteady batches: the levels of a launch resolved from the design's store
template <typename R, bool TH, int NT, int NPT, int NMAX>
__global__ __launch_bounds__(NT) void lks_multi_ubatch_kernel(
    const BatchFwd<R>* __restrict__ d, const BatchStore<R>* __restrict__ st,
    const int* __restrict__ tmap, int total, int k, LevelRef in, MultiRefs lv, int level,
    int use_acc) {
  const int t = xcd_tile(total);
  if (t < 0) return;
  const int di = tmap[2 * t];
  const BatchStore<R> s = st[di];
  const Geo g = d[di].g;
  FwdArgs<R> a = d[di].a[0];
  a.d0 = level_field(s, in, 0);
  a.ux0 = level_field(s, in, 1);
  a.uy0 = level_field(s, in, 2);
  a.T0 = level_field(s, in, 3);
  a.level_mid = level;
  a.level_out = s.n_ufac - 1;
  if (!use_acc) a.acc = nullptr;
  multi_fwd<R, TH, NT, NPT, NMAX>(
      g, a, {g.ntx, g.nty, k}, tmap[2 * t + 1], [&](int i, R* out[4]) {
        // of a level inside the launch its checkpoint or slot is kept (a slot
        // without density)
        const LevelRef r = lv.r[i];
        const bool last = i == k - 1, held = last || r.kind != LVL_PING;
        out[0] = last || r.kind == LVL_CKPT ? level_field(s, r, 0) : nullptr;
        out[1] = held ? level_field(s, r, 1) : nullptr;
        out[2] = held ? level_field(s, r, 2) : nullptr;
        out[3] = held ? level_field(s, r, 3) : nullptr;
      });
}
template <typename R, bool TH, int NT, int NPT, int NMAX>
__global__ __launch_bounds__(NT) void alks_multi_ubatch_kernel(
    const BatchAdj<R>* __restrict__ d, const BatchStore<R>* __restrict__ st,
    const int* __restrict__ tmap, int total, int k, int parity, MultiRefs lv, int unseeded) {
  const int t = xcd_tile(total);
  if (t < 0) return;
  const int di = tmap[2 * t];
  const BatchStore<R> s = st[di];
  const Geo g = d[di].g;
  AdjArgs<R> a = d[di].a[parity];
  a.sens_mode = 1;
  multi_adj<R, TH, NT, NPT, NMAX>(g, a, {g.ntx, g.nty, k}, tmap[2 * t + 1], false, unseeded,
                                  [&](int i, int f) { return level_field(s, lv.r[i], f); });
}

// ---------------------------------------------------------------------------
// launch shapes
// ---------------------------------------------------------------------------
constexpr int LDS_BYTES = 160 * 1024 - 2048;  // of a CU, less the small tables
template <bool TH, bool ADJ>
constexpr int ARRAYS = ADJ ? (TH ? 17 : 11) : (TH ? 19 : 10);
// region nodes of the two-nodes-per-thread block
template <typename R, bool TH, bool ADJ>
constexpr int NODES2 =
    std::min(2048, LDS_BYTES / int(ARRAYS<TH, ADJ> * sizeof(R)) / 32 * 32);

// threads of the block of 1024 nodes: one node each, but two each in the FP64
// thermal adjoint, whose node does not fit the 128 registers of 1024 threads
template <typename R, bool TH, bool ADJ>
constexpr int THREADS1 = TH && ADJ && sizeof(R) == 8 ? 512 : 1024;

template <int N>
using IntC = std::integral_constant<int, N>;

struct Block {
  int threads, nodes, region;  // threads, node slots, LDS positions
};
// variant 0: 512 threads, 1: 1024 threads, 2: 1024 threads with two nodes each
Block block_of(int variant, int rsz, bool th, bool adj) {
  if (variant == 0) return {512, 512, 512};
  if (variant == 1)
    return {rsz == 8 && th && adj ? THREADS1<double, true, true> : 1024, 1024, 1024};
  int n = 0;
  if (rsz == 4) n = th ? (adj ? NODES2<float, true, true> : NODES2<float, true, false>)
                       : (adj ? NODES2<float, false, true> : NODES2<float, false, false>);
  else n = th ? (adj ? NODES2<double, true, true> : NODES2<double, true, false>)
              : (adj ? NODES2<double, false, true> : NODES2<double, false, false>);
  return {1024, n > 1024 ? 2048 : 0, n > 1024 ? n : 0};
}

// largest region (LDS positions) and slot count over the tiles
// (lead: first slot that ring nodes may take)
void region_of(const Geo& g, int ntx, int nty, int k, int lead, int* nodes, int* slots) {
  int mw = 0, mh = 0, ms = 0;
  const int h = 2 * k;
  auto span = [&](int b, int nt, int n, int* lo, int* hi) {
    *lo = int((long long)b * n / nt) - h;
    *hi = int((long long)(b + 1) * n / nt) + h;
    if (!g.periodic) {
      *lo = std::max(*lo, 0);
      *hi = std::min(*hi, n);
    }
  };
  for (int by = 0; by < nty; ++by) {
    int y0, y1;
    span(by, nty, g.ny, &y0, &y1);
    mh = std::max(mh, y1 - y0);
    for (int bx = 0; bx < ntx; ++bx) {
      int x0, x1;
      span(bx, ntx, g.nx, &x0, &x1);
      mw = std::max(mw, x1 - x0);
      int wi = x1 - x0, hi = y1 - y0, nr = 0;
      if (!g.periodic) {
        wi = std::min(x1, g.nx - 1) - std::max(x0, 1);
        hi = std::min(y1, g.ny - 1) - std::max(y0, 1);
        nr = (x1 - x0) * (y1 - y0) - wi * hi;
      }
      ms = std::max(ms, nr ? std::max((wi * hi + 63) & ~63, lead) + nr : wi * hi);
    }
  }
  *nodes = mw * mh;
  *slots = ms;
}

}  // namespace

// tile counts for at most `most` tiles: the ones whose tiles with a halo of 4
// nodes have the smallest area (tiles at least 2 nodes wide and tall, so that
// one-sided differences at the ends stay inside the region)
void tiles_for(const Geo& g, int most, int* ntx, int* nty) {
  long long best = 0;
  for (int x = 1; x <= std::min(most, g.nx / 2); ++x) {
    const int y = std::max(1, std::min(most / x, g.ny / 2));
    const long long area = (long long)((g.nx + x - 1) / x + 8) * ((g.ny + y - 1) / y + 8);
    if (!best || area < best) {
      best = area;
      *ntx = x;
      *nty = y;
    }
  }
}

MultiPlan multi_plan(const Geo& g, int rsz, bool adj, int max_tiles) {
  const bool th = g.thermal;
  // rounds of one block per CU of the 256. FP32 without temperature: the tile kernels'
  // 64 x 8 and 64 x 16 blocks overlap their loads with each other's work and
  // need no halo of 2k nodes, and are ahead from 1024 x 768 on (8.8 against
  // 9.5 us per forward step; 1024 x 512: 6.7 against 6.4). FP32 thermal: 1536 x
  // 1024 25.4 against 24.1, 2048 x 1024 30.8 against 30.6 us. FP64: ahead
  // through 2048 x 2048 (57.6 against 53.1 us, thermal 163 against 122).
  const int rmax = rsz == 8 ? 32 : (th ? 6 : 2);
  const long long first = (long long)g.N / (256 * 2048);
  for (int rounds = int(std::max(1LL, std::min(first, 64LL))); rounds <= rmax; ++rounds) {
    MultiPlan p;
    tiles_for(g, 256 * rounds, &p.ntx, &p.nty);
    if (p.ntx * p.nty > max_tiles) break;
    auto most_steps = [&](int variant) {
      const Block b = block_of(variant, rsz, th, adj);
      int k = 0;
      for (int t = 1; t <= (variant == 2 ? 7 : 6) && b.region; ++t) {
        int nodes, slots;
        region_of(g, p.ntx, p.nty, t, b.nodes - b.threads, &nodes, &slots);
        if (nodes <= b.region && slots <= b.nodes) k = t;
      }
      return k;
    };
    // The smaller block where it holds enough steps (its stages are shorter:
    // 201 x 201 thermal FP32 adjoint, 4 steps of 1024 nodes 3.2 us per step, 5 of
    // 2048 4.0), the larger one otherwise (384 x 384: 5 steps 2.5 us, where 1024
    // nodes hold 2 and take 3.6); 512 nodes only in the FP64 thermal adjoint, whose
    // larger blocks keep two nodes per thread (64 x 64: 4 steps 3.1 against 3.7).
    const int k1 = most_steps(1);
    if (rsz == 8 && th && adj) {
      const int k0 = most_steps(0);
      p.variant = k0 >= 3 ? 0 : 1;
      p.k = k0 >= 3 ? k0 : k1;
    } else {
      const int k2 = most_steps(2);
      const bool one = k1 >= (th || adj ? 4 : 5) || k2 <= k1;
      p.variant = one ? 1 : 2;
      p.k = one ? k1 : k2;
    }
    if (p.k >= 2) return p;
  }
  return MultiPlan();
}

// tile counts of a design whose tiles are at most `tile` nodes wide and tall
void multi_batch_tiles(const Geo& g, int tile, int* ntx, int* nty) {
  *ntx = std::max(1, std::min((g.nx + tile - 1) / tile, g.nx / 2));
  *nty = std::max(1, std::min((g.ny + tile - 1) / tile, g.ny / 2));
}

// Batches. While the tiles of all designs fit one round of blocks, the
// smallest tiles that do, with the steps their region holds (8 designs of 64 to
// 256 nodes a side, FP32: 28 x 28 tiles, 4 steps, 2.9 us per step of all; 36 x
// 36, 2 steps, 4.2; the tile kernels 6.4. 4 designs of 64 x 64: 8 x 8 tiles, 6
// steps, 2.2 us against 5.4 of the 64 x 4 tile kernels, FP64 2.4 and 5.7, thermal 3.6
// and 7.9, FP64 4.6 and 8.6). Over several rounds larger tiles with
// fewer steps: 32 designs of 128 to 512, 3.26M nodes, FP32 36 x 36 and 2 steps
// 37.3 forward and 38.4 us adjoint against 41.0 and 39.6 of the 64 x 8 tile
// kernels, FP64 30 x 30 and 3 steps 46.9, 48.4 against 65.9, 79.3; 16 thermal
// ones, 1.46M nodes, FP32 33.9, 38.0 against 39.5, 41.6, FP64 24 x 24 and 2 steps
// 61.9, 71.5 against 82.8, 92.5.
// What several rounds cost grows with the rounds, whatever the tiles hold, and
// the tile kernels' time with their blocks, so designs a few tiles wide or tall
// and, in FP32 without temperature, whole rounds of it are left to those. us per
// step, tile kernels -> R rounds instead of B blocks: FP32 5 designs of 256 x 256 8.6
// -> 7.9 (R = 2, B = 640), 24 of 200 x 200 18.3 -> 16.7 (4, 2400), but one of 1000 x 1000
// 13.7 -> 14.8 (4, 2000) and 30 of 300 x 40 9.6 -> 11.4 (3, 750); FP64 100 of 64 x 64
// 17.4 -> 14.8 (4, 800), 16 of 1000 x 10 8.7 -> 9.5 (3, 512); thermal FP32 5 of 256 x 256
// 16.0 -> 13.8 (2, 1280), 20 of 700 x 5 11.1 -> 12.8 (2, 440); thermal FP64 16 of 1000 x 10
// 18.1 -> 17.8 (3, 768), 20 of 700 x 5 11.9 -> 16.5 (3, 440).
bool worth_rounds(const Geo* const* g, int n, int rsz, bool th, long long tiles) {
  const long long R = (tiles + 255) / 256;
  long long B = 0;
  for (int d = 0; d < n; ++d)
    B += (long long)tiles_along(g[d]->nx, TX) * tiles_along(g[d]->ny, th ? 4 : 8);
  if (th) return B >= (rsz == 4 ? 500 : 250) * R;
  return R <= 2 || B >= (rsz == 4 ? 850 * R - 1050 : 180 * R);
}

// The first candidate that `holds`: from the smallest tiles of one round of
// blocks on to the largest ones.
BatchPlan multi_batch_plan(const Geo* const* g, int n, int rsz, bool th,
                           const std::function<bool(const BatchPlan&)>& holds) {
  struct Cand {
    int tile, k, variant;
  };
  static const Cand f32[] = {{8, 6, 1}, {12, 5, 1}, {16, 4, 1}, {20, 6, 2},
                             {24, 5, 2}, {28, 4, 2}, {32, 3, 2}, {36, 2, 2}};
  static const Cand f64[] = {{8, 6, 1}, {12, 5, 1}, {16, 4, 1}, {18, 6, 2},
                             {22, 5, 2}, {26, 4, 2}, {30, 3, 2}};
  static const Cand f64t[] = {{8, 6, 1}, {12, 5, 1}, {16, 4, 1}, {20, 3, 1}, {24, 2, 1}};
  const Cand* c = rsz == 4 ? f32 : (th ? f64t : f64);
  const int nc = rsz == 4 ? 8 : (th ? 5 : 7);
  for (int i = 0; i < nc; ++i) {
    BatchPlan p;
    p.tile = c[i].tile;
    p.kf = p.ka = c[i].k;
    p.vf = p.va = c[i].variant;
    long long tiles = 0;
    for (int d = 0; d < n; ++d) {
      int x, y;
      multi_batch_tiles(*g[d], p.tile, &x, &y);
      tiles += (long long)x * y;
    }
    if ((tiles <= 256 || (i == nc - 1 && worth_rounds(g, n, rsz, th, tiles))) && holds(p))
      return p;
  }
  return BatchPlan();
}

// whether `steps` steps of a design's tiles fit the block of a variant
bool multi_fits(const Geo& g, int ntx, int nty, int rsz, bool adj, int variant, int steps) {
  const Block b = block_of(variant, rsz, g.thermal, adj);
  if (!b.region) return false;
  int nodes, slots;
  region_of(g, ntx, nty, steps, b.nodes - b.threads, &nodes, &slots);
  return nodes <= b.region && slots <= b.nodes;
}

// f(TH, NT, NPT, NMAX) of the block a variant names (as integral constants)
template <typename R, bool ADJ, typename F>
void with_block(bool th, int variant, F&& f) {
  auto go = [&](auto t) {
    constexpr bool TH = decltype(t)::value;
    constexpr int N2 = NODES2<R, TH, ADJ>, NT1K = THREADS1<R, TH, ADJ>;
    if (variant == 0) f(t, IntC<512>(), IntC<1>(), IntC<512>());
    else if (variant == 1) f(t, IntC<NT1K>(), IntC<1024 / NT1K>(), IntC<1024>());
    else if constexpr (N2 > 1024) f(t, IntC<1024>(), IntC<2>(), IntC<N2>());
  };
  if (th) go(std::true_type());
  else go(std::false_type());
}

template <typename R>
void launch_lks_multi(const Geo& g, const MultiPlan& p, int steps, const FwdArgs<R>& a,
                      const MultiLevels<R>& lv, hipStream_t s) {
  if (p.variant == MARCH) {
    FwdArgs<R> b = a;
    b.d1 = lv.f[steps - 1][0];
    b.ux1 = lv.f[steps - 1][1];
    b.uy1 = lv.f[steps - 1][2];
    return launch_lks_march<R>(g, steps, b, s);
  }
  const MultiShape ms{p.ntx, p.nty, steps};
  with_block<R, false>(g.thermal, p.variant, [&](auto th, auto nt, auto npt, auto nmax) {
    lks_multi_kernel<R, decltype(th)::value, nt.value, npt.value, nmax.value>
        <<<unsigned(xcd_blocks(ms.ntx * ms.nty)), nt.value, 0, s>>>(g, a, ms, lv);
  });
}
template <typename R>
void launch_alks_multi(const Geo& g, const MultiPlan& p, int steps, const AdjArgs<R>& a,
                       const MultiStates<R>& sv, hipStream_t s) {
  if (p.variant == MARCH) return launch_alks_march<R>(g, steps, a, s);
  const MultiShape ms{p.ntx, p.nty, steps};
  with_block<R, true>(g.thermal, p.variant, [&](auto th, auto nt, auto npt, auto nmax) {
    alks_multi_kernel<R, decltype(th)::value, nt.value, npt.value, nmax.value>
        <<<unsigned(xcd_blocks(ms.ntx * ms.nty)), nt.value, 0, s>>>(g, a, ms, sv);
  });
}
template <typename R>
void launch_lks_multi_batch(const BatchFwd<R>* d, const int* tmap, int total, bool thermal,
                            int variant, int steps, int parity, hipStream_t s) {
  with_block<R, false>(thermal, variant, [&](auto th, auto nt, auto npt, auto nmax) {
    lks_multi_batch_kernel<R, decltype(th)::value, nt.value, npt.value, nmax.value>
        <<<unsigned(xcd_blocks(total)), nt.value, 0, s>>>(d, tmap, total, steps, parity);
  });
}
template <typename R>
void launch_alks_multi_batch(const BatchAdj<R>* d, const int* tmap, int total, bool thermal,
                             int variant, int steps, int parity, int last, hipStream_t s) {
  with_block<R, true>(thermal, variant, [&](auto th, auto nt, auto npt, auto nmax) {
    alks_multi_batch_kernel<R, decltype(th)::value, nt.value, npt.value, nmax.value>
        <<<unsigned(xcd_blocks(total)), nt.value, 0, s>>>(d, tmap, total, steps, parity, last);
  });
}
template <typename R>
void launch_lks_multi_ubatch(const BatchFwd<R>* d, const BatchStore<R>* st, const int* tmap,
                             int total, bool thermal, int variant, int steps, LevelRef in,
                             const MultiRefs& lv, int level, int use_acc, hipStream_t s) {
  with_block<R, false>(thermal, variant, [&](auto th, auto nt, auto npt, auto nmax) {
    lks_multi_ubatch_kernel<R, decltype(th)::value, nt.value, npt.value, nmax.value>
        <<<unsigned(xcd_blocks(total)), nt.value, 0, s>>>(d, st, tmap, total, steps, in, lv, level,
                                                          use_acc);
  });
}
template <typename R>
void launch_alks_multi_ubatch(const BatchAdj<R>* d, const BatchStore<R>* st, const int* tmap,
                              int total, bool thermal, int variant, int steps, int parity,
                              const MultiRefs& lv, int unseeded, hipStream_t s) {
  with_block<R, true>(thermal, variant, [&](auto th, auto nt, auto npt, auto nmax) {
    alks_multi_ubatch_kernel<R, decltype(th)::value, nt.value, npt.value, nmax.value>
        <<<unsigned(xcd_blocks(total)), nt.value, 0, s>>>(d, st, tmap, total, steps, parity, lv,
                                                          unseeded);
  });
}

#define LKS_MULTI_INSTANTIATE(R)                                                             \
  template void launch_lks_multi<R>(const Geo&, const MultiPlan&, int, const FwdArgs<R>&,    \
                                    const MultiLevels<R>&, hipStream_t);                     \
  template void launch_alks_multi<R>(const Geo&, const MultiPlan&, int, const AdjArgs<R>&,   \
                                     const MultiStates<R>&, hipStream_t);                    \
  template void launch_lks_multi_batch<R>(const BatchFwd<R>*, const int*, int, bool, int, int, \
                                          int, hipStream_t);                                 \
  template void launch_alks_multi_batch<R>(const BatchAdj<R>*, const int*, int, bool, int, int, \
                                           int, int, hipStream_t);                           \
  template void launch_lks_multi_ubatch<R>(const BatchFwd<R>*, const BatchStore<R>*, const int*, \
                                           int, bool, int, int, LevelRef, const MultiRefs&, int, \
                                           int, hipStream_t);                                \
  template void launch_alks_multi_ubatch<R>(const BatchAdj<R>*, const BatchStore<R>*,        \
                                            const int*, int, bool, int, int, int,            \
                                            const MultiRefs&, int, hipStream_t);
LKS_MULTI_INSTANTIATE(float)
LKS_MULTI_INSTANTIATE(double)

}  // namespace lks
