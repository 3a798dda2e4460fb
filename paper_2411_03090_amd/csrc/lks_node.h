// Device functions of the D2Q9 LKS and ALKS steps that act on one node, shared
// by the tile kernels (lks_kernels.hip), the several-steps kernels of small
// grids (lks_multi.hip) and the marching kernels of large ones (lks_march.hip).
// They take values rather than positions and contract
// multiply-adds only within a source expression, so that every kernel built on
// them gives the same bits.
#pragma once
#include <hip/hip_runtime.h>

#include "lks_device.h"

namespace lks {

// D2Q9 velocities and weights (Sec. 2.3, eq:D2Q9w)
__device__ constexpr int CX[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
__device__ constexpr int CY[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
__device__ constexpr double WD[9] = {4.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9,
                                     1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36};

__device__ inline int wrapi(int a, int n) { return a < 0 ? a + n : (a >= n ? a - n : a); }

// ---------------------------------------------------------------------------
// block reduction helper (deterministic)
// ---------------------------------------------------------------------------
template <int NT = NTHREADS>
__device__ inline double block_sum(double v, double* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < NT / 64; ++w) s += red[w];
  return s;
}

// Global tile of this block under the XCD-aware mapping, or -1.
__device__ inline int xcd_tile(int T) {
  const int nper = (T + NXCD - 1) / NXCD;
  const int b = blockIdx.x;
  const int tile = (b % NXCD) * nper + b / NXCD;
  return tile < T ? tile : -1;
}

// true on the boundary ring of a bounded domain, and outside it
__device__ inline bool on_ring(const Geo& g, int i, int j) {
  return i <= 0 || j <= 0 || i >= g.nx - 1 || j >= g.ny - 1;
}

// The ring nodes of the node rectangle [x0, x0 + w) x [y0, y0 + h) clipped
// to a bounded domain: its parts of the columns i = 0 and i = nx - 1, then
// of the rows j = 0 and j = ny - 1 without the end nodes of those rows.
struct RingSet {
  int ry0, bx0, nl, nr, nb;
};

__device__ inline int ring_set(const Geo& g, int x0, int y0, int w, int h, RingSet& s) {
  const int rx0 = max(x0, 0), rx1 = min(x0 + w, g.nx) - 1;
  const int ry0 = max(y0, 0), ry1 = min(y0 + h, g.ny) - 1;
  const int hc = ry1 - ry0 + 1;
  s.ry0 = ry0;
  s.nl = rx0 == 0 ? hc : 0;
  s.nr = rx1 == g.nx - 1 ? hc : 0;
  s.bx0 = max(rx0, 1);
  const int wr = max(min(rx1, g.nx - 2) - s.bx0 + 1, 0);
  s.nb = ry0 == 0 ? wr : 0;
  const int nt = ry1 == g.ny - 1 ? wr : 0;
  return s.nl + s.nr + s.nb + nt;
}

__device__ inline void ring_at(const Geo& g, const RingSet& s, int t, int* i, int* j) {
  if (t < s.nl) {
    *i = 0;
    *j = s.ry0 + t;
  } else if (t < s.nl + s.nr) {
    *i = g.nx - 1;
    *j = s.ry0 + t - s.nl;
  } else if (t < s.nl + s.nr + s.nb) {
    *i = s.bx0 + t - s.nl - s.nr;
    *j = 0;
  } else {
    *i = s.bx0 + t - s.nl - s.nr - s.nb;
    *j = g.ny - 1;
  }
}

// LDS finite difference along one axis at position p of a field with the
// given step: central (e = 0), or second-order one-sided at the low (e = 1)
// or high (e = -1) end of the axis. Without branches: a wave of ring nodes
// holds all three kinds, and each branch would wait for LDS on its own. The
// product by 3 is the one that rounds, and is fused here rather than where the
// compiler likes, so that all kernels round alike.
template <typename R>
__device__ inline R end_f(R f0, R f1, R f2, int e) {
  const R mid = R(0.5) * (f1 - f2);
  const R lo = R(0.5) * (__builtin_elementwise_fma(R(-3), f0, R(4) * f1) - f2);
  const R hi = R(0.5) * (__builtin_elementwise_fma(R(3), f0, R(-4) * f1) + f2);
  return e == 0 ? mid : (e > 0 ? lo : hi);
}
template <typename R>
__device__ inline R end_d(const R* s, int p, int step, int e) {
  return end_f(s[p], s[p + (e == 0 ? step : e * step)], s[p + (e == 0 ? -step : 2 * e * step)], e);
}
// end kind of node coordinate c on an axis of n nodes
__device__ inline int end_of(int c, int n, int periodic) {
  return periodic ? 0 : (c == 0 ? 1 : (c == n - 1 ? -1 : 0));
}
template <typename R>
__device__ inline R lds_d(const R* s, int p, int step, int c, int n, int periodic) {
  return end_d(s, p, step, end_of(c, n, periodic));
}

// lds_d for a position whose tile is interior (INT: the tile and a 2-node
// halo lie off the boundary ring and need no wrap), where the central
// difference always applies
template <bool INT, typename R>
__device__ inline R lds_dx(const R* s, int p, int step, int c, int n, int periodic) {
  if constexpr (INT) return R(0.5) * (s[p + step] - s[p - step]);
  else return lds_d(s, p, step, c, n, periodic);
}

// the same difference of the product a*b of two LDS fields with their own
// positions and row steps
template <bool INT, typename R>
__device__ inline R lds_dxp(const R* a, int pa, int sa, const R* b, int pb, int sb, int c, int n,
                            int periodic) {
#pragma clang fp contract(off)
  const int e = INT ? 0 : end_of(c, n, periodic);
  const int o1 = e == 0 ? 1 : e, o2 = e == 0 ? -1 : 2 * e;
  const R f0 = a[pa] * b[pb], f1 = a[pa + o1 * sa] * b[pb + o1 * sb];
  const R f2 = a[pa + o2 * sa] * b[pb + o2 * sb];
  return end_f(f0, f1, f2, e);
}

// The nine post-collision values f'_i (and W of the temperature) of a node
// from its state and the differences of its velocity and temperature. put(i, f'_i)
// takes each as it is formed: a kernel that stores them to LDS from an array
// holds all nine first (2048 x 1024 FP32, 64 x 4 and 64 x 16 tiles: 27.3 and 21.2 us
// instead of 25.6 and 20.4).
template <typename R, typename Put>
__device__ inline void fwd_post(R A, R d, R ux, R uy, R uxx, R uxy, R uyx, R uyy, Put&& put) {
#pragma clang fp contract(on)
  // f'_i = w_i [P + 3 c.u + cx^2 Xx + cy^2 Yy + cx cy Xy]
  const R P = d - R(1.5) * (ux * ux + uy * uy);
  const R Xx = R(4.5) * ux * ux + R(2) * A * uxx;
  const R Yy = R(4.5) * uy * uy + R(2) * A * uyy;
  const R Xy = R(9) * ux * uy + R(2) * A * (uxy + uyx);
  const R u3x = R(3) * ux, u3y = R(3) * uy;
  const R w0 = R(4.0 / 9), w1 = R(1.0 / 9), w5 = R(1.0 / 36);
  const R diag = P + Xx + Yy;
  put(0, w0 * P);
  put(1, w1 * (P + u3x + Xx));
  put(2, w1 * (P + u3y + Yy));
  put(3, w1 * (P - u3x + Xx));
  put(4, w1 * (P - u3y + Yy));
  put(5, w5 * (diag + u3x + u3y + Xy));
  put(6, w5 * (diag - u3x + u3y - Xy));
  put(7, w5 * (diag - u3x - u3y + Xy));
  put(8, w5 * (diag + u3x - u3y - Xy));
}
template <typename R>
__device__ inline void fwd_flux(R T, R B, R ux, R uy, R Tx, R Ty, R& Wx, R& Wy) {
#pragma clang fp contract(on)
  Wx = R(3) * T * ux + B * Tx;
  Wy = R(3) * T * uy + B * Ty;
}

// g_q = w_q [T + c_q.W] (eq:geq2) of the node whose temperature is T and
// whose W is (Wx, Wy)
template <typename R>
__device__ inline R g_eq(int q, R T, R Wx, R Wy) {
#pragma clang fp contract(on)
  const R w0 = R(4.0 / 9), w1 = R(1.0 / 9), w5 = R(1.0 / 36);
  switch (q) {
    case 0: return w0 * T;
    case 1: return w1 * (T + Wx);
    case 2: return w1 * (T + Wy);
    case 3: return w1 * (T - Wx);
    case 4: return w1 * (T - Wy);
    case 5: return w5 * (T + Wx + Wy);
    case 6: return w5 * (T - Wx + Wy);
    case 7: return w5 * (T - Wx - Wy);
    default: return w5 * (T + Wx - Wy);
  }
}

// New state of an interior node from the pulled f'_i and g_i; s is its
// 1 / (1 + alpha), src says whether b is the heat-source coefficient.
template <typename R, bool TH>
__device__ inline void fwd_interior(const Geo& g, const R f[9], const R gg[9], R s, bool src, R b,
                                    R& dn, R& uxn, R& uyn, R& Tn) {
#pragma clang fp contract(on)
  dn = f[0] + f[1] + f[2] + f[3] + f[4] + f[5] + f[6] + f[7] + f[8];
  R Ux = f[1] - f[3] + f[5] - f[6] - f[7] + f[8];
  R Uy = f[2] - f[4] + f[5] + f[6] - f[7] - f[8];
  if constexpr (TH) {
    Tn = gg[0] + gg[1] + gg[2] + gg[3] + gg[4] + gg[5] + gg[6] + gg[7] + gg[8];
    // heat source Q = beta (1 - T) at the new level (eq:lbeg_ex,
    // eq:heatsource): T (1 + beta) = T* + beta
    if (src) Tn = (Tn + b) / (R(1) + b);
    // Boussinesq force at the new level, u (1 + alpha) = U* + G
    // (eq:lbef_ex, eq:boussinesqforce); zero when g beta is zero
    const R dT = Tn - R(g.Tref);
    Ux += R(g.gbx) * dT;
    Uy += R(g.gby) * dT;
  }
  uxn = Ux * s;
  uyn = Uy * s;
}

// Populations that arrive at a ring node of side o (0 -x, 1 +x, 2 -y, 3 +y):
// direction c of the five moving ones in ascending order, first the two along
// the wall (c.n = 0), then the three moving outwards (c.n > 0). A packed
// table: a runtime index into an array would go to memory.
__device__ inline int ring_in(int o, int c) {
  constexpr unsigned T[4] = {0x76342u, 0x85142u, 0x87431u, 0x65231u};
  const unsigned t = o < 2 ? (o ? T[1] : T[0]) : (o == 2 ? T[2] : T[3]);
  return int((t >> (4 * c)) & 15u);
}
// velocity of direction q computed (CX, CY need a compile-time index)
__device__ inline int dir_x(int q) {
  return (q == 1 || q == 5 || q == 8) - (q == 3 || q == 6 || q == 7);
}
__device__ inline int dir_y(int q) {
  return (q == 2 || q == 5 || q == 6) - (q == 4 || q == 7 || q == 8);
}
// side of a ring node that is not a corner
__device__ inline int ring_side(const Geo& g, int i, int j) {
  return i == 0 ? 0 : (i == g.nx - 1 ? 1 : (j == 0 ? 2 : 3));
}

// New state of a ring node of side o and class m from the sums of the
// populations that arrive along the wall and at rest (S0) and from inside
// (Sp): ub(c) is component c of the prescribed velocity, fac() the level's inflow
// factor, Tb() the prescribed temperature or heat flux, each asked for where it
// is used only.
template <typename R, bool TH, typename U, typename F, typename B>
__device__ inline void fwd_ring(const Geo& g, R S0, R Sp, R S0g, R Spg, int o, int m, U&& ub,
                                F&& fac, B&& Tb, R& dn, R& uxn, R& uyn, R& Tn) {
#pragma clang fp contract(on)
  const int nx_ = o == 0 ? -1 : (o == 1 ? 1 : 0), ny_ = o == 2 ? -1 : (o == 3 ? 1 : 0);
  R un;
  if ((m & 3) == FLOW_VELOCITY) {
    const double f = fac();
    uxn = R(double(ub(0)) * f);
    uyn = R(double(ub(1)) * f);
    un = uxn * R(nx_) + uyn * R(ny_);
    dn = S0 + R(2) * Sp - un;
  } else {
    const R dout = R(g.drho_out);
    dn = dout;
    un = S0 + R(2) * Sp - dout;
    uxn = un * R(nx_);
    uyn = un * R(ny_);
  }
  if constexpr (TH) {
    // heat-flux node: -q.n = qbar with q = sum c_i g_i - u T (Sec. 2.4); Tb
    // holds qbar there (0: adiabatic)
    if (((m >> 2) & 3) == THERM_DIRICHLET) Tn = Tb();
    else Tn = (S0g + R(2) * Spg + Tb()) / (R(1) + un);
  }
}

// the objective's term of a node with class m and source coefficient beta at a new level (pressure drop,
// probe enthalpy flux, heat exchange or heated-node temperature)
template <typename R, bool TH>
__device__ inline void obj_add(int objective, int m, R beta, R dn, R uxn, R Tn, double& part) {
  if (objective == 1) {
    if (m & TAG_PROBE) part += double(uxn) * double(Tn);
  } else if (objective == 2) {
    if constexpr (TH) part += double(beta) * (double(Tn) - 1.0);
  } else if (objective == 3) {
    if (m & TAG_PROBE) part += double(Tn);
  } else {
    if (m & TAG_J_INLET) part += double(dn);
    if (m & TAG_J_OUTLET) part -= double(dn);
  }
}

// Least-squares completion of the adjoint populations at a ring node (see
// RingFillT) and the raw moments rho~, U~, s~ (xx, xy, yy), T~, q~ of the
// completed set. In the node's frame (outward normal n, tangent t) f holds
// the known populations: rest, t, -t, -n, -n + t, -n - t. Bound by the length
// of its chain (one wave of an edge tile runs it while the others wait): the
// reflection t -> -t splits the fixed linear map of the known populations
// into an even and an odd part, and the moments need only three sums over
// the unknown ones, so the flow part takes 10 products instead of the 27 of
// the full 3 x 9 map, and one operator serves the four sides.
template <typename R, bool TH>
__device__ inline void ring_fill(const AdjArgs<R>& a, int o, int m, R ux, R uy, R Tn,
                                 const R f[6], const R gq[6], R mom[9]) {
#pragma clang fp contract(on)
  const R w0 = R(4.0 / 9), w1 = R(1.0 / 9), w5 = R(1.0 / 36);
  const auto* op = as_scalar(a.ops);
  const R sg = (o & 1) ? R(1) : R(-1);
  const R un = sg * (o < 2 ? ux : uy);
  const bool diri = ((m >> 2) & 3) == THERM_DIRICHLET;
  R kappa = R(0), Tt = R(0), qn = R(0), qt = R(0);
  if constexpr (TH) {
    const R b1 = gq[1] + gq[2], b3 = gq[4] + gq[5], c1 = gq[1] - gq[2], c2 = gq[4] - gq[5];
    const R q0 = w1 * gq[3] + w5 * b3;
    R Y, X;
    if (diri) {
      Y = op->Dy[0] * gq[0] + op->Dy[1] * b1 + op->Dy[2] * gq[3] + op->Dy[3] * b3;
      X = op->Dx[0] * c1 + op->Dx[1] * c2;
    } else {
      // zero-flux completion in Schur form (no row seed)
      const R na = op->ka[0] * gq[0] + op->ka[1] * b1 + op->ka[2] * gq[3] + op->ka[3] * b3;
      const R ne = op->ke[0] * gq[0] + op->ke[1] * b1 + op->ke[2] * gq[3] + op->ke[3] * b3;
      const R den = op->A0 - R(2) * un * op->A1 + un * un * op->A2;
      kappa = (un * ne - na) / den;
      Y = op->Gy[0] * gq[0] + op->Gy[1] * b1 + op->Gy[2] * gq[3] + op->Gy[3] * b3;
      Y = Y - kappa * (op->Hc - un * op->H1);
      X = op->Gx[0] * c1 + op->Gx[1] * c2;
    }
    Tt = w0 * gq[0] + w1 * b1 + q0 + Y;
    qn = Y - q0;
    qt = w1 * c1 + w5 * c2 + X;
  }
  // boundary seed of the pressure-drop objective: its derivative with
  // respect to the boundary pressure, the same in every row
  R s = R(0);
  if (m & TAG_J_INLET) s += R(a.seed_dp);
  if (m & TAG_J_OUTLET) s -= R(a.seed_dp);
  const R kT = TH ? kappa * Tn : R(0);
  const R b1 = f[1] + f[2], b3 = f[4] + f[5], c1 = f[1] - f[2], c2 = f[4] - f[5];
  // sums over the unknown populations: Y weighted, Z those with a tangential
  // component, X their difference. A wave holds nodes of one type mostly;
  // the operator of each type present is read through the scalar unit.
  R Y = R(0), Z = R(0), X = R(0);
  const int v = (m & 3) == FLOW_VELOCITY ? 0 : 1;
#pragma nounroll
  for (int t = 0; t < 2; ++t) {
    if (!__any(v == t)) continue;
    const R y = op->Y[t][0] * f[0] + op->Y[t][1] * b1 + op->Y[t][2] * f[3] + op->Y[t][3] * b3 +
                op->Ys[t] * s + op->Yk[t] * kT;
    const R z = op->Z[t][0] * f[0] + op->Z[t][1] * b1 + op->Z[t][2] * f[3] + op->Z[t][3] * b3 +
                op->Zs[t] * s + op->Zk[t] * kT;
    const R x = op->X[t][0] * c1 + op->X[t][1] * c2;
    Y = v == t ? y : Y;
    Z = v == t ? z : Z;
    X = v == t ? x : X;
  }
  const R in = w1 * f[3] + w5 * b3;
  const R Un = Y - in, Ut = w1 * c1 + w5 * c2 + X;
  const R snn = in + Y, stt = w1 * b1 + w5 * b3 + Z, snt = X - w5 * c2;
  mom[0] = w0 * f[0] + w1 * b1 + in + Y;
  const bool ax = o < 2;  // normal along x: n = (sg, 0), t = (0, sg); else n = (0, sg), t = (-sg, 0)
  mom[1] = ax ? sg * Un : -sg * Ut;
  mom[2] = ax ? sg * Ut : sg * Un;
  mom[3] = ax ? snn : stt;
  mom[4] = ax ? snt : -snt;
  mom[5] = ax ? stt : snn;
  R qx = ax ? sg * qn : -sg * qt, qy = ax ? sg * qt : sg * qn;
  if constexpr (TH) {
    // heat-sink objective: the heated node's temperature is the flux closure
    // T (1 + u.n) = S0 + 2 S+ + qbar of the arriving populations, so
    // seed_bt w^cl / (1 + u.n) (w^cl = 1 along the wall, 2 moving outwards,
    // 0 inwards) leaves every completed adjoint population; its weighted
    // moments are -seed/(1 + u.n) on T~ and -seed/(1 + u.n) n/3 on q~
    if ((m & TAG_PROBE) && a.seed_bt != 0.0) {
      const R sb = R(a.seed_bt) / (R(1) + un);
      Tt -= sb;
      qx -= sb * (ax ? sg : R(0)) / R(3);
      qy -= sb * (ax ? R(0) : sg) / R(3);
    }
    // exact mode: the temperature of a prescribed-temperature node does not
    // depend on the populations that arrive there, so their adjoint is zero
    if (a.exact && diri) Tt = qx = qy = R(0);
  }
  mom[6] = Tt;
  mom[7] = qx;
  mom[8] = qy;
}

// lattice velocities of the known directions of ring_fill for orientation o
__device__ inline void ring_dirs(int o, int cx[6], int cy[6]) {
  const int sg = (o & 1) ? 1 : -1;
  const int nx_ = o < 2 ? sg : 0, ny_ = o < 2 ? 0 : sg;
  const int tx = -ny_, ty = nx_;
  cx[0] = cy[0] = 0;
  cx[1] = tx;
  cy[1] = ty;
  cx[2] = -tx;
  cy[2] = -ty;
  cx[3] = -nx_;
  cy[3] = -ny_;
  cx[4] = tx - nx_;
  cy[4] = ty - ny_;
  cx[5] = -tx - nx_;
  cy[5] = -ty - ny_;
}

// Moments rho~, U~, s~ (xx, xy, yy), T~, q~ of the pulled values f~_q, g~_q
// of an interior node, summed by weight class.
template <typename R, bool TH>
__device__ inline void adj_mom(const R E[9], const R G[9], R mom[9]) {
#pragma clang fp contract(on)
  const R w0 = R(4.0 / 9), w1 = R(1.0 / 9), w5 = R(1.0 / 36);
  const R sa = E[1] + E[3], sb = E[2] + E[4];
  const R p = E[5] + E[7], q = E[6] + E[8], pm = E[5] - E[7], qm = E[8] - E[6];
  const R ps = p + q;
  mom[0] = w0 * E[0] + w1 * (sa + sb) + w5 * ps;
  mom[1] = w1 * (E[1] - E[3]) + w5 * (pm + qm);
  mom[2] = w1 * (E[2] - E[4]) + w5 * (pm - qm);
  mom[3] = w1 * sa + w5 * ps;
  mom[4] = w5 * (p - q);
  mom[5] = w1 * sb + w5 * ps;
  mom[6] = mom[7] = mom[8] = R(0);
  if constexpr (TH) {
    const R gm = G[5] - G[7], hm = G[8] - G[6];
    const R gs = (G[5] + G[7]) + (G[6] + G[8]);
    mom[6] = w0 * G[0] + w1 * ((G[1] + G[3]) + (G[2] + G[4])) + w5 * gs;
    mom[7] = w1 * (G[1] - G[3]) + w5 * (gm + hm);
    mom[8] = w1 * (G[2] - G[4]) + w5 * (gm - hm);
  }
}

// a + b, rounded as written: the halves of a divergence are products by 0.5,
// which a fused add would not round where they are denormal
template <typename R>
__device__ inline R add2(R a, R b) {
#pragma clang fp contract(off)
  return a + b;
}

// What the local terms of a node need beside its moments: 1 / (1 + alpha),
// the velocity, and (thermal) T, u_x and the probe tag of the node whose
// moments were taken (the y-neighbour for corners), B with its differences
// (paper mode) and the heat-source coefficient.
template <typename R>
struct AdjNode {
  R s, ux, uy;
  R Tl, uxl, B, dBx, dBy, beta;
  int ring, probe;
};

// The local terms of eq:albef_ex / eq:albeg_ex at level n (seeds, 3 T q~
// coupling, implicit Brinkman), then V and Theta of the new level from the
// node's moments, div s~ = (dsx, dsy) and dq = div q~ (paper) or div (B q~)
// (exact). pair is the Brinkman pairing of the sensitivity, adj_T the T~ or
// Theta that pairs with the heat source.
template <typename R, bool TH>
__device__ inline void adj_node(const Geo& g, const AdjArgs<R>& a, const AdjNode<R>& n,
                                const R mom[9], R dsx, R dsy, R dq, R& r_out, R& Vx, R& Vy, R& Th,
                                double& pair, double& adj_T) {
#pragma clang fp contract(on)
  const R A2 = R(2.0 * g.A);
  const R r = mom[0], sxx = mom[3], sxy = mom[4], syy = mom[5];
  R Ux = mom[1], Uy = mom[2], Tt = R(0), qx = R(0), qy = R(0);
  if constexpr (TH) {
    Tt = mom[6];
    qx = mom[7];
    qy = mom[8];
    Ux += n.Tl * qx;
    Uy += n.Tl * qy;
    if (n.probe && a.seed_heat != 0.0) {
      Ux -= R(a.seed_heat / 3.0) * n.Tl;
      Tt -= R(a.seed_heat) * n.uxl;
    }
  }
  // paper: u~ = U~ / (1 + alpha) here; exact: V is divided by 1 + alpha
  // instead, after it is formed from the undivided u~
  const R su = a.exact ? R(1) : n.s;
  const R utx = Ux * su, uty = Uy * su;
  if constexpr (TH) {
    // paper: the Boussinesq coupling of eq:albeg_ex, 3 g beta . u~ on T~ at
    // interior nodes (zero when g beta is zero)
    if (!n.ring && !a.exact) Tt += R(3) * (R(g.gbx) * utx + R(g.gby) * uty);
    // heat source (interior nodes; beta = 0 on the ring): the heat-exchange
    // seed dJ/dg_i = seed_src beta, and in paper mode the implicit
    // T~ (1 + beta) of eq:albeg_ex
    if (a.beta && !n.ring) {
      Tt -= R(a.seed_src) * n.beta;
      if (!a.exact) Tt /= R(1) + n.beta;
    }
  }
  r_out = r;
  const R sux = sxx * n.ux + sxy * n.uy, suy = sxy * n.ux + syy * n.uy;
  Vx = R(3) * utx + R(9) * sux - R(3) * r * n.ux - A2 * dsx;
  Vy = R(3) * uty + R(9) * suy - R(3) * r * n.uy - A2 * dsy;
  // the Brinkman pairing of the sensitivity: 3 alpha' u.u~ (paper) or
  // alpha' u.V / (1 + alpha) with the undivided V (exact)
  pair = a.exact ? double(n.s) / 3.0 * (double(n.ux) * double(Vx) + double(n.uy) * double(Vy))
                 : double(n.ux) * double(utx) + double(n.uy) * double(uty);
  if (a.exact) {
    Vx *= n.s;
    Vy *= n.s;
  }
  adj_T = 0.0;
  if constexpr (TH) {
    const R qu = qx * n.ux + qy * n.uy;
    if (a.exact) {
      // exact: the transpose of the forward B c.grad_h T, -div_h (B q~)
      Th = Tt + R(3) * qu - dq;
      // the propagated Theta carries the force's dependence on the new
      // temperature, g beta . V / (1 + alpha), at interior nodes, and the
      // division by 1 + beta acts on it
      if (!n.ring) Th += R(g.gbx) * Vx + R(g.gby) * Vy;
      if (a.beta && !n.ring) Th /= R(1) + n.beta;
    } else {
      const R bq = n.dBx * qx + n.dBy * qy;
      Th = Tt + R(3) * qu - n.B * dq - bq;
    }
    adj_T = double(a.exact ? Th : Tt);
  }
}

// the sensitivity integrand 3 alpha' u.u~ - B' grad T . q~ of an interior
// node, with the heat source's beta' (T - 1)(w_J + T~) (the propagated Theta
// in exact mode). Exact mode at level 0 keeps only the conductivity term:
// alpha and beta act on the levels the steps produce, B on the equilibria used
template <typename R, bool TH>
__device__ inline double adj_sens(const AdjArgs<R>& a, double pair, double adj_T, R dA3, R dB,
                                  R dbeta, R T, R dTx, R dTy, R qx, R qy) {
#pragma clang fp contract(on)
  double v = a.sens_b_only ? 0.0 : double(dA3) * pair;
  if constexpr (TH) {
    const double tq = double(dTx) * double(qx) + double(dTy) * double(qy);
    v -= double(dB) * tq;
    if (a.beta && !a.sens_b_only) v += double(dbeta) * (double(T) - 1.0) * (a.seed_src + adj_T);
  }
  return v;
}

}  // namespace lks
