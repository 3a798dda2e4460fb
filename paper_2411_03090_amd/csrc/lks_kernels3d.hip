// D3Q19 kernels: the LKS step and the ALKS step of the three-dimensional
// extension (the equations of Sec. 2.3-2.5 with indices running over x, y,
// z, Sec. 2.1), on gfx950.
//
// LKS step: one z-marching kernel. A block owns 64 x 4 columns and walks
// through a range of z-planes with the state of two planes in LDS; per plane
// the tile and its ring leave a0 = drho - 3/2 u.u, P = 9/2 u u + A (grad u +
// grad u^T), G = 3 T u + B grad T in LDS, from which the columns form the
// equilibria f'_i^eq = w_i [a0 + 3 c.u + c.P.c], g_i^eq = w_i [T + c.G] (eq:feq2,
// eq:geq2) that reach them, and the plane behind is closed with the implicit
// Brinkman division and the face closures. Edge and corner nodes are copied by
// a small second kernel.
// ALKS step: the boundary nodes' moments (the pull of f~_i^eq = rho~ + c_i.V and
// g~_i^eq = Theta from x + c_i, eq:afeq, eq:ageq, the face least-squares completion
// and the local terms) go to a scratch; one z-march then forms the moments
// rho~, u~, s~, T~, q~ of the other nodes and from them V and Theta of the new
// level and the sensitivity 3 alpha' u.u~ - B' grad T.q~; a last kernel does the
// end planes. The same step as three passes over the grid (pull, faces,
// z-marching update) is kept beside it.
// Blocks are mapped so that each XCD works on a contiguous slab of nodes,
// keeping the neighbour planes of a block in that XCD's L2.
#include <hip/hip_runtime.h>

#include <climits>
#include <vector>

#include "lks_device.h"

namespace lks {
namespace {

__device__ constexpr int QX[19] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0};
__device__ constexpr int QY[19] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1};
__device__ constexpr int QZ[19] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1};
__device__ constexpr double QW[19] = {1.0 / 3,  1.0 / 18, 1.0 / 18, 1.0 / 18, 1.0 / 18,
                                      1.0 / 18, 1.0 / 18, 1.0 / 36, 1.0 / 36, 1.0 / 36,
                                      1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36,
                                      1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36};
// symmetric index of (a, b) into xx xy xz yy yz zz
__device__ constexpr int SI[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};

constexpr int NT3 = 256;
constexpr int FLOW_VELOCITY3 = 1;
constexpr int THERM_DIRICHLET3 = 1;
constexpr int TAG_J_INLET3 = 16, TAG_J_OUTLET3 = 32, TAG_PROBE3 = 64, TAG_SOLID3 = 128;

// node of this thread: the blocks of XCD x (blockIdx % 8) cover the x-th
// eighth of the node range
__device__ inline int node3(int N) {
  const int per = int(gridDim.x) / NXCD;
  const int lb = (int(blockIdx.x) % NXCD) * per + int(blockIdx.x) / NXCD;
  const int k = lb * NT3 + int(threadIdx.x);
  return k < N ? k : -1;
}
__device__ inline int logical_block() {
  const int per = int(gridDim.x) / NXCD;
  return (int(blockIdx.x) % NXCD) * per + int(blockIdx.x) / NXCD;
}

struct P3 {
  int i, j, l;
};
__device__ inline P3 decode(const Geo3& g, int k) {
  const int t = k / g.nx;
  return {k - t * g.nx, t % g.ny, t / g.ny};
}
__device__ inline int wrapc(int x, int n) { return x < 0 ? x + n : (x >= n ? x - n : x); }
// node at p + d; periodic axes wrap, the caller never steps past the end of
// a non-periodic axis
__device__ inline int nbr(const Geo3& g, P3 p, int dx, int dy, int dz) {
  int a = p.i + dx, b = p.j + dy, c = p.l + dz;
  if (g.periodic & 1) a = wrapc(a, g.nx);
  if (g.periodic & 2) b = wrapc(b, g.ny);
  if (g.periodic & 4) c = wrapc(c, g.nz);
  return (c * g.ny + b) * g.nx + a;
}
// coordinates at an end of a non-periodic axis; *o = 2 axis + (at the high
// end) of the last one found
__device__ inline int ends(const Geo3& g, P3 p, int* o) {
  int c = 0;
  *o = -1;
  if (!(g.periodic & 1)) {
    if (p.i == 0) { ++c; *o = 0; }
    else if (p.i == g.nx - 1) { ++c; *o = 1; }
  }
  if (!(g.periodic & 2)) {
    if (p.j == 0) { ++c; *o = 2; }
    else if (p.j == g.ny - 1) { ++c; *o = 3; }
  }
  if (!(g.periodic & 4)) {
    if (p.l == 0) { ++c; *o = 4; }
    else if (p.l == g.nz - 1) { ++c; *o = 5; }
  }
  return c;
}
// the node an edge or corner node copies from: inwards along y and z
__device__ inline P3 copy_src(const Geo3& g, P3 p) {
  P3 s = p;
  if (!(g.periodic & 2)) s.j = p.j == 0 ? 1 : (p.j == g.ny - 1 ? g.ny - 2 : p.j);
  if (!(g.periodic & 4)) s.l = p.l == 0 ? 1 : (p.l == g.nz - 1 ? g.nz - 2 : p.l);
  return s;
}

// derivative along axis ax: central inside or across a periodic axis,
// second-order one-sided at the ends of a non-periodic axis
template <typename R>
__device__ inline R dd(const Geo3& g, const R* f, P3 p, int k, int ax) {
  int c, n, per, step;
  if (ax == 0) { c = p.i; n = g.nx; per = g.periodic & 1; step = 1; }
  else if (ax == 1) { c = p.j; n = g.ny; per = g.periodic & 2; step = g.nx; }
  else { c = p.l; n = g.nz; per = g.periodic & 4; step = g.nx * g.ny; }
  if (c > 0 && c < n - 1) return R(0.5) * (f[k + step] - f[k - step]);
  if (per) {
    const int kp = c == n - 1 ? k - (n - 1) * step : k + step;
    const int km = c == 0 ? k + (n - 1) * step : k - step;
    return R(0.5) * (f[kp] - f[km]);
  }
  if (c == 0) return R(0.5) * (R(-3) * f[k] + R(4) * f[k + step] - f[k + 2 * step]);
  return R(0.5) * (R(3) * f[k] - R(4) * f[k - step] + f[k - 2 * step]);
}

__device__ inline double block_sum3(double v, double* red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  const int w = int(threadIdx.x) / 64, lane = int(threadIdx.x) % 64;
  if (lane == 0) red[w] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < NT3 / 64; ++i) s += red[i];
  return s;
}

// ---------------------------------------------------------------------------
// design coefficients and initial state
// ---------------------------------------------------------------------------
template <typename R>
__global__ __launch_bounds__(NT3) void coef3_kernel(Geo3 g, const uint8_t* __restrict__ mask,
                                                    const double* __restrict__ gamma, double amax,
                                                    double qa, double Kf, double Ks, double qk,
                                                    R* inv1pa, R* B, R* dA3, R* dB) {
  const int k = node3(g.N);
  if (k < 0) return;
  int o;
  if (ends(g, decode(g, k), &o)) {
    inv1pa[k] = R(1);
    B[k] = R(3.0 * (1.0 / 6.0 - Kf));
    dA3[k] = R(0);
    dB[k] = R(0);
    return;
  }
  const double gm = gamma[k];
  const double alpha = amax * qa * (1.0 - gm) / (qa + gm);
  const double dalpha = -amax * qa * (1.0 + qa) / ((qa + gm) * (qa + gm));
  const double K = Kf + (Ks - Kf) * qk * (1.0 - gm) / (qk + gm);
  const double dK = -(Ks - Kf) * qk * (1.0 + qk) / ((qk + gm) * (qk + gm));
  const bool solid = mask[k] & TAG_SOLID3;
  inv1pa[k] = R(1.0 / (1.0 + alpha));
  B[k] = R(3.0 * (1.0 / 6.0 - K));
  dA3[k] = solid ? R(0) : R(3.0 * dalpha);
  dB[k] = solid ? R(0) : R(-3.0 * dK);
}

template <typename R>
__global__ __launch_bounds__(NT3) void init3_kernel(Geo3 g, const uint8_t* __restrict__ mask,
                                                    const R* ubx, const R* uby, const R* ubz,
                                                    const R* Tb, double f0, R* d, R* ux, R* uy,
                                                    R* uz, R* T) {
  const int k = node3(g.N);
  if (k < 0) return;
  const P3 p = decode(g, k);
  int o;
  const int ne = ends(g, p, &o);
  const int m = mask[k];
  d[k] = R(0);
  const bool vel = ne == 1 && (m & 3) == FLOW_VELOCITY3;
  ux[k] = vel ? R(double(ubx[k]) * f0) : R(0);
  uy[k] = vel ? R(double(uby[k]) * f0) : R(0);
  uz[k] = vel ? R(double(ubz[k]) * f0) : R(0);
  if (g.thermal) {
    int kt = k;
    if (ne >= 2) {
      const P3 s = copy_src(g, p);
      kt = (s.l * g.ny + s.j) * g.nx + s.i;
    }
    T[k] = ((mask[kt] >> 2) & 3) == THERM_DIRICHLET3 ? Tb[kt] : R(0);
  }
}

// ---------------------------------------------------------------------------
// z-marching tiles
// ---------------------------------------------------------------------------
// A block owns a tile of ZX x ZY columns and marches through a range of
// z-planes. Each iteration loads one plane of the inputs (the tile plus a
// 2-node halo, rows coalesced) into LDS, so a field plane leaves HBM once per
// block and every neighbour gather reads LDS. The last tile along x or y is
// shifted to end at the domain end (its overlap with the previous tile is
// computed but not written), so one-sided differences at the ends stay
// inside the tile.
constexpr int ZX = 64, ZY = 4, ZT = ZX * ZY;
constexpr int SX = ZX + 4, NSR = SX * (ZY + 4);    // tile + 2-node halo
constexpr int CXN = ZX + 2, NCR = CXN * (ZY + 2);  // tile + 1-node halo
constexpr int SRL = (NSR + ZT - 1) / ZT;           // halo-region loads per thread
static_assert(ZT == NT3, "one block size for the 3D kernels");

__host__ __device__ inline int zchunks(const Geo3& g) { return g.zc; }
__host__ __device__ inline int ztiles(int n, int t) { return (n + t - 1) / t; }

struct ZTile {
  int x0, y0, w, h;  // origin and extent of the tile
  int xo, yo;        // first column and row the block writes
  int z0, z1;        // output planes
  int lb;            // logical block
};

// tile of this block; logical blocks run x fastest, then y, then z-chunk, and
// the blocks of XCD x (blockIdx % 8) take the x-th eighth of them
// (output planes: chunks of [zlo, zhi), nch of them when given)
__device__ inline bool ztile(const Geo3& g, ZTile& t, int zlo = 0, int zhi = -1, int nch = 0) {
  if (zhi < 0) zhi = g.nz;
  if (nch <= 0) nch = zchunks(g);
  const int ntx = ztiles(g.nx, ZX), nty = ztiles(g.ny, ZY);
  const int per = int(gridDim.x) / NXCD;
  t.lb = (int(blockIdx.x) % NXCD) * per + int(blockIdx.x) / NXCD;
  if (t.lb >= ntx * nty * nch) return false;
  const int ix = t.lb % ntx, iy = (t.lb / ntx) % nty, ic = t.lb / (ntx * nty);
  t.w = g.nx < ZX ? g.nx : ZX;
  t.h = g.ny < ZY ? g.ny : ZY;
  t.xo = ix * ZX;
  t.yo = iy * ZY;
  t.x0 = t.xo < g.nx - t.w ? t.xo : g.nx - t.w;
  t.y0 = t.yo < g.ny - t.h ? t.yo : g.ny - t.h;
  t.z0 = zlo + int((long long)ic * (zhi - zlo) / nch);
  t.z1 = zlo + int((long long)(ic + 1) * (zhi - zlo) / nch);
  return true;
}

// coordinate c of an axis of n nodes, wrapped on a periodic axis, -1 beyond a
// non-periodic one (c is at most 2 nodes outside, and n >= 3)
__device__ inline int axc(int c, int n, int per) {
  if (c < 0) return per ? c + n : -1;
  if (c >= n) return per ? c - n : -1;
  return c;
}
// -1 / +1 at the low / high end of a non-periodic axis, else 0
__device__ inline int endof(int c, int n, int per) {
  return per ? 0 : (c == 0 ? -1 : (c == n - 1 ? 1 : 0));
}
__device__ inline int zwrap(int s, int n) { return s < 0 ? s + n : (s >= n ? s - n : s); }

// a column of the tile or of its 1-node ring
struct ZNode {
  int on;      // the thread has this column
  int dx, dy;  // tile-local position, -1 .. w and -1 .. h
  int lds;     // index in the 2-node halo region
  int ci;      // index in the 1-node halo region
  int off;     // in-plane offset j nx + i, -1 off the domain
  int ex, ey;  // end flags of the column
};

__device__ inline ZNode znode(const Geo3& g, const ZTile& t, int dx, int dy, bool on) {
  ZNode n;
  n.on = on;
  n.dx = dx;
  n.dy = dy;
  n.lds = (dy + 2) * SX + dx + 2;
  n.ci = (dy + 1) * CXN + dx + 1;
  const int x = axc(t.x0 + dx, g.nx, g.periodic & 1), y = axc(t.y0 + dy, g.ny, g.periodic & 2);
  n.off = (x < 0 || y < 0) ? -1 : y * g.nx + x;
  n.ex = x < 0 ? 0 : endof(x, g.nx, g.periodic & 1);
  n.ey = y < 0 ? 0 : endof(y, g.ny, g.periodic & 2);
  return n;
}

// the ring column at position r of the ring around the tile: the row below
// the tile, the row above, the column left of it, the column right of it
__device__ inline ZNode zring_at(const Geo3& g, const ZTile& t, int r) {
  const int a = t.w + 2;
  int dx, dy;
  if (r < a) {
    dx = r - 1;
    dy = -1;
  } else if (r < 2 * a) {
    dx = r - a - 1;
    dy = t.h;
  } else if (r < 2 * a + t.h) {
    dx = -1;
    dy = r - 2 * a;
  } else {
    dx = t.w;
    dy = r - 2 * a - t.h;
  }
  const bool on = r >= 0 && r < 2 * a + 2 * t.h;
  return znode(g, t, on ? dx : 0, on ? dy : 0, on);
}
// the thread's ring column: three of the four waves take a third of the ring
// each, in consecutive positions (neighbouring lanes touch neighbouring LDS
// words); the wave left out rotates with the block, so that over the blocks
// resident on a CU the ring work is spread evenly over the SIMDs, and a wave
// runs the ring code only where it holds ring columns
__device__ inline ZNode zring(const Geo3& g, const ZTile& t) {
  const int per = (2 * (t.w + 2) + 2 * t.h + 2) / 3;  // at most 47 for 64 x 4 tiles
  const int lane = int(threadIdx.x) % 64, w = int(threadIdx.x) / 64;
  const int k = (w - (t.lb & 3) + 4) & 3;  // 0: the wave without ring columns
  return zring_at(g, t, (k > 0 && lane < per) ? (k - 1) * per + lane : -1);
}

// in-plane offsets of the thread's elements of the 2-node halo region; -1
// off the domain or beyond the tile's region
__device__ inline void zregion(const Geo3& g, const ZTile& t, int off[SRL]) {
#pragma unroll
  for (int r = 0; r < SRL; ++r) {
    const int e = int(threadIdx.x) + r * ZT;
    const int dx = e % SX - 2, dy = e / SX - 2;
    off[r] = -1;
    if (e < NSR && dx < t.w + 2 && dy < t.h + 2) {
      const int x = axc(t.x0 + dx, g.nx, g.periodic & 1);
      const int y = axc(t.y0 + dy, g.ny, g.periodic & 2);
      if (x >= 0 && y >= 0) off[r] = y * g.nx + x;
    }
  }
}

// ---------------------------------------------------------------------------
// LKS step
// ---------------------------------------------------------------------------
// Per plane s of the march, every column of the tile and its ring forms the
// coefficients a0 = drho - 3/2 u.u, P = 9/2 u u + A (grad u + grad u^T),
// G = 3 T u + B grad T of its node (eq:feq2, eq:geq2), all times w = 1/36, and
// leaves in LDS what its neighbours need of them. A column then forms the
// values f'_q = w_q [a0 + 3 c.u + c.P.c], g_q = w_q [T + c.G] that reach it from
// the nine columns x - c_q and adds them to the moments of the planes s - 1, s,
// s + 1 that it keeps in registers (the pull of f_i^eq(x - c_i)). Plane s - 1 is
// then complete. The three values that an in-plane neighbour e sends to the
// planes s and s +- 1 are 2 b, E + O, E - O (units of w) with
//   b = a0 + c.P.c + 3 c.u along e,  E = b + Pzz,  O = 3 uz + 2 c.P.ez,
// so the sums of a plane need 2 b, E and O of four neighbours and one value of
// each of the four diagonal ones; all that arrives from below has c_z = 1, so
// its u_z sum is its density sum. A source off the domain leaves zeros, so a
// face node's sums over the directions it receives are rho + sg (c_n . f) with
// n its normal.
// Bound by instructions. Forming all 19 values at the source and sending each
// behind a test of its target, with a branch for each difference, took 135 us
// on 256 x 128 x 128 in FP32 and 74 us on 97 x 61 x 53 in FP64; this way it is
// 75 and 41 us, the second 29 us in whole rounds of blocks. In the first 260 MB pass
// below the L2, 3.5 TB/s; a copy of that size reaches 5.3.
template <typename R>
struct alignas(2 * sizeof(R)) V2 {
  R x, y;
};
template <typename R>
struct alignas(16) V4 {
  R x, y, z, w;
};
template <typename R, bool TH>
struct FwdZLds {
  V4<R> st[2][NSR];  // u, T of planes s and s + 1
  // coefficients of the columns of the tile and its ring (1-node halo region):
  // 3 uz, Pzz, T, Gz; a0 + Pxx, 2 Pxz; a0 + Pyy, 2 Pyz; a0 + Pxx + Pyy, 2 Pxy;
  // 3 ux, Gx; 3 uy, Gy
  V4<R> z[NCR];
  V2<R> fx[NCR], fy[NCR], fd[NCR], gx[NCR], gy[NCR];
  double red[ZT / 64];
};

// moments of a column: planes s - 1 (complete but for what arrives from above)
// and s; the part of U_z from below is a density sum
template <typename R, bool TH>
struct FwdAcc {
  R r0, r1, Ux0, Ux1, Uy0, Uy1, Uz0, Uz1;
  R T0, T1, Qx0, Qx1, Qy0, Qy1, Qz0, Qz1;
};

// z difference of a field at plane s from its values at s - 1 (zp), s (fc)
// and s + 1 (zn); z2 is plane 2 (low end) or nz - 3 (high end)
template <typename R>
__device__ inline R dz3(int ez, R fc, R zp, R zn, R z2) {
#pragma clang fp contract(on)
  if (ez < 0) return R(0.5) * (R(-3) * fc + R(4) * zn - z2);
  if (ez > 0) return R(0.5) * (R(3) * fc - R(4) * zp + z2);
  return R(0.5) * (zn - zp);
}

// the node of a uniform plane pointer at byte offset o
template <typename T>
__device__ inline T at_b(const T* p, unsigned o) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(p) + o);
}

template <typename T>
__device__ inline void put_b(T* p, unsigned o, T x) {
  *reinterpret_cast<T*>(reinterpret_cast<char*>(p) + o) = x;
}

// x, formed anew by every loop iteration that uses it: without this the
// compiler keeps an address per field and column across the march (24 registers
// and then spills)
__device__ inline unsigned anew(unsigned x) {
  asm volatile("" : "+v"(x));
  return x;
}

// The second argument of a kernel whose first one is a Geo3, read anew through
// the scalar cache where it is used: a march has more field pointers than scalar
// registers, and spilled ones cost two vector instructions at each use.
template <typename A>
__device__ inline const __attribute__((address_space(4))) A* arg2() {
  using Bytes = const __attribute__((address_space(4))) char;
  constexpr size_t off = (sizeof(Geo3) + alignof(A) - 1) / alignof(A) * alignof(A);
  Bytes* p = (Bytes*)__builtin_amdgcn_kernarg_segment_ptr() + off;
  asm volatile("" : "+s"(p));
  return (const __attribute__((address_space(4))) A*)p;
}

// values of a source column that stay with it
template <typename R>
struct FwdOwn {
  R A, Pzz, Uz, T, Gz;
};

// coefficients of the node of column n at plane sw, left in LDS. zp holds u and
// T of plane sw - 1 and is advanced to plane sw.
template <typename R, bool TH>
__device__ inline void fwd_src(const Geo3& g, const Fwd3Args<R>& a, FwdZLds<R, TH>& L,
                               const ZNode& n, int cur, int sw, size_t nxy, R dk, R Bk, V4<R>& zp,
                               FwdOwn<R>& o) {
  const int i = n.lds;
  const int ez = endof(sw, g.nz, g.periodic & 4);
  const V4<R> c = L.st[cur][i], zn = L.st[cur ^ 1][i];
  const V4<R> xp = L.st[cur][i + 1], xm = L.st[cur][i - 1];
  const V4<R> yp = L.st[cur][i + SX], ym = L.st[cur][i - SX];
  auto cen = [](const V4<R>& p, const V4<R>& m) {
    return V4<R>{R(0.5) * (p.x - m.x), R(0.5) * (p.y - m.y), R(0.5) * (p.z - m.z),
                 TH ? R(0.5) * (p.w - m.w) : R(0)};
  };
  // second-order one-sided difference, f1 and f2 one and two steps inwards of
  // the low (e < 0) or high end
  auto one = [](int e, const V4<R>& f, const V4<R>& f1, const V4<R>& f2) {
    const R h = e < 0 ? R(-0.5) : R(0.5);
    return V4<R>{h * (R(3) * f.x - R(4) * f1.x + f2.x), h * (R(3) * f.y - R(4) * f1.y + f2.y),
                 h * (R(3) * f.z - R(4) * f1.z + f2.z),
                 TH ? h * (R(3) * f.w - R(4) * f1.w + f2.w) : R(0)};
  };
  V4<R> dx = cen(xp, xm), dy = cen(yp, ym), dz = cen(zn, zp);
  if (n.ex) dx = one(n.ex, c, L.st[cur][i - n.ex], L.st[cur][i - 2 * n.ex]);
  if (n.ey) dy = one(n.ey, c, L.st[cur][i - n.ey * SX], L.st[cur][i - 2 * n.ey * SX]);
  if (ez) {
    const size_t b2 = size_t(ez < 0 ? 2 : g.nz - 3) * nxy;
    const unsigned ob = anew(unsigned(n.off)) * unsigned(sizeof(R));
    const V4<R> z2{at_b(a.s0[1] + b2, ob), at_b(a.s0[2] + b2, ob), at_b(a.s0[3] + b2, ob),
                   TH ? at_b(a.s0[4] + b2, ob) : R(0)};
    dz = one(ez, c, ez < 0 ? zn : zp, z2);
  }
  zp = c;
  const R w = R(1.0 / 36), A2 = R(g.A / 18.0);
  const R A = w * (dk - R(1.5) * (c.x * c.x + c.y * c.y + c.z * c.z));
  const R h = R(0.125) * c.x;  // 9/2 w ux
  const R hy = R(0.125) * c.y, hz = R(0.125) * c.z;
  const R Pxx = h * c.x + A2 * dx.x, Pyy = hy * c.y + A2 * dy.y, Pzz = hz * c.z + A2 * dz.z;
  const R Pxy = R(2) * h * c.y + A2 * (dx.y + dy.x);
  const R Pxz = R(2) * h * c.z + A2 * (dx.z + dz.x);
  const R Pyz = R(2) * hy * c.z + A2 * (dy.z + dz.y);
  const R U = R(1.0 / 12);
  o.A = A;
  o.Pzz = Pzz;
  o.Uz = U * c.z;
  o.T = o.Gz = R(0);
  R Gx = R(0), Gy = R(0);
  if constexpr (TH) {
    const R t = U * c.w, b = w * Bk;
    o.T = w * c.w;
    Gx = t * c.x + b * dx.w;
    Gy = t * c.y + b * dy.w;
    o.Gz = t * c.z + b * dz.w;
  }
  const R axx = A + Pxx;
  const int ci = n.ci;
  L.z[ci] = V4<R>{o.Uz, Pzz, o.T, o.Gz};
  L.fx[ci] = V2<R>{axx, Pxz};
  L.fy[ci] = V2<R>{A + Pyy, Pyz};
  L.fd[ci] = V2<R>{axx + Pyy, Pxy};
  L.gx[ci] = V2<R>{U * c.x, Gx};
  L.gy[ci] = V2<R>{U * c.y, Gy};
}

// what column ci receives from plane s, added to its moments; the moments of
// plane s - 1 are then complete in A.*0
template <typename R, bool TH>
__device__ inline void fwd_recv(const FwdZLds<R, TH>& L, int ci, const FwdOwn<R>& o,
                                FwdAcc<R, TH>& A, R& r2, R& x2, R& y2, R& t2, R& qx2, R& qy2) {
  // neighbours that send along +x, -x, +y, -y
  const V4<R> zl = L.z[ci - 1], zr = L.z[ci + 1], zd = L.z[ci - CXN], zu = L.z[ci + CXN];
  const V2<R> fl = L.fx[ci - 1], fr = L.fx[ci + 1], fd = L.fy[ci - CXN], fu = L.fy[ci + CXN];
  const V2<R> gl = L.gx[ci - 1], gr = L.gx[ci + 1], gd = L.gy[ci - CXN], gu = L.gy[ci + CXN];
  const R bl = fl.x + gl.x, br = fr.x - gr.x, bd = fd.x + gd.x, bu = fu.x - gu.x;
  const R El = bl + zl.y, Er = br + zr.y, Ed = bd + zd.y, Eu = bu + zu.y;
  const R Ol = zl.x + fl.y, Or = zr.x - fr.y, Od = zd.x + fd.y, Ou = zu.x - fu.y;
  const R e = R(2) * (o.A + o.Pzz) + ((El + Er) + (Ed + Eu));
  const R od = R(2) * o.Uz + ((Ol + Or) + (Od + Ou));
  const R ex = El - Er, ey = Ed - Eu, ox = Ol - Or, oy = Od - Ou;
  r2 = e + od;
  x2 = ex + ox;
  y2 = ey + oy;
  const R rz = e - od;
  A.r0 += rz;
  A.Uz0 -= rz;
  A.Ux0 += ex - ox;
  A.Uy0 += ey - oy;
  A.r1 += R(12) * o.A + R(2) * ((bl + br) + (bd + bu));
  A.Ux1 += R(2) * (bl - br);
  A.Uy1 += R(2) * (bd - bu);
  if constexpr (TH) {
    const R hl = zl.z + gl.y, hr = zr.z - gr.y, hd = zd.z + gd.y, hu = zu.z - gu.y;
    const R hs = (hl + hr) + (hd + hu), hx = hl - hr, hy = hd - hu;
    const R Z = R(2) * o.Gz + ((zl.w + zr.w) + (zd.w + zu.w)), S = R(2) * o.T + hs;
    const R gx = zl.w - zr.w, gy = zd.w - zu.w;
    t2 = S + Z;
    qx2 = hx + gx;
    qy2 = hy + gy;
    const R tz = S - Z;
    A.T0 += tz;
    A.Qz0 -= tz;
    A.Qx0 += hx - gx;
    A.Qy0 += hy - gy;
    A.T1 += R(12) * o.T + R(2) * hs;
    A.Qx1 += R(2) * hx;
    A.Qy1 += R(2) * hy;
  }
  // (the reads below wait: all of them at once cost a wave per SIMD)
  __builtin_amdgcn_sched_barrier(0);
  // diagonal neighbours that send along ++, --, +-, -+
  const int c1 = ci - CXN - 1, c2 = ci + CXN + 1, c3 = ci + CXN - 1, c4 = ci - CXN + 1;
  const V2<R> d1 = L.fd[c1], d2 = L.fd[c2], d3 = L.fd[c3], d4 = L.fd[c4];
  const V2<R> x1 = L.gx[c1], x2_ = L.gx[c2], x3 = L.gx[c3], x4 = L.gx[c4];
  const V2<R> y1 = L.gy[c1], y2_ = L.gy[c2], y3 = L.gy[c3], y4 = L.gy[c4];
  {
    const R F1 = (d1.x + d1.y) + (x1.x + y1.x), F2 = (d2.x + d2.y) - (x2_.x + y2_.x);
    const R F3 = (d3.x - d3.y) + (x3.x - y3.x), F4 = (d4.x - d4.y) - (x4.x - y4.x);
    const R p = F1 - F2, m = F3 - F4;
    A.r1 += (F1 + F2) + (F3 + F4);
    A.Ux1 += p + m;
    A.Uy1 += p - m;
  }
  if constexpr (TH) {
    const R F1 = L.z[c1].z + (x1.y + y1.y), F2 = L.z[c2].z - (x2_.y + y2_.y);
    const R F3 = L.z[c3].z + (x3.y - y3.y), F4 = L.z[c4].z - (x4.y - y4.y);
    const R p = F1 - F2, m = F3 - F4;
    A.T1 += (F1 + F2) + (F3 + F4);
    A.Qx1 += p + m;
    A.Qy1 += p - m;
  }
}

// component ax of (v0, v1, v2)
template <typename R>
__device__ inline R pick3(int ax, R v0, R v1, R v2) {
  return (ax == 0 ? v0 : R(0)) + (ax == 1 ? v1 : R(0)) + (ax == 2 ? v2 : R(0));
}

// new-level values of a node from its moments: the implicit Brinkman
// division inside, the velocity / pressure closures and the temperature
// closure on faces; edge and corner nodes are copied afterwards
template <typename R, bool TH>
__device__ inline void fwd3_out(const Geo3& g, const Fwd3Args<R>& a, size_t plane, unsigned off,
                                int ex, int ey, int ez, int m, R s, R Tb, const R ubk[3],
                                double fac, R rho, const R U[3], R Ts, const R Q[3],
                                double& part) {
  const int ne = (ex != 0) + (ey != 0) + (ez != 0);
  if (ne >= 2) return;
  R d, u[3], T = R(0);
  if (!ne) {
    d = rho;
#pragma unroll
    for (int x = 0; x < 3; ++x) u[x] = U[x] * s;
    if constexpr (TH) T = ((m >> 2) & 3) == THERM_DIRICHLET3 ? Tb : Ts;
  } else {
    const int ax = ex ? 0 : (ey ? 1 : 2);
    const int sg = ex ? ex : (ey ? ey : ez);
    // components along the normal as masked sums (no indexing by ax, which
    // would move the register arrays to memory)
    const R Un = pick3(ax, U[0], U[1], U[2]);
    const R sn = rho + R(sg) * Un;  // S0 + 2 S+ over the received directions
    R un;
    if ((m & 3) == FLOW_VELOCITY3) {
#pragma unroll
      for (int x = 0; x < 3; ++x) u[x] = R(double(ubk[x]) * fac);
      un = R(sg) * pick3(ax, u[0], u[1], u[2]);
      d = sn - un;
    } else {
      const R dro = R(g.drho_out);
      d = dro;
      un = sn - dro;
#pragma unroll
      for (int x = 0; x < 3; ++x) u[x] = x == ax ? R(sg) * un : R(0);
    }
    if constexpr (TH) {
      const R Qn = pick3(ax, Q[0], Q[1], Q[2]);
      if (((m >> 2) & 3) == THERM_DIRICHLET3) T = Tb;
      // heat-flux face: Tb holds the flux qbar into the domain (0: adiabatic)
      else T = (Ts + R(sg) * Qn + Tb) / (R(1) + un);
    }
  }
  const unsigned ob = off * unsigned(sizeof(R));
  put_b(a.s1[0] + plane, ob, d);
  put_b(a.s1[1] + plane, ob, u[0]);
  put_b(a.s1[2] + plane, ob, u[1]);
  put_b(a.s1[3] + plane, ob, u[2]);
  if constexpr (TH) put_b(a.s1[4] + plane, ob, T);
  if (a.acc) {
    if (a.objective == 1) {
      if (m & TAG_PROBE3) part += double(u[0]) * double(T);
    } else {
      if (m & TAG_J_INLET3) part += double(d);
      if (m & TAG_J_OUTLET3) part -= double(d);
    }
  }
}

template <typename R, bool TH>
__global__ __launch_bounds__(ZT, sizeof(R) == 4 ? 4 : 2) void lks3z_kernel(Geo3 g, Fwd3Args<R> a) {
  __shared__ FwdZLds<R, TH> L;
  ZTile t;
  if (!ztile(g, t)) return;
  const int tid = int(threadIdx.x), lx = tid % ZX, ly = tid / ZX;
  const int pz = g.periodic & 4;
  const size_t nxy = size_t(g.nx) * size_t(g.ny);
  // byte offsets in a plane of the thread's elements of the 2-node halo region;
  // an element off the domain reads the plane's first node, which nothing uses
  unsigned roff[SRL];
  {
    int off[SRL];
    zregion(g, t, off);
#pragma unroll
    for (int r = 0; r < SRL; ++r)
      roff[r] = off[r] < 0 ? 0u : unsigned(off[r]) * unsigned(sizeof(R));
  }
  ZNode n0 = znode(g, t, lx, ly, lx < t.w && ly < t.h);
  ZNode n1 = zring(g, t);
  n1.on = n1.on && n1.off >= 0;
  const bool own = n0.on && t.x0 + lx >= t.xo && t.y0 + ly >= t.yo;
  unsigned ob0 = unsigned(n0.off) * unsigned(sizeof(R));
  unsigned ob1 = unsigned(n1.off) * unsigned(sizeof(R));
  // columns off the domain send nothing: their entries stay zero
  for (int e = tid; e < NCR; e += ZT) {
    L.z[e] = V4<R>{R(0), R(0), R(0), R(0)};
    L.fx[e] = L.fy[e] = L.fd[e] = L.gx[e] = L.gy[e] = V2<R>{R(0), R(0)};
  }
  // source planes: one beyond the output range on each side where it exists
  const int sb = (t.z0 == 0 && !pz) ? 0 : t.z0 - 1;
  const int se = (t.z1 == g.nz && !pz) ? g.nz - 1 : t.z1;
  auto has = [&](int s) { return pz || (s >= 0 && s < g.nz); };
  auto plane = [&](int s) { return size_t(zwrap(s, g.nz)) * nxy; };
  V4<R> v[SRL];
  auto load = [&](int s) {
    const size_t b = plane(s);
    const R *F1 = a.s0[1] + b, *F2 = a.s0[2] + b, *F3 = a.s0[3] + b;
    const R* F4 = TH ? a.s0[4] + b : F1;
#pragma unroll
    for (int r = 0; r < SRL; ++r)
      if ((r + 1) * ZT <= NSR || tid + r * ZT < NSR) {
        v[r].x = at_b(F1, roff[r]);
        v[r].y = at_b(F2, roff[r]);
        v[r].z = at_b(F3, roff[r]);
        v[r].w = TH ? at_b(F4, roff[r]) : R(0);
      }
  };
  auto store = [&](int slot) {
#pragma unroll
    for (int r = 0; r < SRL; ++r)
      if ((r + 1) * ZT <= NSR || tid + r * ZT < NSR) L.st[slot][tid + r * ZT] = v[r];
  };
  auto zload = [&](int s, unsigned ob) {
    const size_t b = plane(s);
    return V4<R>{at_b(a.s0[1] + b, ob), at_b(a.s0[2] + b, ob), at_b(a.s0[3] + b, ob),
                 TH ? at_b(a.s0[4] + b, ob) : R(0)};
  };
  load(sb);
  store(0);
  if (has(sb + 1)) load(sb + 1);
  V4<R> zp0{R(0), R(0), R(0), R(0)}, zp1 = zp0;
  if (has(sb - 1)) {
    if (n0.on) zp0 = zload(sb - 1, ob0);
    if (n1.on) zp1 = zload(sb - 1, ob1);
  }
  // per-node inputs one iteration ahead: drho and B of the source nodes,
  // class, Brinkman factor and prescribed temperature of the output node; the
  // prescribed velocity of a velocity face node is read with the rest (not
  // waiting for its class), and the level's inflow factor once
  const double fac = a.ufac[a.level_out];
  R dd0, dd1, b0 = R(0), b1 = R(0), ip, tb = R(0), ub[3];
  int mk;
  auto node_in = [&](int s) {
    const size_t b = plane(s);
    dd0 = dd1 = R(0);
    if (n0.on) {
      dd0 = at_b(a.s0[0] + b, ob0);
      if constexpr (TH) b0 = at_b(a.B + b, ob0);
    }
    if (n1.on) {
      dd1 = at_b(a.s0[0] + b, ob1);
      if constexpr (TH) b1 = at_b(a.B + b, ob1);
    }
    const int p = s - 1;
    mk = 0;
    ip = ub[0] = ub[1] = ub[2] = R(0);
    if (p >= t.z0 && own) {
      const size_t q = size_t(p) * nxy;
      mk = at_b(a.mask + q, unsigned(n0.off));
      ip = at_b(a.inv1pa + q, ob0);
      if constexpr (TH) tb = at_b(a.Tb + q, ob0);
      if (n0.ex || n0.ey || endof(p, g.nz, pz))
#pragma unroll
        for (int x = 0; x < 3; ++x) ub[x] = at_b(a.ub[x] + q, ob0);
    }
  };
  node_in(sb);
  FwdAcc<R, TH> A = {};
  double part = 0.0;
  for (int s = sb; s <= se; ++s) {
    const int cur = (s - sb) & 1;
    ob0 = anew(ob0);
    ob1 = anew(ob1);
    n0.off = int(anew(unsigned(n0.off)));
    n1.lds = int(anew(unsigned(n1.lds)));
    n0.lds = int(anew(unsigned(n0.lds)));
#pragma unroll
    for (int r = 0; r < SRL; ++r) roff[r] = anew(roff[r]);
    if (has(s + 1)) store(cur ^ 1);
    lds_barrier();
    if (has(s + 2)) load(s + 2);
    const R cd0 = dd0, cd1 = dd1, cb0 = b0, cb1 = b1, cip = ip, ctb = tb;
    const R cub[3] = {ub[0], ub[1], ub[2]};
    const int cmk = mk;
    if (s + 1 <= se) node_in(s + 1);
    const int sw = zwrap(s, g.nz);
    FwdOwn<R> own_v, ring_v;
    if (n1.on) fwd_src<R, TH>(g, a, L, n1, cur, sw, nxy, cd1, cb1, zp1, ring_v);
    if (n0.on) fwd_src<R, TH>(g, a, L, n0, cur, sw, nxy, cd0, cb0, zp0, own_v);
    lds_barrier();
    R r2 = R(0), x2 = R(0), y2 = R(0), t2 = R(0), qx2 = R(0), qy2 = R(0);
    if (n0.on) fwd_recv<R, TH>(L, n0.ci, own_v, A, r2, x2, y2, t2, qx2, qy2);
    const int p = s - 1;
    if (own && p >= t.z0 && p < t.z1) {
      const R U[3] = {A.Ux0, A.Uy0, A.Uz0}, Q[3] = {A.Qx0, A.Qy0, A.Qz0};
      fwd3_out<R, TH>(g, a, size_t(p) * nxy, unsigned(n0.off), n0.ex, n0.ey, endof(p, g.nz, pz),
                      cmk, cip, ctb, cub, fac, A.r0, U, A.T0, Q, part);
    }
    A.r0 = A.r1;
    A.Ux0 = A.Ux1;
    A.Uy0 = A.Uy1;
    A.Uz0 = A.Uz1;
    A.r1 = A.Uz1 = r2;
    A.Ux1 = x2;
    A.Uy1 = y2;
    if constexpr (TH) {
      A.T0 = A.T1;
      A.Qx0 = A.Qx1;
      A.Qy0 = A.Qy1;
      A.Qz0 = A.Qz1;
      A.T1 = A.Qz1 = t2;
      A.Qx1 = qx2;
      A.Qy1 = qy2;
    }
  }
  if (!pz && se == g.nz - 1 && own) {
    const size_t q = size_t(g.nz - 1) * nxy;
    const R ubk[3] = {at_b(a.ub[0] + q, ob0), at_b(a.ub[1] + q, ob0), at_b(a.ub[2] + q, ob0)};
    const R U[3] = {A.Ux0, A.Uy0, A.Uz0}, Q[3] = {A.Qx0, A.Qy0, A.Qz0};
    fwd3_out<R, TH>(g, a, q, unsigned(n0.off), n0.ex, n0.ey, 1, at_b(a.mask + q, unsigned(n0.off)),
                    at_b(a.inv1pa + q, ob0), TH ? at_b(a.Tb + q, ob0) : R(0), ubk, fac, A.r0, U,
                    A.T0, Q, part);
  }
  if (a.acc) {
    const double s = block_sum3(part, L.red);
    if (tid == 0) a.acc[t.lb] += s;
  }
}

// edge and corner nodes: density and temperature of the node one step
// inwards along y and z, zero velocity
template <typename R, bool TH>
__global__ __launch_bounds__(NT3) void copy3_kernel(Geo3 g, const int* __restrict__ list, int n,
                                                    R* d, R* ux, R* uy, R* uz, R* T) {
  const int i = int(blockIdx.x) * NT3 + int(threadIdx.x);
  if (i >= n) return;
  const int k = list[i];
  const P3 s = copy_src(g, decode(g, k));
  const int ks = (s.l * g.ny + s.j) * g.nx + s.i;
  d[k] = d[ks];
  ux[k] = R(0);
  uy[k] = R(0);
  uz[k] = R(0);
  if constexpr (TH) T[k] = T[ks];
}

// ---------------------------------------------------------------------------
// ALKS step
// ---------------------------------------------------------------------------
// Sums over the nine columns x + e around a column of one plane's rho~, V and
// Theta, in units of w = 1/36. A node of this plane takes f~ of its in-plane
// directions from them (I*), the nodes of the planes below and above take
// f~ = E +- Vz of the five directions with c_z = +-1 (E = rho~ + e.V): p* goes to
// the plane below (c_z = 1), m* to the plane above. All their values have the
// same c_z, so three sums give rho~, u~, s~zz, s~xz and s~yz of them; g~ does not
// depend on c and its sums serve both planes.
template <typename R>
struct AdjSums {
  R I0, Ix, Iy, Ixx, Iyy, Ixy;
  R pt, px, py, pxx, pyy, mt, mx, my, mxx, myy;
  R G0, Gx, Gy, gt, gx, gy;
};
// at(1 + dx, 1 + dy): rho~, Vx, Vy, Vz of a column; th: its Theta
template <typename R, bool TH, typename AT, typename GT>
__device__ inline void adj_sums(const AT& at, const GT& th, AdjSums<R>& o) {
#pragma clang fp contract(on)
  const V4<R> c = at(1, 1), r = at(2, 1), l = at(0, 1), u = at(1, 2), d = at(1, 0);
  const R er = r.x + r.y, el = l.x - l.y, eu = u.x + u.z, ed = d.x - d.z;
  const R sx = er + el, sy = eu + ed, dx = er - el, dy = eu - ed, S = sx + sy;
  const R zx = r.w + l.w, zy = u.w + d.w, vx = r.w - l.w, vy = u.w - d.w;
  const R te = R(2) * c.x + S, to = R(2) * c.w + (zx + zy);
  o.pt = te + to;
  o.mt = te - to;
  o.px = dx + vx;
  o.mx = dx - vx;
  o.py = dy + vy;
  o.my = dy - vy;
  o.pxx = sx + zx;
  o.mxx = sx - zx;
  o.pyy = sy + zy;
  o.myy = sy - zy;
  // (the reads below wait, here and further down: all at once they cost the
  // registers of a wave per SIMD)
  __builtin_amdgcn_sched_barrier(0);
  const V4<R> a = at(2, 2), b = at(0, 0), e = at(2, 0), f = at(0, 2);
  const R f1 = a.x + (a.y + a.z), f2 = b.x - (b.y + b.z);
  const R f3 = e.x + (e.y - e.z), f4 = f.x - (f.y - f.z);
  const R s1 = f1 + f2, s2 = f3 + f4, d1 = f1 - f2, d2 = f3 - f4, D = s1 + s2;
  const R i0 = R(2) * S + D;
  o.I0 = R(12) * c.x + i0;
  o.Ix = R(2) * dx + (d1 + d2);
  o.Iy = R(2) * dy + (d1 - d2);
  o.Ixx = R(2) * sx + D;
  o.Iyy = R(2) * sy + D;
  o.Ixy = s1 - s2;
  o.G0 = o.Gx = o.Gy = o.gt = o.gx = o.gy = R(0);
  if constexpr (TH) {
    __builtin_amdgcn_sched_barrier(0);
    const R t0 = th(1, 1), tr = th(2, 1), tl = th(0, 1), tu = th(1, 2), td = th(1, 0);
    const R T = (tr + tl) + (tu + td);
    o.gt = R(2) * t0 + T;
    o.gx = tr - tl;
    o.gy = tu - td;
    const R g1 = th(2, 2), g2 = th(0, 0), g3 = th(2, 0), g4 = th(0, 2);
    const R p = g1 - g2, m = g3 - g4;
    const R q0 = R(2) * T + ((g1 + g2) + (g3 + g4));
    o.G0 = R(12) * t0 + q0;
    o.Gx = R(2) * o.gx + (p + m);
    o.Gy = R(2) * o.gy + (p - m);
  }
}
// what a node of a plane keeps until the plane above comes: its in-plane sums
// with what the plane below sent
template <typename R>
struct AdjPart {
  R I0, Ix, Iy, xx, yy, xy, mt, mx, my, T, qx, qy, gm;
};
template <typename R>
__device__ inline AdjPart<R> adj_part(const AdjSums<R>& o, R mt, R mx, R my, R mxx, R myy, R gt,
                                      R gx, R gy) {
  return {o.I0, o.Ix, o.Iy, o.Ixx + mxx, o.Iyy + myy, o.Ixy, mt, mx, my,
          o.G0 + gt, o.Gx + gx, o.Gy + gy, gt};
}
// raw moments of the 19 pulled values: rho~, u~ (3), s~ xx xy xz yy yz zz, T~,
// q~ (3); o: the sums of the plane above
template <typename R, bool TH>
__device__ inline void adj_close(const AdjPart<R>& c, const AdjSums<R>& o, R M[14]) {
  const R w = R(1.0 / 36);
  M[0] = w * (c.I0 + (c.mt + o.pt));
  M[1] = w * (c.Ix + (c.mx + o.px));
  M[2] = w * (c.Iy + (c.my + o.py));
  M[3] = w * (o.pt - c.mt);
  M[4] = w * (c.xx + o.pxx);
  M[5] = w * c.xy;
  M[6] = w * (o.px - c.mx);
  M[7] = w * (c.yy + o.pyy);
  M[8] = w * (o.py - c.my);
  M[9] = w * (o.pt + c.mt);
  M[10] = TH ? w * (c.T + o.gt) : R(0);
  M[11] = TH ? w * (c.qx + o.gx) : R(0);
  M[12] = TH ? w * (c.qy + o.gy) : R(0);
  M[13] = TH ? w * (o.gt - c.gm) : R(0);
}

// Least-squares completion of a face node with orientation o (see FaceFillT)
// and the moments of the completed set. In the node's frame (outward normal n
// along axis o / 2, tangents t1, t2 along the next two axes) the known
// populations are f[0] rest, f[1..4] t1, -t1, t2, -t2, f[5..8] t1 + t2, t1 - t2,
// -t1 + t2, -t1 - t2, f[9] -n, f[10..13] -n + t1, -n - t1, -n + t2, -n - t2.
// The symmetries of the square split the 5 x 14 map into sums of products
// with 15 coefficients, one operator for the six faces.
template <typename R, bool TH>
__device__ inline void face_fill(const Adj3Args<R>& a, int o, int m, R un, R Tn, const R f[14],
                                 const R gq[14], R M[14]) {
#pragma clang fp contract(on)
  const R w0 = R(1.0 / 3), w1 = R(1.0 / 18), w2 = R(1.0 / 36);
  const auto* op = as_scalar(a.ops);
  const bool diri = ((m >> 2) & 3) == THERM_DIRICHLET3;
  R kappa = R(0), Tt = R(0), qn = R(0), q1 = R(0), q2 = R(0);
  if constexpr (TH) {
    const R ea = (gq[1] + gq[2]) + (gq[3] + gq[4]), ed = (gq[5] + gq[8]) + (gq[6] + gq[7]);
    const R eb = (gq[10] + gq[11]) + (gq[12] + gq[13]);
    const R t1 = gq[1] - gq[2], t2 = gq[3] - gq[4], i1 = gq[10] - gq[11], i2 = gq[12] - gq[13];
    const R d1 = (gq[5] - gq[8]) + (gq[6] - gq[7]), d2 = (gq[5] - gq[8]) - (gq[6] - gq[7]);
    auto even = [&](const auto& c) {
      return c[0] * gq[0] + c[1] * ea + c[2] * ed + c[3] * gq[9] + c[4] * eb;
    };
    auto odd = [&](const auto& c, R t, R d, R i) { return c[0] * t + c[1] * d + c[2] * i; };
    R Y, X1, X2;
    if (diri) {
      Y = even(op->Dy);
      X1 = odd(op->Dx, t1, d1, i1);
      X2 = odd(op->Dx, t2, d2, i2);
    } else {
      const R na = even(op->ka), ne = even(op->ke);
      const R den = op->A0 - R(2) * un * op->A1 + un * un * op->A2;
      kappa = (un * ne - na) / den;
      Y = even(op->Gy);
      Y = Y - kappa * (op->Hc - un * op->H1);
      X1 = odd(op->Gx, t1, d1, i1);
      X2 = odd(op->Gx, t2, d2, i2);
    }
    const R in = w1 * gq[9] + w2 * eb;
    Tt = w0 * gq[0] + w1 * ea + w2 * ed + in + Y;
    qn = Y - in;
    q1 = w1 * t1 + w2 * (d1 + i1) + X1;
    q2 = w1 * t2 + w2 * (d2 + i2) + X2;
  }
  // boundary seed of the pressure-drop objective per unit boundary pressure
  R s = R(0);
  if (m & TAG_J_INLET3) s += R(a.seed_dp);
  if (m & TAG_J_OUTLET3) s -= R(a.seed_dp);
  const R kT = kappa * Tn;
  const R s1 = f[1] + f[2], s2 = f[3] + f[4], ea = s1 + s2;
  const R dp = f[5] + f[8], dm = f[6] + f[7], ed = dp + dm;
  const R b1 = f[10] + f[11], b2 = f[12] + f[13], eb = b1 + b2;
  const R t1 = f[1] - f[2], t2 = f[3] - f[4], i1 = f[10] - f[11], i2 = f[12] - f[13];
  const R d1 = (f[5] - f[8]) + (f[6] - f[7]), d2 = (f[5] - f[8]) - (f[6] - f[7]);
  R Y = R(0), Zs = R(0), Zd = R(0), X1 = R(0), X2 = R(0);
  const int v = (m & 3) == FLOW_VELOCITY3 ? 0 : 1;
#pragma nounroll
  for (int t = 0; t < 2; ++t) {
    if (!__any(v == t)) continue;
    auto even = [&](const auto& c) {
      return c[0] * f[0] + c[1] * ea + c[2] * ed + c[3] * f[9] + c[4] * eb;
    };
    auto odd = [&](R x, R d, R i) {
      return op->X[t][0] * x + op->X[t][1] * d + op->X[t][2] * i;
    };
    const R y = even(op->Y[t]) + op->Ys[t] * s + op->Yk[t] * kT;
    const R zs = even(op->Zs[t]) + op->Zss[t] * s + op->Zsk[t] * kT;
    const R zd = op->Zd[t][0] * (s1 - s2) + op->Zd[t][1] * (b1 - b2);
    const R x1 = odd(t1, d1, i1), x2 = odd(t2, d2, i2);
    Y = v == t ? y : Y;
    Zs = v == t ? zs : Zs;
    Zd = v == t ? zd : Zd;
    X1 = v == t ? x1 : X1;
    X2 = v == t ? x2 : X2;
  }
  const R in = w1 * f[9] + w2 * eb;
  const R r = w0 * f[0] + w1 * ea + w2 * ed + in + Y;
  const R Un = Y - in, U1 = w1 * t1 + w2 * (d1 + i1) + X1, U2 = w1 * t2 + w2 * (d2 + i2) + X2;
  const R snn = in + Y;
  const R s11 = w1 * s1 + w2 * (ed + b1) + R(0.5) * (Zs + Zd);
  const R s22 = w1 * s2 + w2 * (ed + b2) + R(0.5) * (Zs - Zd);
  const R sn1 = X1 - w2 * i1, sn2 = X2 - w2 * i2, s12 = w2 * (dp - dm);
  // back to x, y, z: t1 and t2 are the axes after the normal's
  const int ax = o >> 1;
  const R sg = (o & 1) ? R(1) : R(-1);
  auto pick = [&](R x0, R x1, R x2) { return ax == 0 ? x0 : (ax == 1 ? x1 : x2); };
  M[0] = r;
  M[1] = pick(sg * Un, U2, U1);
  M[2] = pick(U1, sg * Un, U2);
  M[3] = pick(U2, U1, sg * Un);
  M[4] = pick(snn, s22, s11);
  M[5] = pick(sg * sn1, sg * sn2, s12);
  M[6] = pick(sg * sn2, s12, sg * sn1);
  M[7] = pick(s11, snn, s22);
  M[8] = pick(s12, sg * sn1, sg * sn2);
  M[9] = pick(s22, s11, snn);
  M[10] = Tt;
  M[11] = pick(sg * qn, q2, q1);
  M[12] = pick(q1, sg * qn, q2);
  M[13] = pick(q2, q1, sg * qn);
}

// local terms of the adjoint moments: the probe seed, the prescribed
// temperature inside, the T q~ coupling and the Brinkman factor of u~
template <typename R, bool TH>
__device__ inline void adj_local(const Adj3Args<R>& a, int m, int ne, R Tn, R s, R M[14], R u0) {
#pragma clang fp contract(on)
  if constexpr (TH) {
    const bool probe = (m & TAG_PROBE3) && a.seed_heat != 0.0;
    if (probe) M[10] -= R(a.seed_heat) * u0;
    // a prescribed temperature does not depend on the arriving populations:
    // zero thermal adjoint inside (both modes) and on faces (exact mode)
    if (((m >> 2) & 3) == THERM_DIRICHLET3 && (!ne || a.exact)) {
      M[10] = R(0);
      M[11] = M[12] = M[13] = R(0);
    }
#pragma unroll
    for (int x = 0; x < 3; ++x) M[1 + x] += Tn * M[11 + x];
    if (probe) M[1] -= R(a.seed_heat / 3.0) * Tn;
  }
#pragma unroll
  for (int x = 0; x < 3; ++x) M[1 + x] *= s;
}

// moments of the interior node p
template <typename R, bool TH>
__device__ inline void alks3_node(const Geo3& g, const Adj3Args<R>& a, P3 p, int k, R M[14]) {
  AdjSums<R> below, here, above;
  auto plane = [&](int dz, AdjSums<R>& o) {
    auto at = [&](int dx, int dy) {
      const int z = nbr(g, p, dx - 1, dy - 1, dz);
      return V4<R>{a.p0[0][z], a.p0[1][z], a.p0[2][z], a.p0[3][z]};
    };
    auto th = [&](int dx, int dy) { return TH ? a.p0[4][nbr(g, p, dx - 1, dy - 1, dz)] : R(0); };
    adj_sums<R, TH>(at, th, o);
  };
  plane(-1, below);
  plane(0, here);
  plane(1, above);
  adj_close<R, TH>(adj_part(here, below.mt, below.mx, below.my, below.mxx, below.myy, below.gt,
                            below.gx, below.gy),
                   above, M);
  const int m = a.mask[k];
  const R Tn = TH ? a.T[k] : R(0);
  // exact mode: u~ stays undivided; the update pass divides V instead
  const bool probe = TH && (m & TAG_PROBE3) && a.seed_heat != 0.0;
  adj_local<R, TH>(a, m, 0, Tn, a.exact ? R(1) : a.inv1pa[k], M, probe ? a.u[0][k] : R(0));
}

// ALKS pass 1 at the interior nodes; the boundary nodes are left to
// alks3_face_kernel, so the face completion does not diverge inside the
// waves of the rows that end on an x face
template <typename R, bool TH>
__global__ __launch_bounds__(NT3) void alks3_pull_kernel(Geo3 g, Adj3Args<R> a) {
  const int k = node3(g.N);
  if (k < 0) return;
  const P3 p = decode(g, k);
  int o;
  if (ends(g, p, &o)) return;
  R mom[14];
  alks3_node<R, TH>(g, a, p, k, mom);
  const size_t N = size_t(g.N);
  constexpr int NM = TH ? 14 : 10;
#pragma unroll
  for (int c = 0; c < NM; ++c) a.m[c * N + k] = mom[c];
}

// Tiles of the face nodes: a block takes FP x FQ nodes of one face, p along the
// axis with the smaller stride (64 x 4 where that is x, whose rows are contiguous,
// 16 x 16 on the x faces). The face nodes of an axis: all of a periodic one, else
// those that are not at its ends.
struct FaceTiles {
  int np, nq;  // face nodes along p and q
  int tp, tq;  // tiles
};
__host__ __device__ inline FaceTiles face_tiles(const Geo3& g, int ax) {
  const int n[3] = {g.nx - ((g.periodic & 1) ? 0 : 2), g.ny - ((g.periodic & 2) ? 0 : 2),
                    g.nz - ((g.periodic & 4) ? 0 : 2)};
  FaceTiles t;
  t.np = ax == 0 ? n[1] : n[0];
  t.nq = ax == 2 ? n[1] : n[2];
  const int FP = ax == 0 ? 16 : 64, FQ = NT3 / FP;
  t.tp = (t.np + FP - 1) / FP;
  t.tq = (t.nq + FQ - 1) / FQ;
  return t;
}

// Where the scratch of the fused step holds the moments of an x-face node (end
// flag ex, row j) of plane l, in its plane: in a row of the faces' own where the
// march leaves the plane's interior free (it uses that of planes 1, 2, nz-3 and
// nz-2). At the node's own place, a row away from the next one, each of the 14
// values would dirty a line of its own: on 256 x 128 x 128 the face pass took 22.8
// us and the march 123.6, packed 17.9 and 107.7. Not in FP64, whose march has no
// registers left for the second address (97 x 61 x 53: face pass 11.9 -> 10.4 us,
// march 41.2 -> 43.5).
template <typename R>
__device__ inline bool xface_packed(const Geo3& g, int l) {
  return sizeof(R) == 4 && g.fused && g.nx >= 8 && g.ny >= 8 &&
         ((g.periodic & 4) || (l >= 3 && l <= g.nz - 4));
}
__device__ inline int xface_row(const Geo3& g, int ex, int j) {
  return g.nx + (ex > 0 ? g.ny : 0) + j;
}

// ALKS pass 1 at the boundary nodes: blocks of face tiles (two faces of each
// non-periodic axis), then the host-built list of the edge and corner nodes that
// copy the moments of an interior node (those that copy a face node's are written
// with it; all of them lie on the x faces).
// A tile's rho~, V and Theta of the face plane and the plane inwards (all that
// the 14 known populations need) pass through LDS: on the x faces, where every
// node has a cache line of its own, the block reads each line it needs once and
// not once per population. Bound by latency: 48 us on 256 x 128 x 128 in FP32 (160k
// boundary nodes) and 19 us on 97 x 61 x 53 in FP64 with 50 reads per node, 23 and
// 12 us this way.
template <typename R, bool TH>
__global__ __launch_bounds__(NT3) void alks3_face_kernel(Geo3 g, Adj3Args<R> a) {
  constexpr int NM = TH ? 14 : 10;
  constexpr int NREG = (64 + 2) * (4 + 2);  // tile with a 1-node halo, the larger one
  // face plane: rho~, V1, V2, Theta; plane inwards: rho~, Vn, V1, V2, Theta
  __shared__ R L[TH ? 9 : 7][NREG];
  const int tid = int(threadIdx.x);
  const size_t N = size_t(g.N);
  int b = int(blockIdx.x), ax = 0, face = -1;
  FaceTiles ft{};
  for (; ax < 3; ++ax) {
    if ((g.periodic >> ax) & 1) continue;
    ft = face_tiles(g, ax);
    const int nt = ft.tp * ft.tq;
    if (b < 2 * nt) {
      face = b / nt;
      b -= face * nt;
      break;
    }
    b -= 2 * nt;
  }
  if (face < 0) {
    const int t = b * NT3 + tid;
    if (t >= a.nface) return;
    const int k = a.face[t];
    const P3 s = copy_src(g, decode(g, k));
    R mom[14];
    alks3_node<R, TH>(g, a, s, (s.l * g.ny + s.j) * g.nx + s.i, mom);
#pragma unroll
    for (int c = 0; c < NM; ++c) a.m[c * N + k] = mom[c];
    return;
  }
  const int sg = face ? 1 : -1;
  const int FP = ax == 0 ? 16 : 64, FQ = NT3 / FP, PW = FP + 2;
  // axes p, q: extents, strides and periodicity
  const int ap = ax == 0 ? 1 : 0, aq = ax == 2 ? 1 : 2;
  const int st[3] = {1, g.nx, g.nx * g.ny}, n3[3] = {g.nx, g.ny, g.nz};
  auto at3 = [](const int (&x)[3], int e) { return e == 0 ? x[0] : (e == 1 ? x[1] : x[2]); };
  const int Np = at3(n3, ap), Nq = at3(n3, aq), sp = at3(st, ap), sq = at3(st, aq);
  const int perp = (g.periodic >> ap) & 1, perq = (g.periodic >> aq) & 1;
  const int sn = at3(st, ax), kn = face ? (at3(n3, ax) - 1) * sn : 0;
  const int p0 = (b % ft.tp) * FP, q0 = (b / ft.tp) * FQ;  // within the face nodes
  const int lop = perp ? 0 : 1, loq = perq ? 0 : 1;
  // the node of this thread
  const int lp = tid % FP, lq = tid / FP;
  const bool on = p0 + lp < ft.np && q0 + lq < ft.nq;
  const int cp = p0 + lp + lop, cq = q0 + lq + loq;
  const int k = on ? kn + cp * sp + cq * sq : 0;
  const R* Vn = ax == 0 ? a.p0[1] : (ax == 1 ? a.p0[2] : a.p0[3]);
  const R* V1 = ax == 0 ? a.p0[2] : (ax == 1 ? a.p0[3] : a.p0[1]);
  const R* V2 = ax == 0 ? a.p0[3] : (ax == 1 ? a.p0[1] : a.p0[2]);
#pragma unroll
  for (int r = 0; r < (NREG + NT3 - 1) / NT3; ++r) {
    const int e = tid + r * NT3;
    if (e >= PW * (FQ + 2)) continue;
    // wrapped on a periodic axis; positions beyond the last node are not used
    const int i = p0 + e % PW - 1 + lop, j = q0 + e / PW - 1 + loq;
    const int ci = i < 0 ? i + Np : (i >= Np ? (perp ? (i - Np) % Np : Np - 1) : i);
    const int cj = j < 0 ? j + Nq : (j >= Nq ? (perq ? (j - Nq) % Nq : Nq - 1) : j);
    const int z = kn + ci * sp + cj * sq, y = z - sg * sn;
    L[0][e] = a.p0[0][z];
    L[1][e] = V1[z];
    L[2][e] = V2[z];
    L[3][e] = a.p0[0][y];
    L[4][e] = Vn[y];
    L[5][e] = V1[y];
    L[6][e] = V2[y];
    if constexpr (TH) {
      L[TH ? 7 : 0][e] = a.p0[4][z];
      L[TH ? 8 : 0][e] = a.p0[4][y];
    }
  }
  const int m = a.mask[k];
  const R Tn = TH ? a.T[k] : R(0);
  const R* us = ax == 0 ? a.u[0] : (ax == 1 ? a.u[1] : a.u[2]);
  const R un = TH ? R(sg) * us[k] : R(0);
  const R ip = a.exact ? R(1) : a.inv1pa[k];
  const bool probe = TH && (m & TAG_PROBE3) && a.seed_heat != 0.0;
  const R u0 = probe ? a.u[0][k] : R(0);
  __syncthreads();
  if (!on) return;
  // steps of the tangents t1, t2 (the axes after the normal's) in the tile
  const int i0 = (lq + 1) * PW + lp + 1;
  const int s1 = ax == 1 ? PW : 1, s2 = ax == 1 ? 1 : PW;
  constexpr int C1[14] = {0, 1, -1, 0, 0, 1, 1, -1, -1, 0, 1, -1, 0, 0};
  constexpr int C2[14] = {0, 0, 0, 1, -1, 1, -1, 1, -1, 0, 0, 0, 1, -1};
  R f[14], gq[14], M[14];
#pragma unroll
  for (int q = 0; q < 14; ++q) {
    const int i = i0 + C1[q] * s1 + C2[q] * s2;
    R x = L[q < 9 ? 0 : 3][i];
    if (q >= 9) x -= R(sg) * L[4][i];
    if (C1[q]) x += R(C1[q]) * L[q < 9 ? 1 : 5][i];
    if (C2[q]) x += R(C2[q]) * L[q < 9 ? 2 : 6][i];
    f[q] = x;
    gq[q] = TH ? L[TH ? (q < 9 ? 7 : 8) : 0][i] : R(0);
  }
  face_fill<R, TH>(a, 2 * ax + face, m, un, Tn, f, gq, M);
  adj_local<R, TH>(a, m, 1, Tn, ip, M, u0);
  // place of the x-face node (j, l)
  auto at_x = [&](int j, int l) {
    return xface_packed<R>(g, l) ? l * sq + xface_row(g, sg, j) : kn + j * sp + l * sq;
  };
  int k0 = k;
  if constexpr (sizeof(R) == 4)
    if (ax == 0) k0 = at_x(cp, cq);
#pragma unroll
  for (int c = 0; c < NM; ++c) a.m[c * N + k0] = M[c];
  if (ax != 0) return;
  // the edges and corners of an x face copy the node one step inwards
  const int j[3] = {cp, cp == 1 && !perp ? 0 : -1, cp == Np - 2 && !perp ? Np - 1 : -1};
  const int l[3] = {cq, cq == 1 && !perq ? 0 : -1, cq == Nq - 2 && !perq ? Nq - 1 : -1};
#pragma unroll
  for (int x = 0; x < 9; ++x) {
    const int jj = j[x % 3], ll = l[x / 3];
    if (x == 0 || jj < 0 || ll < 0) continue;
    const int z = at_x(jj, ll);
#pragma unroll
    for (int c = 0; c < NM; ++c) a.m[c * N + z] = M[c];
  }
}

// in-plane offsets of the thread's elements of the 1-node halo region; -1
// off the domain or beyond the tile's region
__device__ inline void zregion1(const Geo3& g, const ZTile& t, int off[2]) {
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int e = int(threadIdx.x) + r * ZT;
    const int dx = e % CXN - 1, dy = e / CXN - 1;
    off[r] = -1;
    if (e < NCR && dx < t.w + 1 && dy < t.h + 1) {
      const int x = axc(t.x0 + dx, g.nx, g.periodic & 1);
      const int y = axc(t.y0 + dy, g.ny, g.periodic & 2);
      if (x >= 0 && y >= 0) off[r] = y * g.nx + x;
    }
  }
}

// per-node inputs of the ALKS update at one node: its moments rho~, u~,
// T~, its velocity, the coefficients' derivatives, 1/(1 + alpha) and class
template <typename R>
struct AdjIn {
  R r, U[3], Tt, u[3], dA, dB, ip;
  int mk;
  double so;  // the node's accumulated sensitivity (sens_mode 1), read ahead
};

// in-plane moment fields of a plane, 1-node halo: s~xy T B q~x; s~xx s~xz;
// s~yy s~yz; q~y, grouped by the differences that read them
template <typename R>
struct AdjE {
  V4<R> c[NCR];
  V2<R> x[NCR], y[NCR];
  R q[NCR];
};
template <typename R>
__device__ inline void adj_e_put(AdjE<R>& E, int ci, const R M[14], R T, R B) {
  E.c[ci] = V4<R>{M[5], T, B, M[11]};
  E.x[ci] = V2<R>{M[4], M[6]};
  E.y[ci] = V2<R>{M[7], M[8]};
  E.q[ci] = M[12];
}

// The ALKS update at a node of a z-march column (eq:afp - eq:agq): V and Theta
// of the new level from the node's moments (cu), the plane's moment fields
// (column ci, end flags ex, ey) and the z differences zd of s~xz s~yz s~zz q~z
// T B (z window zc, zm1, zn, z2 for the product difference of the exact mode),
// and the sensitivity 3 alpha' u.u~ - B' grad T.q~ (paper) or its exact-mode
// counterpart. The node lies at offset off of the plane.
template <typename R, bool TH>
__device__ inline void adj3_update(const Adj3Args<R>& a, const Geo3& g, size_t plane, unsigned off,
                                   const AdjE<R>& E, int ci, int ex, int ey, int ez,
                                   const AdjIn<R>& cu, const R zd[6], const R zc[6],
                                   const R zm1[6], const R zn[6], const R z2[6]) {
  // products are fused with sums only within a statement, so that the fused
  // step and the update pass round alike
#pragma clang fp contract(on)
  struct DV {
    R s[3], q, T, B, Bq;  // s~x. or s~y., q~x or q~y, T, B, B q~
  };
  auto vx = [&](int o) {
    const V4<R> c = E.c[ci + o];
    const V2<R> x = E.x[ci + o];
    return DV{{x.x, c.x, x.y}, c.w, c.y, c.z, c.z * c.w};
  };
  auto vy = [&](int o) {
    const V4<R> c = E.c[ci + o * CXN];
    const V2<R> y = E.y[ci + o * CXN];
    const R q = E.q[ci + o * CXN];
    return DV{{c.x, y.x, y.y}, q, c.y, c.z, c.z * q};
  };
  auto cen = [](R p, R m) { return R(0.5) * (p - m); };
  auto one = [](R h, R f, R f1, R f2) { return h * (R(3) * f - R(4) * f1 + f2); };
  auto diff = [&](const DV& p, const DV& m) {
    return DV{{cen(p.s[0], m.s[0]), cen(p.s[1], m.s[1]), cen(p.s[2], m.s[2])},
              TH ? cen(p.q, m.q) : R(0), TH ? cen(p.T, m.T) : R(0), TH ? cen(p.B, m.B) : R(0),
              TH ? cen(p.Bq, m.Bq) : R(0)};
  };
  // second-order one-sided, f1 and f2 one and two steps inwards
  auto end = [&](int e, const DV& f, const DV& f1, const DV& f2) {
    const R h = e < 0 ? R(-0.5) : R(0.5);
    return DV{{one(h, f.s[0], f1.s[0], f2.s[0]), one(h, f.s[1], f1.s[1], f2.s[1]),
               one(h, f.s[2], f1.s[2], f2.s[2])},
              TH ? one(h, f.q, f1.q, f2.q) : R(0), TH ? one(h, f.T, f1.T, f2.T) : R(0),
              TH ? one(h, f.B, f1.B, f2.B) : R(0), TH ? one(h, f.Bq, f1.Bq, f2.Bq) : R(0)};
  };
  const DV c = vx(0), cy = vy(0);
  DV dx = diff(vx(1), vx(-1));
  if (ex) dx = end(ex, c, vx(-ex), vx(-2 * ex));
  __builtin_amdgcn_sched_barrier(0);
  DV dy = diff(vy(1), vy(-1));
  if (ey) dy = end(ey, cy, vy(-ey), vy(-2 * ey));
  const R S[6] = {c.s[0], c.s[1], c.s[2], cy.s[1], cy.s[2], zc[2]};
  const R A2 = R(2.0 * g.A);
  R V[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const R ds = dx.s[i] + dy.s[i] + zd[i];
    const R su = S[SI[i][0]] * cu.u[0] + S[SI[i][1]] * cu.u[1] + S[SI[i][2]] * cu.u[2];
    const R ru = cu.r * cu.u[i];
    V[i] = R(3) * cu.U[i] + R(9) * su - R(3) * ru - A2 * ds;
  }
  // the Brinkman pairing of the sensitivity: 3 alpha' u.u~ (paper) or
  // alpha' u.V / (1 + alpha) with the undivided V, which then propagates
  // divided by 1 + alpha (exact)
  double pair = 0.0;
  if (a.sens_mode) {
#pragma unroll
    for (int i = 0; i < 3; ++i) pair += double(cu.u[i]) * double(a.exact ? V[i] : cu.U[i]);
    if (a.exact) pair *= double(cu.ip) / 3.0;
  }
  if (a.exact) {
#pragma unroll
    for (int i = 0; i < 3; ++i) V[i] *= cu.ip;
  }
  const unsigned ob = off * unsigned(sizeof(R));
  const auto* out = arg2<Adj3Args<R>>();
  put_b(out->p1[0] + plane, ob, cu.r);
  put_b(out->p1[1] + plane, ob, V[0]);
  put_b(out->p1[2] + plane, ob, V[1]);
  put_b(out->p1[3] + plane, ob, V[2]);
  const R qv[3] = {c.q, cy.q, zc[3]};
  if constexpr (TH) {
    const R qu = qv[0] * cu.u[0] + qv[1] * cu.u[1] + qv[2] * cu.u[2];
    R th = cu.Tt + R(3) * qu;
    if (a.exact) {
      // exact: the transpose of the forward B c.grad_h T, -div_h (B q~)
      const R zbq = dz3(ez, zc[3] * zc[5], zm1[3] * zm1[5], zn[3] * zn[5], z2[3] * z2[5]);
      th -= dx.Bq + dy.Bq + zbq;
    } else {
      const R divq = dx.q + dy.q + zd[3];
      const R gbq = dx.B * qv[0] + dy.B * qv[1] + zd[5] * qv[2];
      th = th - c.B * divq - gbq;
    }
    put_b(out->p1[4] + plane, ob, th);
  }
  if (a.sens_mode) {
    double sv = 0.0;
    if (!ex && !ey && !ez && !(cu.mk & TAG_SOLID3)) {
      sv = a.sens_b_only ? 0.0 : double(cu.dA) * pair;
      if constexpr (TH) {
        double gq = double(dx.T) * double(qv[0]);
        gq += double(dy.T) * double(qv[1]);
        gq += double(zd[4]) * double(qv[2]);
        sv -= double(cu.dB) * gq;
      }
    }
    // the accumulated value was read with the node's other inputs, a plane
    // ahead, so that the read-modify-write does not wait for it here
    put_b(out->sens + plane, off * 8u, a.sens_mode == 1 ? cu.so + sv : sv);
  }
}

// ALKS pass 2, z-marching: V, Theta (eq:afp - eq:agq) and the sensitivity
// from the moments; x and y differences from an LDS plane, z differences
// from a window of three planes in registers.
// ENDS: only the two end planes of a non-periodic z axis (after the fused
// step, which leaves them): tile chunk 0 takes plane 0, chunk 1 plane nz - 1
template <typename R, bool TH, bool ENDS = false>
__global__ __launch_bounds__(ZT) void alks3e_kernel(Geo3 g, Adj3Args<R> a) {
  constexpr int NE = TH ? 9 : 5;  // s~xx s~xy s~xz s~yy s~yz (q~x q~y T B)
  constexpr int NZ = TH ? 6 : 3;  // z window: s~xz s~yz s~zz (q~z T B)
  __shared__ AdjE<R> L[ENDS ? 1 : 2];
  ZTile t;
  if constexpr (ENDS) {
    if (!ztile(g, t, 0, 2, 2)) return;
    if (t.z0 == 1) {
      t.z0 = g.nz - 1;
      t.z1 = g.nz;
    }
  } else {
    if (!ztile(g, t)) return;
  }
  const int tid = int(threadIdx.x), lx = tid % ZX, ly = tid / ZX;
  const int pz = g.periodic & 4;
  const unsigned nxy = unsigned(g.nx) * unsigned(g.ny);
  const unsigned N = unsigned(g.N);
  int coff[2];
  zregion1(g, t, coff);
  const ZNode n0 = znode(g, t, lx, ly, lx < t.w && ly < t.h);
  const bool own = n0.on && t.x0 + lx >= t.xo && t.y0 + ly >= t.yo;
  // plane fields: moments 4, 5, 6, 7, 8 (11, 12) and T, B
  const R* FE[9];
  FE[0] = a.m + 4 * N;
  FE[1] = a.m + 5 * N;
  FE[2] = a.m + 6 * N;
  FE[3] = a.m + 7 * N;
  FE[4] = a.m + 8 * N;
  FE[5] = a.m + 11 * N;
  FE[6] = a.m + 12 * N;
  FE[7] = a.T;
  FE[8] = a.B;
  // z window fields: moments 6, 8, 9 (13) and T, B
  const R* FZ[6] = {a.m + 6 * N, a.m + 8 * N, a.m + 9 * N, a.m + 13 * N, a.T, a.B};
  auto has = [&](int s) { return pz || (s >= 0 && s < g.nz); };
  R v[2][NE];
  auto load = [&](int s) {
    const bool e = has(s);
    const unsigned b = unsigned(zwrap(s, g.nz)) * nxy;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int f = 0; f < NE; ++f) v[r][f] = (e && coff[r] >= 0) ? FE[f][b + coff[r]] : R(0);
  };
  auto store = [&](int slot) {
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int e = tid + r * ZT;
      if (e >= NCR) continue;
      R M[14];
#pragma unroll
      for (int f = 0; f < 5; ++f) M[4 + f] = v[r][f];
      M[11] = TH ? v[r][TH ? 5 : 0] : R(0);
      M[12] = TH ? v[r][TH ? 6 : 0] : R(0);
      adj_e_put(L[slot], e, M, TH ? v[r][TH ? 7 : 0] : R(0), TH ? v[r][TH ? 8 : 0] : R(0));
    }
  };
  auto zload = [&](int s, R z[6]) {
#pragma unroll
    for (int f = 0; f < 6; ++f) z[f] = R(0);
    if (!own || !has(s)) return;
    const unsigned k = unsigned(zwrap(s, g.nz)) * nxy + unsigned(n0.off);
#pragma unroll
    for (int f = 0; f < NZ; ++f) z[f] = FZ[f][k];
  };
  // per-node inputs one plane ahead
  using In = AdjIn<R>;
  auto node_in = [&](int p, In& q) {
    q.r = q.Tt = q.dA = q.dB = R(0);
    q.ip = R(1);
    q.mk = 0;
    q.so = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) q.U[c] = q.u[c] = R(0);
    if (!own || p >= t.z1) return;
    const unsigned k = unsigned(p) * nxy + unsigned(n0.off);
    q.r = a.m[k];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      q.U[c] = a.m[(1 + c) * N + k];
      q.u[c] = a.u[c][k];
    }
    if constexpr (TH) q.Tt = a.m[10 * N + k];
    q.mk = a.mask[k];
    if (a.exact) q.ip = a.inv1pa[k];
    if (a.sens_mode) {
      q.dA = a.dA3[k];
      if constexpr (TH) q.dB = a.dB[k];
      if (a.sens_mode == 1) q.so = a.sens[k];
    }
  };
  if constexpr (ENDS) {
    // one plane: all that it reads is in flight together (5.7 us on 256 x 128 x 128 in
    // FP32; 13 us when the reads waited for each other)
    const int in = t.z0 == 0 ? 1 : -1;
    R zc[6], z1[6], z2[6], zd[6];
    In q;
    load(t.z0);
    zload(t.z0, zc);
    zload(t.z0 + in, z1);
    zload(t.z0 + 2 * in, z2);
    node_in(t.z0, q);
    store(0);
    lds_barrier();
#pragma unroll
    for (int f = 0; f < 6; ++f) zd[f] = dz3(-in, zc[f], z1[f], z1[f], z2[f]);
    if (own)
      adj3_update<R, TH>(a, g, size_t(t.z0) * nxy, unsigned(n0.off), L[0], n0.ci, n0.ex, n0.ey,
                         -in, q, zd, zc, z1, z1, z2);
    return;
  }
  load(t.z0);
  store(0);
  load(t.z0 + 1);
  R zm1[6], zc[6], zn[6];
  zload(t.z0 - 1, zm1);
  zload(t.z0, zc);
  zload(t.z0 + 1, zn);
  In nx;
  node_in(t.z0, nx);
  const int ci = n0.ci;
  for (int p = t.z0; p < t.z1; ++p) {
    const int it = p - t.z0, sc = it & 1;
    lds_barrier();
    if (p + 1 < t.z1) {
      store(sc ^ 1);
      load(p + 2);
    }
    const In cu = nx;
    node_in(p + 1, nx);
    R znn[6];
    zload(p + 2, znn);  // the window's next plane, in flight during this one
    R z2[6] = {R(0), R(0), R(0), R(0), R(0), R(0)};
    const int ez = endof(zwrap(p, g.nz), g.nz, pz);
    if (ez < 0) zload(2, z2);
    if (ez > 0) zload(g.nz - 3, z2);
    R zd[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) zd[f] = dz3(ez, zc[f], zm1[f], zn[f], z2[f]);
    if (own)
      adj3_update<R, TH>(a, g, size_t(p) * nxy, unsigned(n0.off), L[sc], ci, n0.ex, n0.ey, ez, cu,
                         zd, zc, zm1, zn, z2);
#pragma unroll
    for (int f = 0; f < 6; ++f) {
      zm1[f] = zc[f];
      zc[f] = zn[f];
      zn[f] = znn[f];
    }
  }
}

// ---------------------------------------------------------------------------
// ALKS step, fused
// ---------------------------------------------------------------------------
// One z-march per block over the planes 1 .. nz-2 of a non-periodic z axis
// (every plane of a periodic one). At plane s every column of the tile and of
// its 1-node ring forms the sums of plane s (adj_sums) from the level-(n+1)
// coefficients in LDS (tile plus a 2-node halo; the next plane waits in
// registers). They close the moments of plane s - 1 (eq:afeq, eq:ageq), to which
// the local terms are applied as in the pull pass; a boundary node takes the
// moments the face pass left in the scratch. Plane s - 2 is then updated
// (adj3_update) from its in-plane moment fields in LDS and the own column's
// moments of planes s - 3, s - 2 and s - 1, after which the fields of plane s - 1
// and the coefficients of plane s + 1 take their places in LDS. The moments
// that never leave the block are not stored; only the z-window moments of
// planes 1, 2, nz-3 and nz-2 go to the scratch, for the end planes that
// alks3e<ENDS> updates afterwards.
// Bound by instructions. Reading the 19 values of a node from three planes of
// LDS took 157 us on 256 x 128 x 128 in FP32 and 58 us on 97 x 61 x 53 in FP64;
// this way it is 121 and 41 us, the first 106 us with packed x-face moments (417 MB
// pass below the L2 then, 3.9 TB/s; a copy of that size reaches 5.3).
template <typename R>
struct AdjFLds {
  V4<R> p[NSR];  // rho~, V of plane s
  R t[NSR];      // Theta
  AdjE<R> e;     // moment fields of plane s - 2
};

template <typename R, bool TH>
__global__ __launch_bounds__(ZT, sizeof(R) == 4 ? 3 : 1) void alks3f_kernel(Geo3 g, Adj3Args<R> a) {
  constexpr int NM = TH ? 14 : 10;
  __shared__ AdjFLds<R> L;
  const int pz = g.periodic & 4;
  ZTile t;
  if (!ztile(g, t, pz ? 0 : 1, pz ? g.nz : g.nz - 1)) return;
  const int tid = int(threadIdx.x), lx = tid % ZX, ly = tid / ZX;
  const size_t nxy = size_t(g.nx) * size_t(g.ny);
  const size_t N = size_t(g.N);
  // byte offsets in a plane of the thread's elements of the 2-node halo region;
  // an element off the domain reads the plane's first node, which nothing uses
  unsigned roff[SRL];
  {
    int off[SRL];
    zregion(g, t, off);
#pragma unroll
    for (int r = 0; r < SRL; ++r)
      roff[r] = off[r] < 0 ? 0u : unsigned(off[r]) * unsigned(sizeof(R));
  }
  const ZNode n0 = znode(g, t, lx, ly, lx < t.w && ly < t.h);
  ZNode n1 = zring(g, t);
  n1.on = n1.on && n1.off >= 0;
  const bool own = n0.on && t.x0 + lx >= t.xo && t.y0 + ly >= t.yo;
  const bool xy0 = n0.ex || n0.ey, xy1 = n1.ex || n1.ey;
  // offsets in a plane, and the positions from which the LDS reads count up
  unsigned off0 = n0.on ? unsigned(n0.off) : 0u, off1 = n1.on ? unsigned(n1.off) : 0u;
  // ... those of an x-face column's moments (xface_packed)
  auto packed = [&](const ZNode& n, unsigned off) {
    return n.ex ? unsigned(xface_row(g, n.ex, int(off) / g.nx)) : off;
  };
  unsigned pk0 = 0, pk1 = 0;
  if constexpr (sizeof(R) == 4) {
    pk0 = packed(n0, off0);
    pk1 = packed(n1, off1);
  }
  unsigned i0 = unsigned(n0.lds - SX - 1), i1 = unsigned(n1.lds - SX - 1);
  unsigned e0 = unsigned(n0.ci), e1 = unsigned(n1.ci);
  // first node of plane q (of the nearest one that exists)
  auto plane = [&](int q) {
    if (pz) {
      const int c = zwrap(q, g.nz);
      return size_t(c < 0 ? c + g.nz : (c >= g.nz ? c - g.nz : c)) * nxy;  // nz >= 3, -4 <= q < nz + 4
    }
    return size_t(q < 0 ? 0 : (q >= g.nz ? g.nz - 1 : q)) * nxy;
  };
  auto zend = [&](int q) { return !pz && (q <= 0 || q >= g.nz - 1); };
  V4<R> v[SRL];
  R vt[SRL];
  auto load = [&](const auto* in, size_t b) {
    const R *F0 = in->p0[0] + b, *F1 = in->p0[1] + b, *F2 = in->p0[2] + b, *F3 = in->p0[3] + b;
    const R* F4 = TH ? in->p0[4] + b : F0;
#pragma unroll
    for (int r = 0; r < SRL; ++r) {
      v[r].x = at_b(F0, roff[r]);
      v[r].y = at_b(F1, roff[r]);
      v[r].z = at_b(F2, roff[r]);
      v[r].w = at_b(F3, roff[r]);
      if constexpr (TH) vt[r] = at_b(F4, roff[r]);
    }
  };
  auto store = [&]() {
#pragma unroll
    for (int r = 0; r < SRL; ++r)
      if ((r + 1) * ZT <= NSR || tid + r * ZT < NSR) {
        L.p[tid + r * ZT] = v[r];
        if constexpr (TH) L.t[tid + r * ZT] = vt[r];
      }
  };
  // class, T and B of a column's node
  struct Col {
    int m;
    R T, B;
  };
  auto col_in = [&](const auto* in, size_t b, unsigned off) {
    const unsigned ob = off * unsigned(sizeof(R));
    return Col{int(at_b(in->mask + b, off)), TH ? at_b(in->T + b, ob) : R(0),
               TH ? at_b(in->B + b, ob) : R(0)};
  };
  // sums of the plane in LDS
  auto sums = [&](unsigned i, AdjSums<R>& o) {
    adj_sums<R, TH>([&](int dx, int dy) { return L.p[i + unsigned(dy * SX + dx)]; },
                    [&](int dx, int dy) { return TH ? L.t[i + unsigned(dy * SX + dx)] : R(0); }, o);
  };
  const int first = t.z0 - 2, last = t.z1 + 1;  // planes the sums are taken of
  load(&a, plane(first));
  store();
  Col c0 = col_in(&a, plane(first), off0);  // own node at plane s - 1
  int mc = 0;                           // class of the own node at plane s - 2
  AdjPart<R> P0 = {}, P1 = {};  // partial moments of the columns at plane s - 1
  // what plane s - 1 sends to plane s: t, x, y, xx, yy; T, x, y
  R m0[8] = {}, m1[8] = {};
  R Mc[5] = {};  // rho~, u~, T~ of the own node at plane s - 2
  R zm1[6] = {}, zc[6] = {}, zn[6] = {};
  const R z0v[6] = {};
  lds_barrier();
  // first nodes of the planes s - 2 .. s + 1
  size_t b2 = plane(first - 2), b1 = plane(first - 1), b0 = plane(first), bn = plane(first + 1);
  for (int s = first; s <= last; ++s) {
    off0 = anew(off0);
    off1 = anew(off1);
    i0 = anew(i0);
    i1 = anew(i1);
    e0 = anew(e0);
    e1 = anew(e1);
#pragma unroll
    for (int r = 0; r < SRL; ++r) roff[r] = anew(roff[r]);
    const unsigned ob0 = off0 * unsigned(sizeof(R));
    const auto* in = arg2<Adj3Args<R>>();
    // Inputs of the update, of the ring's E fields and of the own node's next
    // closing, and the face pass's moments of boundary nodes; then the next plane
    AdjIn<R> cu;
    cu.dA = cu.dB = R(0);
    cu.ip = R(1);
    cu.so = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) cu.u[c] = R(0);
    Col c0n = {}, c1 = {};
    if (n0.on) c0n = col_in(in, b0, off0);
    if (own && s - 2 >= t.z0) {
#pragma unroll
      for (int c = 0; c < 3; ++c) cu.u[c] = at_b(in->u[c] + b2, ob0);
      cu.ip = at_b(in->inv1pa + b2, ob0);
      cu.dA = at_b(in->dA3 + b2, ob0);
      cu.dB = TH ? at_b(in->dB + b2, ob0) : R(0);
      if (a.sens_mode == 1) cu.so = at_b(in->sens + b2, anew(off0) * 8u);
    }
    const bool close = s >= t.z0;  // plane s - 1 is one whose moments are used
    const bool bnd0 = xy0 || zend(s - 1), bnd1 = xy1 || zend(s - 1);
    R M[14], Mr[14];
#pragma unroll
    for (int i = 0; i < 14; ++i) M[i] = Mr[i] = R(0);
    if (close) {
      if (n1.on) c1 = col_in(in, b1, off1);
      if (n0.on && bnd0) {
        unsigned om = ob0;
        if constexpr (sizeof(R) == 4)
          if (xface_packed<R>(g, s - 1)) om = pk0 * unsigned(sizeof(R));
#pragma unroll
        for (int i = 0; i < NM; ++i) M[i] = at_b(in->m + (size_t(i) * N + b1), om);
      }
      if (n1.on && bnd1) {
        unsigned om = off1;
        if constexpr (sizeof(R) == 4)
          if (xface_packed<R>(g, s - 1)) om = pk1;
#pragma unroll
        for (int i = 4; i < NM; ++i)
          if (i < 9 || i == 11 || i == 12)
            Mr[i] = at_b(in->m + (size_t(i) * N + b1), om * unsigned(sizeof(R)));
      }
    }
    load(in, bn);
    if (n0.on) {
      AdjSums<R> o;
      sums(i0, o);
      if (close && !bnd0) {
        adj_close<R, TH>(P0, o, M);
        if (TH && ((c0.m >> 2) & 3) == THERM_DIRICHLET3) M[11] = M[12] = M[13] = R(0);
      }
      P0 = adj_part(o, m0[0], m0[1], m0[2], m0[3], m0[4], m0[5], m0[6], m0[7]);
      const R nm[8] = {o.mt, o.mx, o.my, o.mxx, o.myy, o.gt, o.gx, o.gy};
#pragma unroll
      for (int i = 0; i < 8; ++i) m0[i] = nm[i];
    }
    __builtin_amdgcn_sched_barrier(0);
    if (n1.on) {
      AdjSums<R> o;
      sums(i1, o);
      if (close && !bnd1) {
        adj_close<R, TH>(P1, o, Mr);
        if (TH && ((c1.m >> 2) & 3) == THERM_DIRICHLET3) Mr[11] = Mr[12] = R(0);
      }
      P1 = adj_part(o, m1[0], m1[1], m1[2], m1[3], m1[4], m1[5], m1[6], m1[7]);
      const R nm[8] = {o.mt, o.mx, o.my, o.mxx, o.myy, o.gt, o.gx, o.gy};
#pragma unroll
      for (int i = 0; i < 8; ++i) m1[i] = nm[i];
    }
    zn[0] = M[6];
    zn[1] = M[8];
    zn[2] = M[9];
    zn[3] = M[13];
    zn[4] = c0.T;
    zn[5] = c0.B;
    if (own && s - 2 >= t.z0) {
      if (!xy0) {
        R m[14];
#pragma unroll
        for (int c = 0; c < 4; ++c) m[c] = Mc[c];
        m[10] = Mc[4];
        m[11] = L.e.c[e0].w;
        m[12] = L.e.q[e0];
        m[13] = zc[3];
        adj_local<R, TH>(a, mc, 0, zc[4], a.exact ? R(1) : cu.ip, m, cu.u[0]);
#pragma unroll
        for (int c = 0; c < 4; ++c) Mc[c] = m[c];
        Mc[4] = m[10];
      }
      cu.mk = mc;
      cu.r = Mc[0];
#pragma unroll
      for (int c = 0; c < 3; ++c) cu.U[c] = Mc[1 + c];
      cu.Tt = Mc[4];
      R zd[6];
#pragma unroll
      for (int f = 0; f < 6; ++f) zd[f] = dz3(0, zc[f], zm1[f], zn[f], R(0));
      adj3_update<R, TH>(a, g, b2, off0, L.e, int(e0), n0.ex, n0.ey, 0, cu, zd, zc, zm1, zn, z0v);
    }
    // the z-window moments next to the end planes, for alks3e<ENDS>
    const int q = s - 1;
    if (!pz && own && !bnd0 && q >= t.z0 && q < t.z1 && (q <= 2 || q >= g.nz - 3)) {
      put_b(a.m + (6 * N + b1), ob0, M[6]);
      put_b(a.m + (8 * N + b1), ob0, M[8]);
      put_b(a.m + (9 * N + b1), ob0, M[9]);
      if constexpr (TH) put_b(a.m + (13 * N + b1), ob0, M[13]);
    }
    lds_barrier();
    if (n1.on) adj_e_put(L.e, int(e1), Mr, c1.T, c1.B);
    if (n0.on) adj_e_put(L.e, int(e0), M, c0.T, c0.B);
    store();
    lds_barrier();
#pragma unroll
    for (int f = 0; f < 6; ++f) {
      zm1[f] = zc[f];
      zc[f] = zn[f];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) Mc[i] = M[i];
    Mc[4] = M[10];
    mc = c0.m;
    c0 = c0n;
    b2 = b1;
    b1 = b0;
    b0 = bn;
    bn = plane(s + 2);
  }
}

// objective sum over tagged nodes (steady runs): pressure-drop tags of
// drho, or the probe enthalpy flux u_x T. TS blocks stride over the nodes in
// a fixed order and leave one partial sum each.
constexpr int TS = 256;
template <typename R>
__global__ __launch_bounds__(NT3) void tag_sum3_kernel(Geo3 g, const uint8_t* __restrict__ mask,
                                                       const R* d, const R* ux, const R* T,
                                                       int objective, double* part) {
  __shared__ double red[NT3 / 64];
  double s = 0.0;
  for (int k = int(blockIdx.x) * NT3 + int(threadIdx.x); k < g.N; k += TS * NT3) {
    const int m = mask[k];
    if (objective == 1) {
      if (m & TAG_PROBE3) s += double(ux[k]) * double(T[k]);
    } else {
      if (m & TAG_J_INLET3) s += double(d[k]);
      if (m & TAG_J_OUTLET3) s -= double(d[k]);
    }
  }
  s = block_sum3(s, red);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

}  // namespace

int blocks3(int N) {
  const int b = (N + NT3 - 1) / NT3;
  return NXCD * ((b + NXCD - 1) / NXCD);
}

int zblocks3(const Geo3& g) { return ztiles(g.nx, ZX) * ztiles(g.ny, ZY) * zchunks(g); }

namespace {
// Chunks a march of the planes is split into: the number for which the rounds of
// the kernel's resident blocks, times the planes a block walks through (its
// chunk and halo planes more), are fewest. On 97 x 61 x 53 (32 tiles, FP64) the
// forward step takes 30 us with 16 chunks and 41 us with the 17 of three planes
// that overflow one round.
template <typename K>
int chunks_for(const Geo3& g, K kernel, int planes, int halo) {
  int dev = 0, ncu = 0, bpc = 0;
  const int most = g.nz / 2 > 1 ? g.nz / 2 : 1;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&bpc, kernel, ZT, 0) != hipSuccess ||
      ncu <= 0 || bpc <= 0)
    return zchunks_default(g.nz);
  const long long tiles = (long long)ztiles(g.nx, ZX) * ztiles(g.ny, ZY), res = (long long)bpc * ncu;
  long long best = LLONG_MAX;
  int nch = 1;
  for (int n = 1; n <= most; ++n) {
    const long long cost = ((tiles * n + res - 1) / res) * ((planes + n - 1) / n + halo);
    if (cost < best) {
      best = cost;
      nch = n;
    }
  }
  return nch;
}
}  // namespace

int zchunks_default(int nz) { return nz / 16 > 1 ? nz / 16 : 1; }

template <typename R, bool TH>
void zplan3(Geo3& g) {
  const int pz = g.periodic & 4;
  g.zc = chunks_for(g, lks3z_kernel<R, TH>, g.nz, 2);
  g.zca = chunks_for(g, alks3e_kernel<R, TH>, g.nz, 2);
  g.zcf = chunks_for(g, alks3f_kernel<R, TH>, pz ? g.nz : g.nz - 2, 4);
}
void zplan3(Geo3& g, int rsz) {
  if (rsz == 8) g.thermal ? zplan3<double, true>(g) : zplan3<double, false>(g);
  else g.thermal ? zplan3<float, true>(g) : zplan3<float, false>(g);
}

int copy_nodes3(const Geo3& g, int* out) {
  const int n3[3] = {g.nx, g.ny, g.nz};
  int n = 0;
  for (int l = 0; l < g.nz; ++l)
    for (int j = 0; j < g.ny; ++j)
      for (int i = 0; i < g.nx; ++i) {
        const int c[3] = {i, j, l};
        int ne = 0;
        for (int ax = 0; ax < 3; ++ax)
          if (!((g.periodic >> ax) & 1) && (c[ax] == 0 || c[ax] == n3[ax] - 1)) ++ne;
        if (ne < 2) continue;
        if (out) out[n] = (l * g.ny + j) * g.nx + i;
        ++n;
      }
  return n;
}

int edge_nodes3(const Geo3& g, int* out) {
  const bool py = g.periodic & 2, pz = g.periodic & 4, px = g.periodic & 1;
  if (py || pz) return 0;
  int n = 0;
  for (int l : {0, g.nz - 1})
    for (int j : {0, g.ny - 1})
      for (int i = px ? 0 : 1; i < (px ? g.nx : g.nx - 1); ++i) {
        if (out) out[n] = (l * g.ny + j) * g.nx + i;
        ++n;
      }
  return n;
}

namespace {
// blocks of alks3_face_kernel
unsigned face_blocks(const Geo3& g, int nedge) {
  int n = (nedge + NT3 - 1) / NT3;
  for (int ax = 0; ax < 3; ++ax) {
    if ((g.periodic >> ax) & 1) continue;
    const FaceTiles t = face_tiles(g, ax);
    n += 2 * t.tp * t.tq;
  }
  return unsigned(n);
}
}  // namespace

template <typename R>
void launch_coef3(const Geo3& g, const uint8_t* mask, const double* gamma, double alpha_max,
                  double q_alpha, double Kf, double Ks, double qK, R* inv1pa, R* B, R* dA3,
                  R* dB, hipStream_t s) {
  coef3_kernel<R><<<blocks3(g.N), NT3, 0, s>>>(g, mask, gamma, alpha_max, q_alpha, Kf, Ks, qK,
                                               inv1pa, B, dA3, dB);
}

template <typename R>
void launch_init3(const Geo3& g, const uint8_t* mask, const R* const ub[3], const R* Tb,
                  double ufac0, R* const st[5], hipStream_t s) {
  init3_kernel<R><<<blocks3(g.N), NT3, 0, s>>>(g, mask, ub[0], ub[1], ub[2], Tb, ufac0, st[0],
                                               st[1], st[2], st[3], st[4]);
}

template <typename R>
void launch_lks3_step(const Geo3& g, const Fwd3Args<R>& a, hipStream_t s) {
  const unsigned nb = unsigned(NXCD * ((zblocks3(g) + NXCD - 1) / NXCD));
  const unsigned nc = unsigned((a.ncopy + NT3 - 1) / NT3);
  if (g.thermal) {
    lks3z_kernel<R, true><<<nb, ZT, 0, s>>>(g, a);
    if (a.ncopy)
      copy3_kernel<R, true><<<nc, NT3, 0, s>>>(g, a.copy, a.ncopy, a.s1[0], a.s1[1], a.s1[2],
                                               a.s1[3], a.s1[4]);
  } else {
    lks3z_kernel<R, false><<<nb, ZT, 0, s>>>(g, a);
    if (a.ncopy)
      copy3_kernel<R, false><<<nc, NT3, 0, s>>>(g, a.copy, a.ncopy, a.s1[0], a.s1[1], a.s1[2],
                                                a.s1[3], a.s1[4]);
  }
}

template <typename R, bool TH>
void launch_alks3_fused(const Geo3& g0, const Adj3Args<R>& a, hipStream_t s) {
  Geo3 g = g0;
  g.zc = g0.zcf;
  const unsigned nz = unsigned(NXCD * ((zblocks3(g) + NXCD - 1) / NXCD));
  const unsigned nf = face_blocks(g, a.nface);
  if (nf) alks3_face_kernel<R, TH><<<nf, NT3, 0, s>>>(g, a);
  alks3f_kernel<R, TH><<<nz, ZT, 0, s>>>(g, a);
  if (!(g.periodic & 4)) {
    const int ends = 2 * ztiles(g.nx, ZX) * ztiles(g.ny, ZY);
    alks3e_kernel<R, TH, true><<<unsigned(NXCD * ((ends + NXCD - 1) / NXCD)), ZT, 0, s>>>(g, a);
  }
}

template <typename R>
void launch_alks3_step(const Geo3& g0, const Adj3Args<R>& a, hipStream_t s) {
  if (g0.fused) {
    if (g0.thermal) launch_alks3_fused<R, true>(g0, a, s);
    else launch_alks3_fused<R, false>(g0, a, s);
    return;
  }
  Geo3 g = g0;
  g.zc = g0.zca;
  const unsigned nb = unsigned(blocks3(g.N));
  const unsigned nz = unsigned(NXCD * ((zblocks3(g) + NXCD - 1) / NXCD));
  const unsigned nf = face_blocks(g, a.nface);
  if (g.thermal) {
    alks3_pull_kernel<R, true><<<nb, NT3, 0, s>>>(g, a);
    if (nf) alks3_face_kernel<R, true><<<nf, NT3, 0, s>>>(g, a);
    alks3e_kernel<R, true><<<nz, ZT, 0, s>>>(g, a);
  } else {
    alks3_pull_kernel<R, false><<<nb, NT3, 0, s>>>(g, a);
    if (nf) alks3_face_kernel<R, false><<<nf, NT3, 0, s>>>(g, a);
    alks3e_kernel<R, false><<<nz, ZT, 0, s>>>(g, a);
  }
}

template <typename R>
void launch_tag_sum3(const Geo3& g, const uint8_t* mask, const R* d, const R* ux, const R* T,
                     int objective, double* part, double* out, hipStream_t s) {
  tag_sum3_kernel<R><<<TS, NT3, 0, s>>>(g, mask, d, ux, T, objective, part);
  launch_sum(part, TS, out, s);
}

int tag_sum3_parts() { return TS; }

#define LKS3_INSTANTIATE(R)                                                                   \
  template void launch_coef3<R>(const Geo3&, const uint8_t*, const double*, double, double,  \
                                double, double, double, R*, R*, R*, R*, hipStream_t);        \
  template void launch_init3<R>(const Geo3&, const uint8_t*, const R* const[3], const R*,    \
                                double, R* const[5], hipStream_t);                           \
  template void launch_lks3_step<R>(const Geo3&, const Fwd3Args<R>&, hipStream_t);           \
  template void launch_alks3_step<R>(const Geo3&, const Adj3Args<R>&, hipStream_t);          \
  template void launch_tag_sum3<R>(const Geo3&, const uint8_t*, const R*, const R*, const R*, \
                                   int, double*, double*, hipStream_t);
LKS3_INSTANTIATE(float)
LKS3_INSTANTIATE(double)

}  // namespace lks
