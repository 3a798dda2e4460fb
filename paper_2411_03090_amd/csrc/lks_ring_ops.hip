// Host construction, in double precision, of the linear operators that
// complete the adjoint populations on the boundary ring (Sec. 2.5 and
// Appendix A of the paper).
//
// On a ring node with outward normal n the ALKS pull leaves the three
// populations with c_i.n > 0 undetermined. The paper fixes them, together
// with the Lagrange multipliers of the boundary conditions, as the
// least-squares (generalized-inverse) solution of the nine boundary
// equations, one per direction i:
//   flow     (n.c_i) f~_i - 2A sum_j w_j (n.c_j)(c_j.c_i) f~_j
//            + [mu~.c_i | lambda~ + mu~_s (c_i.t)] - kappa~ T (c_i.n) + s_i
//   thermal  (n.c_i) g~_i - B (n.q~) + [eta~ | kappa~ (c_i - u).n]
// (eq:afboundaryu, eq:afboundaryp, eq:afboundaryuq, eq:afboundarypq,
// eq:agboundaryT, eq:agboundaryq; the s~ and q~ of the printed conditions are
// expanded through eq:afs and eq:agq, and the reading of the garbled matrix
// M is the one that reproduces the printed closed form eq:ftilde).
// Everything except the zero-flux rows is independent of the node, so the
// solution is a fixed linear map of the known populations, the seed s and
// kappa~ T; the zero-flux case depends on the normal velocity u_n only
// through one column and is kept in Schur-complement form.
#include <cmath>
#include <cstring>

#include "lks_device.h"

namespace lks {
namespace {

const int HX[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
const int HY[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
const double HW[9] = {4.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9,
                      1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36};

// D3Q19 in the numbering of the three-dimensional kernels
const int C19[19][3] = {{0, 0, 0},  {1, 0, 0},   {-1, 0, 0}, {0, 1, 0},   {0, -1, 0},
                        {0, 0, 1},  {0, 0, -1},  {1, 1, 0},  {-1, -1, 0}, {1, -1, 0},
                        {-1, 1, 0}, {1, 0, 1},   {-1, 0, -1}, {1, 0, -1}, {-1, 0, 1},
                        {0, 1, 1},  {0, -1, -1}, {0, 1, -1}, {0, -1, 1}};
const double W19[19] = {1.0 / 3,  1.0 / 18, 1.0 / 18, 1.0 / 18, 1.0 / 18, 1.0 / 18, 1.0 / 18,
                        1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36,
                        1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36};

// inverse of an n x n matrix (n <= 8) by Gauss-Jordan with partial pivoting
void invert(int n, const double* a, double* inv) {
  double m[8][16];
  for (int r = 0; r < n; ++r)
    for (int c = 0; c < 2 * n; ++c) m[r][c] = c < n ? a[r * n + c] : (c - n == r ? 1.0 : 0.0);
  for (int p = 0; p < n; ++p) {
    int piv = p;
    for (int r = p + 1; r < n; ++r)
      if (std::fabs(m[r][p]) > std::fabs(m[piv][p])) piv = r;
    if (piv != p)
      for (int c = 0; c < 2 * n; ++c) std::swap(m[p][c], m[piv][c]);
    const double d = m[p][p];
    for (int c = 0; c < 2 * n; ++c) m[p][c] /= d;
    for (int r = 0; r < n; ++r) {
      if (r == p) continue;
      const double f = m[r][p];
      for (int c = 0; c < 2 * n; ++c) m[r][c] -= f * m[p][c];
    }
  }
  for (int r = 0; r < n; ++r)
    for (int c = 0; c < n; ++c) inv[r * n + c] = m[r][n + c];
}

// P = (K^T K)^-1 K^T for a rows x n matrix K (row-major), P is n x rows
void pseudo_inverse(int rows, int n, const double* K, double* P) {
  double G[64], Gi[64];
  for (int a = 0; a < n; ++a)
    for (int b = 0; b < n; ++b) {
      double s = 0;
      for (int r = 0; r < rows; ++r) s += K[r * n + a] * K[r * n + b];
      G[a * n + b] = s;
    }
  invert(n, G, Gi);
  for (int a = 0; a < n; ++a)
    for (int r = 0; r < rows; ++r) {
      double s = 0;
      for (int b = 0; b < n; ++b) s += Gi[a * n + b] * K[r * n + b];
      P[a * rows + r] = s;
    }
}

}  // namespace

namespace {
// the operator of a node with outward normal +x
void build_ring_op(double A, double Bf, RingOp& op) {
  std::memset(&op, 0, sizeof op);
  const int nx = 1, ny = 0;
  const int tx = -ny, ty = nx;
  int cn[9], nu = 0;
  for (int q = 0; q < 9; ++q) {
    cn[q] = HX[q] * nx + HY[q] * ny;
    if (cn[q] > 0) op.unk[nu++] = q;
  }
  for (int a = 0; a < 3; ++a) op.uw[a] = HW[op.unk[a]];
  // flow rows: coefficient of f~_q in row r
  double M[9][9];
  for (int r = 0; r < 9; ++r)
    for (int q = 0; q < 9; ++q)
      M[r][q] = (r == q ? cn[r] : 0.0) -
                2.0 * A * HW[q] * cn[q] * double(HX[q] * HX[r] + HY[q] * HY[r]);
  for (int v = 0; v < 2; ++v) {
    double K[9 * 5], P[5 * 9];
    for (int r = 0; r < 9; ++r) {
      for (int a = 0; a < 3; ++a) K[r * 5 + a] = M[r][op.unk[a]];
      K[r * 5 + 3] = v == 0 ? double(HX[r]) : 1.0;
      K[r * 5 + 4] = v == 0 ? double(HY[r]) : double(HX[r] * tx + HY[r] * ty);
    }
    pseudo_inverse(9, 5, K, P);
    for (int a = 0; a < 3; ++a) {
      double s = 0, k = 0;
      for (int r = 0; r < 9; ++r) {
        s += P[a * 9 + r];
        k += P[a * 9 + r] * cn[r];
      }
      op.Ls[v][a] = -s;
      op.Lk[v][a] = k;
      for (int q = 0; q < 9; ++q) {
        double t = 0;
        if (cn[q] <= 0)
          for (int r = 0; r < 9; ++r) t += P[a * 9 + r] * M[r][q];
        op.Lf[v][a][q] = -t;
      }
    }
  }
  // thermal rows: coefficient of g~_q in row r
  double Mg[9][9];
  for (int r = 0; r < 9; ++r)
    for (int q = 0; q < 9; ++q) Mg[r][q] = (r == q ? cn[r] : 0.0) - Bf * HW[q] * cn[q];
  {
    double K[9 * 4], P[4 * 9];
    for (int r = 0; r < 9; ++r) {
      for (int a = 0; a < 3; ++a) K[r * 4 + a] = Mg[r][op.unk[a]];
      K[r * 4 + 3] = 1.0;
    }
    pseudo_inverse(9, 4, K, P);
    for (int a = 0; a < 3; ++a)
      for (int q = 0; q < 9; ++q) {
        double t = 0;
        if (cn[q] <= 0)
          for (int r = 0; r < 9; ++r) t += P[a * 9 + r] * Mg[r][q];
        op.Ld[a][q] = -t;
      }
  }
  {
    double K0[9 * 3], G[9], H[9];
    for (int r = 0; r < 9; ++r)
      for (int a = 0; a < 3; ++a) K0[r * 3 + a] = Mg[r][op.unk[a]];
    for (int a = 0; a < 3; ++a)
      for (int b = 0; b < 3; ++b) {
        double s = 0;
        for (int r = 0; r < 9; ++r) s += K0[r * 3 + a] * K0[r * 3 + b];
        G[a * 3 + b] = s;
      }
    invert(3, G, H);
    // HK = H K0^T (3 x 9); Q = I - K0 HK (9 x 9)
    double HK[3 * 9], Q[9][9];
    for (int a = 0; a < 3; ++a)
      for (int r = 0; r < 9; ++r) {
        double s = 0;
        for (int b = 0; b < 3; ++b) s += H[a * 3 + b] * K0[r * 3 + b];
        HK[a * 9 + r] = s;
      }
    for (int r = 0; r < 9; ++r)
      for (int c = 0; c < 9; ++c) {
        double s = 0;
        for (int a = 0; a < 3; ++a) s += K0[r * 3 + a] * HK[a * 9 + c];
        Q[r][c] = (r == c ? 1.0 : 0.0) - s;
      }
    double Qcn[9], Q1[9];
    for (int r = 0; r < 9; ++r) {
      double s = 0, t = 0;
      for (int c = 0; c < 9; ++c) {
        s += Q[r][c] * cn[c];
        t += Q[r][c];
      }
      Qcn[r] = s;
      Q1[r] = t;
    }
    op.A0 = op.A1 = op.A2 = 0;
    for (int r = 0; r < 9; ++r) {
      op.A0 += cn[r] * Qcn[r];
      op.A1 += cn[r] * Q1[r];
      op.A2 += Q1[r];
    }
    for (int q = 0; q < 9; ++q) {
      double ga = 0, ge = 0;
      if (cn[q] <= 0)
        for (int r = 0; r < 9; ++r) {
          ga += Qcn[r] * Mg[r][q];
          ge += Q1[r] * Mg[r][q];
        }
      op.ga[q] = ga;
      op.ge[q] = ge;
    }
    for (int a = 0; a < 3; ++a) {
      double hc = 0, h1 = 0;
      for (int r = 0; r < 9; ++r) {
        hc += HK[a * 9 + r] * cn[r];
        h1 += HK[a * 9 + r];
      }
      op.hc[a] = hc;
      op.h1[a] = h1;
      for (int q = 0; q < 9; ++q) {
        double t = 0;
        if (cn[q] <= 0)
          for (int r = 0; r < 9; ++r) t += HK[a * 9 + r] * Mg[r][q];
        op.Lg0[a][q] = -t;
      }
    }
  }
}
}  // namespace

// Reflection t -> -t of the +x operator: unknown directions in ascending order
// are n, n + t, n - t (1, 5, 8); the known ones rest, t, -t, -n, -n + t,
// -n - t are 0, 2, 4, 3, 6, 7. Entries equal by symmetry are averaged.
void build_ring_fill(double A, double Bf, RingFillT<double>& F) {
  RingOp op;
  build_ring_op(A, Bf, op);
  std::memset(&F, 0, sizeof F);
  const double w = op.uw[0], wd = op.uw[1];
  auto even = [](const double* row, double e[4]) {
    e[0] = row[0];
    e[1] = 0.5 * (row[2] + row[4]);
    e[2] = row[3];
    e[3] = 0.5 * (row[6] + row[7]);
  };
  // Y, Z (even) and X (odd) of a 3 x 9 map
  auto split = [&](const double L[3][9], double Y[4], double Z[4], double X[2]) {
    double y[9], z[9], x[9];
    for (int q = 0; q < 9; ++q) {
      z[q] = wd * (L[1][q] + L[2][q]);
      y[q] = w * L[0][q] + z[q];
      x[q] = wd * (L[1][q] - L[2][q]);
    }
    even(y, Y);
    if (Z) even(z, Z);
    X[0] = 0.5 * (x[2] - x[4]);
    X[1] = 0.5 * (x[6] - x[7]);
  };
  for (int v = 0; v < 2; ++v) {
    split(op.Lf[v], F.Y[v], F.Z[v], F.X[v]);
    F.Zs[v] = wd * (op.Ls[v][1] + op.Ls[v][2]);
    F.Ys[v] = w * op.Ls[v][0] + F.Zs[v];
    F.Zk[v] = wd * (op.Lk[v][1] + op.Lk[v][2]);
    F.Yk[v] = w * op.Lk[v][0] + F.Zk[v];
  }
  split(op.Ld, F.Dy, nullptr, F.Dx);
  split(op.Lg0, F.Gy, nullptr, F.Gx);
  even(op.ga, F.ka);
  even(op.ge, F.ke);
  F.A0 = op.A0;
  F.A1 = op.A1;
  F.A2 = op.A2;
  F.Hc = w * op.hc[0] + wd * (op.hc[1] + op.hc[2]);
  F.H1 = w * op.h1[0] + wd * (op.h1[1] + op.h1[2]);
}

// D3Q19 faces: the same least-squares completion over 19 rows, with the five
// directions c_i.n > 0 unknown; the pressure face has the multipliers
// lambda~ + mu~_1 (c_i.t1) + mu~_2 (c_i.t2) with t1, t2 the two coordinate
// axes normal to n, the velocity face mu~.c_i.
namespace {
// the operator of a face node with outward normal +x
void build_face_op(double A, double Bf, FaceOp3& op) {
  std::memset(&op, 0, sizeof op);
  const int ax = 0, sg = 1;
  const int t1 = (ax + 1) % 3, t2 = (ax + 2) % 3;
  int cn[19], nu = 0;
  for (int q = 0; q < 19; ++q) {
    cn[q] = sg * C19[q][ax];
    if (cn[q] > 0) op.unk[nu++] = q;
  }
  double M[19][19];
  for (int r = 0; r < 19; ++r)
    for (int q = 0; q < 19; ++q) {
      const double cc = C19[q][0] * C19[r][0] + C19[q][1] * C19[r][1] + C19[q][2] * C19[r][2];
      M[r][q] = (r == q ? cn[r] : 0.0) - 2.0 * A * W19[q] * cn[q] * cc;
    }
  for (int v = 0; v < 2; ++v) {
    double K[19 * 8], P[8 * 19];
    for (int r = 0; r < 19; ++r) {
      for (int a = 0; a < 5; ++a) K[r * 8 + a] = M[r][op.unk[a]];
      if (v == 0) {
        for (int d = 0; d < 3; ++d) K[r * 8 + 5 + d] = C19[r][d];
      } else {
        K[r * 8 + 5] = 1.0;
        K[r * 8 + 6] = C19[r][t1];
        K[r * 8 + 7] = C19[r][t2];
      }
    }
    pseudo_inverse(19, 8, K, P);
    for (int a = 0; a < 5; ++a) {
      double s = 0, k = 0;
      for (int r = 0; r < 19; ++r) {
        s += P[a * 19 + r];
        k += P[a * 19 + r] * cn[r];
      }
      op.Ls[v][a] = -s;
      op.Lk[v][a] = k;
      for (int q = 0; q < 19; ++q) {
        double t = 0;
        if (cn[q] <= 0)
          for (int r = 0; r < 19; ++r) t += P[a * 19 + r] * M[r][q];
        op.Lf[v][a][q] = -t;
      }
    }
  }
  double Mg[19][19];
  for (int r = 0; r < 19; ++r)
    for (int q = 0; q < 19; ++q) Mg[r][q] = (r == q ? cn[r] : 0.0) - Bf * W19[q] * cn[q];
  {
    double K[19 * 6], P[6 * 19];
    for (int r = 0; r < 19; ++r) {
      for (int a = 0; a < 5; ++a) K[r * 6 + a] = Mg[r][op.unk[a]];
      K[r * 6 + 5] = 1.0;
    }
    pseudo_inverse(19, 6, K, P);
    for (int a = 0; a < 5; ++a)
      for (int q = 0; q < 19; ++q) {
        double t = 0;
        if (cn[q] <= 0)
          for (int r = 0; r < 19; ++r) t += P[a * 19 + r] * Mg[r][q];
        op.Ld[a][q] = -t;
      }
  }
  {
    // zero-flux face: Schur form in the normal velocity u_n
    double K0[19 * 5], G[25], H[25], HK[5 * 19];
    for (int r = 0; r < 19; ++r)
      for (int a = 0; a < 5; ++a) K0[r * 5 + a] = Mg[r][op.unk[a]];
    for (int a = 0; a < 5; ++a)
      for (int b = 0; b < 5; ++b) {
        double s = 0;
        for (int r = 0; r < 19; ++r) s += K0[r * 5 + a] * K0[r * 5 + b];
        G[a * 5 + b] = s;
      }
    invert(5, G, H);
    for (int a = 0; a < 5; ++a)
      for (int r = 0; r < 19; ++r) {
        double s = 0;
        for (int b = 0; b < 5; ++b) s += H[a * 5 + b] * K0[r * 5 + b];
        HK[a * 19 + r] = s;
      }
    double Qcn[19], Q1[19];
    for (int r = 0; r < 19; ++r) {
      double s = 0, t = 0;
      for (int c = 0; c < 19; ++c) {
        double kk = 0;
        for (int a = 0; a < 5; ++a) kk += K0[r * 5 + a] * HK[a * 19 + c];
        const double q = (r == c ? 1.0 : 0.0) - kk;
        s += q * cn[c];
        t += q;
      }
      Qcn[r] = s;
      Q1[r] = t;
    }
    op.A0 = op.A1 = op.A2 = 0;
    for (int r = 0; r < 19; ++r) {
      op.A0 += cn[r] * Qcn[r];
      op.A1 += cn[r] * Q1[r];
      op.A2 += Q1[r];
    }
    for (int q = 0; q < 19; ++q) {
      double ga = 0, ge = 0;
      if (cn[q] <= 0)
        for (int r = 0; r < 19; ++r) {
          ga += Qcn[r] * Mg[r][q];
          ge += Q1[r] * Mg[r][q];
        }
      op.ga[q] = ga;
      op.ge[q] = ge;
    }
    for (int a = 0; a < 5; ++a) {
      double hc = 0, h1 = 0;
      for (int r = 0; r < 19; ++r) {
        hc += HK[a * 19 + r] * cn[r];
        h1 += HK[a * 19 + r];
      }
      op.hc[a] = hc;
      op.h1[a] = h1;
      for (int q = 0; q < 19; ++q) {
        double t = 0;
        if (cn[q] <= 0)
          for (int r = 0; r < 19; ++r) t += HK[a * 19 + r] * Mg[r][q];
        op.Lg0[a][q] = -t;
      }
    }
  }
}

// index of a lattice velocity
int dir19(int x, int y, int z) {
  for (int q = 0; q < 19; ++q)
    if (C19[q][0] == x && C19[q][1] == y && C19[q][2] == z) return q;
  return -1;
}
}  // namespace

// The +x operator in the combinations that the symmetries of the face leave
// (t1 = y, t2 = z); entries equal by symmetry are averaged.
void build_face_fill(double A, double Bf, FaceFillT<double>& F) {
  FaceOp3 op;
  build_face_op(A, Bf, op);
  std::memset(&F, 0, sizeof F);
  const double w1 = 1.0 / 18, w2 = 1.0 / 36;
  // positions of the unknown directions n, n +- t1, n +- t2
  int u[5];
  const int un[5][3] = {{1, 0, 0}, {1, 1, 0}, {1, -1, 0}, {1, 0, 1}, {1, 0, -1}};
  for (int e = 0; e < 5; ++e)
    for (int a = 0; a < 5; ++a)
      if (op.unk[a] == dir19(un[e][0], un[e][1], un[e][2])) u[e] = a;
  auto sum4 = [](const double* r, const int (&d)[4][3]) {
    double s = 0;
    for (const auto& v : d) s += r[dir19(v[0], v[1], v[2])];
    return 0.25 * s;
  };
  const int tang[4][3] = {{0, 1, 0}, {0, -1, 0}, {0, 0, 1}, {0, 0, -1}};
  const int diag[4][3] = {{0, 1, 1}, {0, 1, -1}, {0, -1, 1}, {0, -1, -1}};
  const int inw[4][3] = {{-1, 1, 0}, {-1, -1, 0}, {-1, 0, 1}, {-1, 0, -1}};
  auto even = [&](const double* r, double e[5]) {
    e[0] = r[0];
    e[1] = sum4(r, tang);
    e[2] = sum4(r, diag);
    e[3] = r[dir19(-1, 0, 0)];
    e[4] = sum4(r, inw);
  };
  // Y, Z1 + Z2 (even), Z1 - Z2 and X1 (odd in t1) of a 5 x 19 map
  auto split = [&](const double L[5][19], double Y[5], double* Zs, double* Zd, double X[3]) {
    double y[19], zs[19], zd[19], x[19];
    for (int q = 0; q < 19; ++q) {
      const double z1 = w2 * (L[u[1]][q] + L[u[2]][q]), z2 = w2 * (L[u[3]][q] + L[u[4]][q]);
      zs[q] = z1 + z2;
      zd[q] = z1 - z2;
      y[q] = w1 * L[u[0]][q] + z1 + z2;
      x[q] = w2 * (L[u[1]][q] - L[u[2]][q]);
    }
    even(y, Y);
    if (Zs) even(zs, Zs);
    if (Zd) {
      Zd[0] = 0.25 * (zd[dir19(0, 1, 0)] + zd[dir19(0, -1, 0)] - zd[dir19(0, 0, 1)] -
                      zd[dir19(0, 0, -1)]);
      Zd[1] = 0.25 * (zd[dir19(-1, 1, 0)] + zd[dir19(-1, -1, 0)] - zd[dir19(-1, 0, 1)] -
                      zd[dir19(-1, 0, -1)]);
    }
    X[0] = 0.5 * (x[dir19(0, 1, 0)] - x[dir19(0, -1, 0)]);
    X[1] = 0.25 * (x[dir19(0, 1, 1)] + x[dir19(0, 1, -1)] - x[dir19(0, -1, 1)] -
                   x[dir19(0, -1, -1)]);
    X[2] = 0.5 * (x[dir19(-1, 1, 0)] - x[dir19(-1, -1, 0)]);
  };
  for (int v = 0; v < 2; ++v) {
    split(op.Lf[v], F.Y[v], F.Zs[v], F.Zd[v], F.X[v]);
    for (int e = 1; e < 5; ++e) {
      F.Zss[v] += w2 * op.Ls[v][u[e]];
      F.Zsk[v] += w2 * op.Lk[v][u[e]];
    }
    F.Ys[v] = w1 * op.Ls[v][u[0]] + F.Zss[v];
    F.Yk[v] = w1 * op.Lk[v][u[0]] + F.Zsk[v];
  }
  split(op.Ld, F.Dy, nullptr, nullptr, F.Dx);
  split(op.Lg0, F.Gy, nullptr, nullptr, F.Gx);
  even(op.ga, F.ka);
  even(op.ge, F.ke);
  F.A0 = op.A0;
  F.A1 = op.A1;
  F.A2 = op.A2;
  F.Hc = w1 * op.hc[u[0]];
  F.H1 = w1 * op.h1[u[0]];
  for (int e = 1; e < 5; ++e) {
    F.Hc += w2 * op.hc[u[e]];
    F.H1 += w2 * op.h1[u[e]];
  }
}

}  // namespace lks
