// Per-Fourier-mode radial solves on gfx950 (section 2.2 of the nsCouette
// paper: the linear terms are independent per mode).  All FP64.
//
// Operators (q = azimuthal order of the family, kappa = k kz):
//   L_q = D2 + R^-1 D1 - q^2 R^-2 - kappa^2 I  (nine-point rows)
//   Helmholtz  H = alpha I - beta L_q, identity (Dirichlet) wall rows;
//   Poisson    L_q with D1 (Neumann) wall rows;
//   mean head  (D2 + D1/r) rows, p(r_i) = 0 in row 0, D1 row at r_o.
// Factors: LU without pivoting (growth factor < 1 on these operators), kept
// in the matrix envelope: row j stores L_{j,j-4..j-1}, 1/U_jj, U_{j,j+1..j+4}
// plus the wider one-sided rows 0..3 (U up to column 8) and N-4..N-1 (L from
// column N-9).  One thread per operator (factor) or per mode (solve); modes
// are laid out so that a wavefront's lanes read consecutive addresses.
#include <cfloat>

#include <type_traits>

#include "solve_common.h"

namespace nsc {
namespace {

// Matrix entry A[i][c] of an operator for c in the window of row i.  pipe:
// row 0 is an inner row (the axis is no boundary) and the derivative rows
// are those of the operator's parity (off: their element offset).
struct OpRow {
  int kind;
  double alpha, beta, q2, k2;
  int pipe, off;
  __device__ __forceinline__ void row(const Grid &g, int n, int i, double *a, int &s) const {
    s = g.s[i];
    const double *w1 = g.d1 + off + i * kStencil;
    const double *w2 = g.d2 + off + i * kStencil;
    const double ri = g.rinv[i];
    const bool inner_wall = i == 0 && !pipe;
    if (kind == OP_HELMHOLTZ) {
      if (inner_wall || i == n - 1) {
#pragma unroll
        for (int t = 0; t < kStencil; ++t) a[t] = (s + t == i) ? 1.0 : 0.0;
        return;
      }
#pragma unroll
      for (int t = 0; t < kStencil; ++t) {
        double v = -beta * (w2[t] + w1[t] * ri);
        if (s + t == i) v += alpha + beta * (q2 * ri * ri + k2);
        a[t] = v;
      }
    } else if (kind == OP_POISSON) {
      if (inner_wall || i == n - 1) {
#pragma unroll
        for (int t = 0; t < kStencil; ++t) a[t] = w1[t];
        return;
      }
#pragma unroll
      for (int t = 0; t < kStencil; ++t) {
        double v = w2[t] + w1[t] * ri;
        if (s + t == i) v -= q2 * ri * ri + k2;
        a[t] = v;
      }
    } else {  // mean pressure head: (D2 + D1/r) p inside, p(r_i) = 0, D1 row at r_o
              // (pipe: p = 0 at the wall, the axis no boundary)
      if (inner_wall || (pipe && i == n - 1)) {
#pragma unroll
        for (int t = 0; t < kStencil; ++t) a[t] = (s + t == i) ? 1.0 : 0.0;
        return;
      }
      if (i == n - 1) {
#pragma unroll
        for (int t = 0; t < kStencil; ++t) a[t] = w1[t];
        return;
      }
#pragma unroll
      for (int t = 0; t < kStencil; ++t) a[t] = w2[t] + w1[t] * ri;
    }
  }
};

// LU factors of every operator, one lane per operator (op = q*(K+1) + |k|),
// row by row: row i subtracts the L_ik-fold of the finished U rows k of its
// window, whose fill stays inside it (no pivoting).  blockIdx.y picks one of
// two operator sets of the same kind and shift (velocity and temperature
// Helmholtz operators differ only in beta): both factorise in one launch.
//
// Rows 8 .. N-5 only need the last four U rows, kept in registers and turned
// over by unrolling four rows; their weights are loaded four rows ahead.  The
// first eight and last four rows read the U rows (up to eight entries there)
// from LDS, where each lane keeps its last eight.  One wavefront per compute
// unit is what the smaller grids have, so the time is one wavefront's
// instruction stream, and past about 16000 operators the factors' writes.
// Before (elimination of a nine-row window in LDS, the band entries also
// stored one array per entry) -> now: 32 x 16 x 16 operators' rows 58 -> 22 us,
// 64 x 64 x 64 twice (heated) 99 -> 30, 128 x 256 x 256 610 -> 145 to 175.
constexpr int kFacThreads = 64;
constexpr int kFacRow = 10;  // LDS doubles per U row: U_{i,i+1..i+8}, 1/U_ii, pad

__global__ void __launch_bounds__(kFacThreads)
k_factor(Dims d, Grid g, Factors F0, Factors F1, int kind, double alpha, double beta0, double beta1) {
  __shared__ __align__(16) double ring[8 * kFacThreads * kFacRow];
  const Factors F = blockIdx.y == 0 ? F0 : F1;
  const double beta = blockIdx.y == 0 ? beta0 : beta1;
  const int tid = threadIdx.x;
  const int op = blockIdx.x * kFacThreads + tid;
  if (op >= F.nops) return;
  const int n = d.nr;
  const int kp1 = d.kmax + 1;
  const int q = op / kp1;
  const int ka = op - q * kp1;
  const double kap = (double)ka * d.kz;
  OpRow R{kind, alpha, beta, (double)q * (double)q, kap * kap, d.pipe, odd_off(g, q)};
  const size_t nops = F.nops;
  // the pure-Neumann Poisson operator of (q = 0, kappa = 0) is singular and
  // never used; its slot holds the mean pressure-head operator instead
  if (kind == OP_POISSON && q == 0 && ka == 0) R.kind = OP_MEAN_PRESSURE;
  auto slot = [&](int i) { return reinterpret_cast<Dbl2 *>(ring + ((i & 7) * kFacThreads + tid) * kFacRow); };
  // row i to memory: L_{i,i-4..i-1}, U_{i,i+1..i+4} and 1/U_ii
  auto store = [&](int i, const double (&lo)[4], const double (&up)[4], double dinv) {
    Dbl2 *o = reinterpret_cast<Dbl2 *>(F.pk + ((size_t)i * 2 * nops + op) * 4);
    o[0] = Dbl2{lo[0], lo[1]};
    o[1] = Dbl2{lo[2], lo[3]};
    o += 2 * nops;
    o[0] = Dbl2{up[0], up[1]};
    o[1] = Dbl2{up[2], up[3]};
    F.di[(size_t)i * nops + op] = dinv;
  };
  // a row by the ring, with its diagonal at entry D of its window
  auto ring_row = [&](auto diag, int i) {
    constexpr int D = decltype(diag)::value;
    double a[kStencil];
    int s;
    R.row(g, n, i, a, s);
#pragma unroll
    for (int t = 0; t < D; ++t) {
      const Dbl2 *u = slot(i - D + t);
      const Dbl2 u01 = u[0], u23 = u[1], u45 = u[2], u67 = u[3];
      const double uk[8] = {u01.x, u01.y, u23.x, u23.y, u45.x, u45.y, u67.x, u67.y};
      a[t] *= u[4].x;
#pragma unroll
      for (int c = t + 1; c < kStencil; ++c) a[c] -= a[t] * uk[c - t - 1];
    }
    const double dinv = 1.0 / a[D];
    double lo[4], uk[8];
#pragma unroll
    for (int t = 0; t < 4; ++t) lo[t] = D - 4 + t >= 0 ? a[D - 4 + t < 0 ? 0 : D - 4 + t] : 0.0;
#pragma unroll
    for (int t = 0; t < 8; ++t) uk[t] = D + 1 + t < kStencil ? a[D + 1 + t < kStencil ? D + 1 + t : 0] : 0.0;
    const double up[4] = {uk[0], uk[1], uk[2], uk[3]};
    store(i, lo, up, dinv);
    Dbl2 *u = slot(i);
    u[0] = Dbl2{uk[0], uk[1]};
    u[1] = Dbl2{uk[2], uk[3]};
    u[2] = Dbl2{uk[4], uk[5]};
    u[3] = Dbl2{uk[6], uk[7]};
    u[4] = Dbl2{dinv, 0.0};
    // entries past the band: U of rows 0..3, L of rows N-4..N-1
#pragma unroll
    for (int c = D + 5; c < kStencil; ++c)
      F.edge[(size_t)(edge_off(D) + c - (D + 5)) * nops + op] = a[c];
#pragma unroll
    for (int c = 0; c <= D - 5; ++c)
      F.edge[(size_t)(10 + edge_off(8 - D) + c) * nops + op] = a[c];
  };
  ring_row(std::integral_constant<int, 0>{}, 0);
  ring_row(std::integral_constant<int, 1>{}, 1);
  ring_row(std::integral_constant<int, 2>{}, 2);
  ring_row(std::integral_constant<int, 3>{}, 3);
  int i = 4;
  for (; i < 8 && i < n - 4; ++i) ring_row(std::integral_constant<int, 4>{}, i);
  if (i + 4 <= n - 4) {
    // rows i .. i+3, the U rows of i-4 .. i-1 in registers
    double uk[4][4], dv[4], w[4][kStencil], ri[4];
    auto weights = [&](int r, int j) {
      const double *p = g.lw + R.off + (j < n ? j : n - 1) * kStencil;
#pragma unroll
      for (int t = 0; t < kStencil; ++t) w[r][t] = p[t];
      ri[r] = g.rinv[j < n ? j : n - 1];
    };
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const Dbl2 *u = slot(4 + r);
      const Dbl2 u01 = u[0], u23 = u[1];
      uk[r][0] = u01.x;
      uk[r][1] = u01.y;
      uk[r][2] = u23.x;
      uk[r][3] = u23.y;
      dv[r] = u[4].x;
      weights(r, i + r);
    }
    const double f = kind == OP_HELMHOLTZ ? -beta : 1.0;
    for (; i + 4 <= n - 4; i += 4) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        double a[kStencil];
#pragma unroll
        for (int t = 0; t < kStencil; ++t) a[t] = f * w[r][t];
        const double sh = R.q2 * ri[r] * ri[r] + R.k2;
        a[4] = kind == OP_HELMHOLTZ ? a[4] + (alpha + beta * sh) : a[4] - sh;
        weights(r, i + r + 4);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int k = (r + t) & 3;  // U row i + r - 4 + t
          a[t] *= dv[k];
#pragma unroll
          for (int c = 0; c < 4; ++c) a[t + 1 + c] -= a[t] * uk[k][c];
        }
        const double dinv = 1.0 / a[4];
        const double lo[4] = {a[0], a[1], a[2], a[3]};
        dv[r] = dinv;
#pragma unroll
        for (int c = 0; c < 4; ++c) uk[r][c] = a[5 + c];
        store(i + r, lo, uk[r], dinv);
        if (i >= n - 16) {  // within reach of the last rows
          Dbl2 *u = slot(i + r);
          u[0] = Dbl2{uk[r][0], uk[r][1]};
          u[1] = Dbl2{uk[r][2], uk[r][3]};
          u[2] = u[3] = Dbl2{0.0, 0.0};
          u[4] = Dbl2{dinv, 0.0};
        }
      }
    }
  }
  for (; i < n - 4; ++i) ring_row(std::integral_constant<int, 4>{}, i);
  ring_row(std::integral_constant<int, 5>{}, n - 4);
  ring_row(std::integral_constant<int, 6>{}, n - 3);
  ring_row(std::integral_constant<int, 7>{}, n - 2);
  ring_row(std::integral_constant<int, 8>{}, n - 1);
}

// Rows of the packed factors of one operator.
struct RowL {
  double l4, l3, l2, l1;  // L_{j,j-4..j-1}
};
struct RowU {
  double u1, u2, u3, u4;  // U_{j,j+1..j+4}
};
struct RowsOf {
  const double *pk, *di;
  size_t nops;
  __device__ __forceinline__ RowsOf(const Factors &F, int op)
      : pk(F.pk + (size_t)op * 4), di(F.di + op), nops(F.nops) {}
  __device__ __forceinline__ RowL l(int j) const {
    const Dbl2 *p = reinterpret_cast<const Dbl2 *>(pk + (size_t)j * 8 * nops);
    const Dbl2 a = p[0], b = p[1];
    return {a.x, a.y, b.x, b.y};
  }
  __device__ __forceinline__ RowU u(int j) const {
    const Dbl2 *p = reinterpret_cast<const Dbl2 *>(pk + ((size_t)j * 2 + 1) * 4 * nops);
    const Dbl2 a = p[0], b = p[1];
    return {a.x, a.y, b.x, b.y};
  }
  __device__ __forceinline__ double dinv(int j) const { return di[(size_t)j * nops]; }
};

// Forward/back substitution for one lane.  RHS(j) gives b_j, COL(j) the
// storage of y_j then x_j (LDS or global, read back by the same lane).  The
// bulk rows carry no branches: the envelope slots outside the matrix are
// stored as zeros, so every row issues the same independent loads and the
// compiler can schedule them ahead of the recurrence; only the one-sided
// wall rows (U to column 8 in rows 0..3, L from column N-9 in rows N-4..N-1)
// take the extra edge terms, in peeled loops.
// The factor rows are loaded AHEAD rows before their use.
template <typename V, int AHEAD = 4, typename RHS, typename COL>
__device__ __forceinline__ void lu_solve(const Factors &F, int op, int n, RHS rhs, COL col) {
  const size_t nops = F.nops;
  const RowsOf R(F, op);
  const double *__restrict__ edge = F.edge + op;
  {
    V y1{}, y2{}, y3{}, y4{};
    RowL v[AHEAD];
#pragma unroll
    for (int r = 0; r < AHEAD; ++r) v[r] = R.l(r < n ? r : n - 1);
    auto row = [&](const RowL &l, int j) {
      V y = rhs(j);
      y = y - l.l1 * y1;
      y = y - l.l2 * y2;
      y = y - l.l3 * y3;
      y = y - l.l4 * y4;
      y4 = y3;
      y3 = y2;
      y2 = y1;
      y1 = y;
      col(j) = y;
    };
    int j = 0;
    for (; j + AHEAD <= n - 4; j += AHEAD) {
#pragma unroll
      for (int r = 0; r < AHEAD; ++r) {
        const RowL l = v[r];
        v[r] = R.l(j + AHEAD + r < n ? j + AHEAD + r : n - 1);
        row(l, j + r);
      }
    }
#pragma unroll
    for (int r = 0; r < AHEAD; ++r)
      if (j + r < n - 4) row(v[r], j + r);
  }
#pragma unroll
  for (int tt = 3; tt >= 0; --tt) {
    const int j = n - 1 - tt;
    const RowL v = R.l(j);
    V y = rhs(j);
    y = y - v.l1 * col(j - 1);
    y = y - v.l2 * col(j - 2);
    y = y - v.l3 * col(j - 3);
    y = y - v.l4 * col(j - 4);
#pragma unroll
    for (int c = 0; c <= 3 - tt; ++c) y = y - edge[(size_t)(10 + edge_off(tt) + c) * nops] * col(n - 9 + c);
    col(j) = y;
  }
  {
    V x1{}, x2{}, x3{}, x4{};
    RowU v[AHEAD];
    double di[AHEAD];
#pragma unroll
    for (int r = 0; r < AHEAD; ++r) {
      const int a = n - 1 - r > 0 ? n - 1 - r : 0;
      v[r] = R.u(a);
      di[r] = R.dinv(a);
    }
    auto row = [&](const RowU &u, double d, int j) {
      V x = col(j);
      x = x - u.u1 * x1;
      x = x - u.u2 * x2;
      x = x - u.u3 * x3;
      x = x - u.u4 * x4;
      x = d * x;
      x4 = x3;
      x3 = x2;
      x2 = x1;
      x1 = x;
      col(j) = x;
    };
    int j = n - 1;
    for (; j - AHEAD >= 3; j -= AHEAD) {
#pragma unroll
      for (int r = 0; r < AHEAD; ++r) {
        const RowU u = v[r];
        const double d = di[r];
        const int a = j - AHEAD - r > 0 ? j - AHEAD - r : 0;
        v[r] = R.u(a);
        di[r] = R.dinv(a);
        row(u, d, j - r);
      }
    }
#pragma unroll
    for (int r = 0; r < AHEAD; ++r)
      if (j - r >= 4) row(v[r], di[r], j - r);
  }
#pragma unroll
  for (int j = 3; j >= 0; --j) {
    const RowU v = R.u(j);
    V x = col(j);
    x = x - v.u1 * col(j + 1);
    x = x - v.u2 * col(j + 2);
    x = x - v.u3 * col(j + 3);
    x = x - v.u4 * col(j + 4);
#pragma unroll
    for (int c = j + 5; c <= 8; ++c) x = x - edge[(size_t)(edge_off(j) + c - (j + 5)) * nops] * col(c);
    col(j) = R.dinv(j) * x;
  }
}

__device__ __forceinline__ Cd d1_row(const Grid &g, int j, const Cd *x, size_t stride, int off = 0) {
  const int s = g.s[j];
  const double *w = g.d1 + off + j * kStencil;
  Cd acc = {0.0, 0.0};
#pragma unroll
  for (int t = 0; t < kStencil; ++t) acc = fmac(w[t], x[(size_t)(s + t) * stride], acc);
  return acc;
}

// Homogeneous responses and inverse influence matrices per (m, |k|), in
// two parts: the pressure responses p_j (Neumann data e_0, e_{N-1}; do not
// depend on the step size, computed once), then the six velocity responses
// (X+, X-, h for each p_j) and the 2x2 influence matrices.  The two responses
// of an operator are solved together, as the parts of a complex number, so that
// a lane reads each factor row once for both.
__global__ void __launch_bounds__(64) k_influence_p(Dims d, Factors fp, Influence I) {
  const int op = blockIdx.x * blockDim.x + threadIdx.x;
  if (op >= I.nops) return;
  const int n = d.nr;
  const int kp1 = d.kmax + 1;
  const int m = op / kp1;
  const int ka = op - m * kp1;
  const size_t ns = I.nops;
  Cd *P = reinterpret_cast<Cd *>(I.resp) + op;
  if (m == 0 && ka == 0) {
    for (int j = 0; j < n; ++j) P[(size_t)j * ns] = Cd{0.0, 0.0};
    return;
  }
  lu_solve<Cd>(fp, op, n, [&](int j) { return Cd{j == 0 ? 1.0 : 0.0, j == n - 1 ? 1.0 : 0.0}; },
               [&](int j) -> Cd & { return P[(size_t)j * ns]; });
}

// Right sides of the velocity responses of pressure p:
// X+ = H_{m+1}^-1 (-(D1 p - m p / r)), X- = H_{|m-1|}^-1 (-(D1 p + m p / r)),
// h = H_m^-1 p so that X_z = -i kappa h (kind 0, 1, 2)
__device__ __forceinline__ Cd response_rhs(const Dims &d, const Grid &g, int kind, int m, int j, const Cd *p,
                                           size_t stride) {
  if ((j == 0 && !d.pipe) || j == d.nr - 1) return Cd{0.0, 0.0};
  const Cd pj = p[(size_t)j * stride];
  if (kind == 2) return pj;
  const Cd dp = d1_row(g, j, p, stride, odd_off(g, m));  // p of order m
  const Cd mp = ((double)m * g.rinv[j]) * pj;
  return kind == 0 ? Cd{0.0, 0.0} - (dp - mp) : Cd{0.0, 0.0} - (dp + mp);
}
// Azimuthal order of a response's operator
__device__ __forceinline__ int response_q(int kind, int m) {
  return kind == 0 ? m + 1 : (kind == 1 ? (m >= 1 ? m - 1 : 1 - m) : m);
}

// Inverse influence matrix of one operator from its responses' columns
// (rows strided by `stride`).
__device__ __forceinline__ void influence_matrix(const Dims &d, const Grid &g, const Influence &I, int op, int m,
                                                 const Cd *Xp, const Cd *Xm, size_t stride) {
  const size_t ns = I.nops;
  const int n = d.nr;
  const double mm = (double)m;
  // A[w][jj] = wall divergence of response jj (walls carry zero velocity)
  double A[2][2];
  const int off = odd_off(g, m + 1);  // X+- of orders m +- 1
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    const int j = w == 0 ? 0 : n - 1;
    const double ri = g.rinv[j];
    const Cd v = 0.5 * ((d1_row(g, j, Xp, stride, off) + ((1.0 + mm) * ri) * Xp[(size_t)j * stride]) +
                        (d1_row(g, j, Xm, stride, off) + ((1.0 - mm) * ri) * Xm[(size_t)j * stride]));
    A[w][0] = v.x;
    A[w][1] = v.y;
  }
  if (d.pipe) {
    // one wall: the first condition becomes lambda_1 = 0 (k_influence gives
    // it a zero right side), the second is the wall's
    A[0][0] = 1.0;
    A[0][1] = 0.0;
  }
  const double det = A[0][0] * A[1][1] - A[0][1] * A[1][0];
  const bool mean = m == 0 && op == 0;  // (0, 0) has no influence matrix
  I.ainv[0 * ns + op] = mean ? 0.0 : A[1][1] / det;
  I.ainv[1 * ns + op] = mean ? 0.0 : -A[0][1] / det;
  I.ainv[2 * ns + op] = mean ? 0.0 : -A[1][0] / det;
  I.ainv[3 * ns + op] = mean ? 0.0 : A[0][0] / det;
}

// Velocity responses and influence matrices of sixteen operators per
// workgroup.  All threads load the pressure columns and form the right sides
// in LDS; three wavefronts then solve one kind each in place, one lane per
// operator, the factor rows loaded eight ahead; all threads write the columns out.
// What bounds it is the serial sweep of a lane.
// Before (one lane per operator and kind with its own LDS columns, the matrices
// in a second kernel) -> now: 32 x 16 x 16 31 -> 15 us, 64 x 64 x 64 51 -> 22;
// 128 x 256 x 256 720 -> 670 (one workgroup per compute unit). With eight
// operators per workgroup: 15, 34 and 839 us.
constexpr int kInfOps = 16;
constexpr int kInfThreads = 256;

__global__ void __launch_bounds__(kInfThreads) k_influence_v(Dims d, Grid g, Factors fv, Influence I) {
  extern __shared__ __align__(16) Cd inf_lds[];  // [p, X+, X-, h][N_r][kInfOps]
  constexpr int groups = kInfThreads / kInfOps;
  const int t = threadIdx.x, o = t % kInfOps;
  const int op = blockIdx.x * kInfOps + o;
  const bool live = op < I.nops;
  const int n = d.nr;
  const int kp1 = d.kmax + 1;
  const int opc = live ? op : I.nops - 1;
  const int m = opc / kp1;
  const int ka = opc - m * kp1;
  const size_t ns = I.nops;
  Cd *resp = reinterpret_cast<Cd *>(I.resp) + opc;
  Cd *col = inf_lds + o;
  const size_t fs = (size_t)n * kInfOps;  // between the columns of one kind and the next
#pragma unroll 4
  for (int j = t / kInfOps; j < n; j += groups) col[j * kInfOps] = resp[(size_t)j * ns];
  __syncthreads();
  for (int j = t / kInfOps; j < n; j += groups)
#pragma unroll
    for (int kind = 0; kind < 3; ++kind)
      col[(1 + kind) * fs + j * kInfOps] = response_rhs(d, g, kind, m, j, col, kInfOps);
  __syncthreads();
  const int kind = t / 64;
  if (kind < 3 && t % 64 < kInfOps) {
    Cd *x = col + (1 + kind) * fs;
    lu_solve<Cd, 8>(fv, response_q(kind, m) * kp1 + ka, n, [&](int j) { return x[j * kInfOps]; },
                     [&](int j) -> Cd & { return x[j * kInfOps]; });
  }
  __syncthreads();
  if (!live) return;
  // (0, 0): no pressure response, zero columns
#pragma unroll
  for (int kd = 0; kd < 3; ++kd)
    for (int j = t / kInfOps; j < n; j += groups)
      resp[((size_t)(1 + kd) * n + j) * ns] = col[(1 + kd) * fs + j * kInfOps];
  if (t < kInfOps) influence_matrix(d, g, I, op, m, col + fs, col + 2 * fs, kInfOps);
}

// The same in two kernels, columns in global memory, for columns past the LDS.
__global__ void __launch_bounds__(64) k_influence_x(Dims d, Grid g, Factors fv, Influence I) {
  const int op = blockIdx.x * blockDim.x + threadIdx.x;
  const int kind = blockIdx.y;
  if (op >= I.nops) return;
  const int n = d.nr;
  const int kp1 = d.kmax + 1;
  const int m = op / kp1;
  const int ka = op - m * kp1;
  const size_t ns = I.nops;
  const Cd *p = reinterpret_cast<const Cd *>(I.resp) + op;
  Cd *out = reinterpret_cast<Cd *>(I.resp) + op + (size_t)(1 + kind) * n * ns;
  lu_solve<Cd>(fv, response_q(kind, m) * kp1 + ka, n, [&](int j) { return response_rhs(d, g, kind, m, j, p, ns); },
               [&](int j) -> Cd & { return out[(size_t)j * ns]; });
}

__global__ void __launch_bounds__(64) k_influence_a(Dims d, Grid g, Influence I) {
  const int op = blockIdx.x * blockDim.x + threadIdx.x;
  if (op >= I.nops) return;
  const size_t ns = I.nops;
  const Cd *Xp = reinterpret_cast<const Cd *>(I.resp) + (size_t)d.nr * ns + op;
  influence_matrix(d, g, I, op, op / (d.kmax + 1), Xp, Xp + (size_t)d.nr * ns, ns);
}

// Nine-point stencil sums over R consecutive rows j0 .. j0+nrow-1 of NF
// fields (field f at x + f * fstride, rows strided by P), with the weights w
// ([N_r][9], row j's window starting at s_j): acc[f][jj] = sum_t
// w[j][t] x_f[s_j + t], summed from the left as a single row would, and
// cen[f][jj] = x_f[j].  The rows the windows share are read once: R + 8 rows
// when every window is centred, from the first window's start to the last
// window's end otherwise.
template <int R, int NF>
__device__ __forceinline__ void stencil_rows(const Grid &g, const double *__restrict__ w, int n,
                                             int j0, int nrow, const double2 *x, size_t fstride,
                                             size_t P, Cd (&acc)[NF][R], Cd (&cen)[NF][R]) {
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int jj = 0; jj < R; ++jj) acc[f][jj] = cen[f][jj] = Cd{0, 0};
  if (j0 >= 4 && j0 + R - 1 <= n - 5) {
    // row j0+jj reads rows j0+jj-4 .. j0+jj+4
#pragma unroll
    for (int rr = 0; rr < R + kStencil - 1; ++rr) {
      const size_t r = (size_t)(j0 - 4 + rr);
      Cd xv[NF];
#pragma unroll
      for (int f = 0; f < NF; ++f) xv[f] = ld(x + f * fstride + r * P);
#pragma unroll
      for (int jj = 0; jj < R; ++jj) {
        const int t = rr - jj;
        if (t >= 0 && t < kStencil) {
          const double wt = w[(j0 + jj) * kStencil + t];
#pragma unroll
          for (int f = 0; f < NF; ++f) acc[f][jj] = fmac(wt, xv[f], acc[f][jj]);
        }
        if (t == 4)
#pragma unroll
          for (int f = 0; f < NF; ++f) cen[f][jj] = xv[f];
      }
    }
  } else {
    const int lo = g.s[j0];
    const int hi = g.s[j0 + nrow - 1] + kStencil;
    for (int r = lo; r < hi; ++r) {
      Cd xv[NF];
#pragma unroll
      for (int f = 0; f < NF; ++f) xv[f] = ld(x + f * fstride + (size_t)r * P);
#pragma unroll
      for (int jj = 0; jj < R; ++jj) {
        const int j = j0 + jj;
        if (jj < nrow) {
          const int t = r - g.s[j];
          if (t >= 0 && t < kStencil) {
            const double wt = w[j * kStencil + t];
#pragma unroll
            for (int f = 0; f < NF; ++f) acc[f][jj] = fmac(wt, xv[f], acc[f][jj]);
          }
          if (r == j)
#pragma unroll
            for (int f = 0; f < NF; ++f) cen[f][jj] = xv[f];
        }
      }
    }
  }
}

// f_X = X^n/dt + (1-c) L_q X^n + c N^q + (1-c) N^n for X in {+, -, z, T}.
// blockIdx.z: 0 the +- pair (from u_r, u_theta), 1 u_z, 2 T -- one stencil
// family per thread keeps the registers (and so the occupancy) of a
// memory-bound kernel moderate.  blockIdx.y: a chunk of R rows per lane.
template <int R, bool PIPE = false>
__global__ void __launch_bounds__(256) k_rhs(Dims d, Grid g, const double2 *__restrict__ u,
                      const double2 *__restrict__ nn, const double2 *__restrict__ nq,
                      double2 *__restrict__ sf, double idt, double cc, int rows_first) {
  int bx, cy, part;
  stencil_block(rows_first, bx, cy, part);
  const int md = bx * blockDim.x + threadIdx.x;
  if (md >= d.nmodes) return;
  const size_t P = d.nmodes;
  const int n = d.nr;
  const int j0 = cy * R;
  const int nrow = n - j0 < R ? n - j0 : R;
  const int m = md / d.mz;
  const int kk = md - m * d.mz;
  const double kap = (double)(kk - d.kmax) * d.kz;
  const double ce = 1.0 - cc;
  const double k2 = kap * kap;
  const size_t fs = (size_t)n * P;  // field stride
  auto N = [&](int f, int j) -> Cd {
    if (!nn) return Cd{0, 0};
    const size_t o = ((size_t)f * n + j) * P + md;
    return cc * ld(nq + o) + ce * ld(nn + o);
  };
  if (part == 0) {
    // stencil sums of (D2 + D1/r) applied to u_r and u_theta (pipe: the
    // rows of parity (-1)^(m+1), per lane)
    Cd l[2][R], x[2][R];
    stencil_rows<R, 2>(g, PIPE ? g.lw + odd_off(g, m + 1) : g.lw, n, j0, nrow, u + md, fs, P, l, x);
    const double qp = (double)(m + 1), qm = (double)(m >= 1 ? m - 1 : 1 - m);
#pragma unroll
    for (int jj = 0; jj < R; ++jj) {
      if (jj >= nrow) break;
      const int j = j0 + jj;
      const double ri = g.rinv[j];
      const double r2 = ri * ri;
      const Cd lr = l[0][jj], lt = l[1][jj];
      const Cd ur = x[0][jj], ut = x[1][jj];
      const Cd xp = ur + ci(ut), xm = ur - ci(ut);
      const Cd lp = lr + ci(lt), lm = lr - ci(lt);
      const Cd Lp = lp - (qp * qp * r2 + k2) * xp;
      const Cd Lm = lm - (qm * qm * r2 + k2) * xm;
      const Cd a = N(0, j), b = N(1, j);
      st(sf + ((size_t)0 * n + j) * P + md, idt * xp + ce * Lp + (a + ci(b)));
      st(sf + ((size_t)1 * n + j) * P + md, idt * xm + ce * Lm + (a - ci(b)));
    }
  } else {
    // u_z (operator L_m) or T (L_m / Pr)
    const int f = part + 1;
    Cd l[1][R], x[1][R];
    stencil_rows<R, 1>(g, PIPE ? g.lw + odd_off(g, m) : g.lw, n, j0, nrow, u + f * fs + md, fs, P,
                       l, x);
    const double cf = f == 3 ? ce / d.pr : ce;
#pragma unroll
    for (int jj = 0; jj < R; ++jj) {
      if (jj >= nrow) break;
      const int j = j0 + jj;
      const double ri = g.rinv[j];
      const double r2 = ri * ri;
      const Cd Lx = l[0][jj] - ((double)m * (double)m * r2 + k2) * x[0][jj];
      st(sf + ((size_t)f * n + j) * P + md, idt * x[0][jj] + cf * Lx + N(f, j));
    }
  }
}

// ---------------------------------------------------------------------------
// Batched sweeps: one lane per (mode, system), the system's right side given
// column-wise in global memory (rows strided by the mode count); y and x stay
// in the output array.
// ---------------------------------------------------------------------------
struct SweepSys {
  Factors F;
  int qmode;   // 0: q = m, 1: q = m + 1, 2: q = |m - 1|
  int zero00;  // 1: mode (0,0) writes zeros (else its operator slot is used)
  const double2 *in;  // right side column base, rows strided by the mode count
  double2 *out;       // solution column base
};
struct SweepArgs {
  SweepSys s[3];
};
constexpr int kSweepLanes = 64;

// FAMILY only names the launch (0: pressure/temperature, 1: velocity), so
// that profiles tell the two apart; the code is the same.
template <int FAMILY>
__global__ void __launch_bounds__(kSweepLanes)
k_sweep(Dims d, SweepArgs a) {
  // logical (mode tile, system) after the XCD remap, system fastest: the
  // two halves of a tile row (m, +-k) use the same operators, and the
  // systems of neighbouring rows share them (q = m - 1, m, m + 1), so these
  // workgroups run next to each other on one XCD and read the factors from
  // its L2 instead of HBM
  const int L = xcd_remap(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
  const int sys = L % gridDim.y;
  const int md = (L / gridDim.y) * kSweepLanes + threadIdx.x;
  if (md >= d.nmodes) return;
  const SweepSys &S = a.s[sys];
  const size_t P = d.nmodes;
  const int n = d.nr;
  const int kp1 = d.kmax + 1;
  const int m = md / d.mz;
  const int kk = md - m * d.mz;
  const int ka = kk >= d.kmax ? kk - d.kmax : d.kmax - kk;
  const double2 *__restrict__ b = S.in + md;
  double2 *__restrict__ x = S.out + md;
  // one factor set for the whole workgroup (its base stays in scalar
  // registers); mode (0,0) of the pressure uses slot 0 of the same set,
  // which holds the mean pressure-head operator
  const Factors F = S.F;
  const int q = S.qmode == 0 ? m : (S.qmode == 1 ? m + 1 : (m >= 1 ? m - 1 : 1 - m));
  if (m == 0 && ka == 0 && S.zero00) {
    for (int j = 0; j < n; ++j) x[(size_t)j * P] = make_double2(0.0, 0.0);
    return;
  }
  lu_solve<Cd>(F, q * kp1 + ka, n, [&](int j) { return ld(b + (size_t)j * P); },
               [&](int j) -> Cd & { return *reinterpret_cast<Cd *>(x + (size_t)j * P); });
}

// Velocity right sides in place of f: f_X - (grad p0)_X inside, wall values
// on rows 0 and N-1; mode (0,0) solves u_theta directly (X+- = +-i u_theta).
// R consecutive rows per lane (blockIdx.y: the chunk).
template <int R, bool PIPE = false>
__global__ void __launch_bounds__(256)
k_vel_rhs(Dims d, Grid g, double2 *__restrict__ sf, const double2 *__restrict__ sp, int walls,
          int rows_first) {
  int bx, cy, unused;
  stencil_block(rows_first, bx, cy, unused);
  const int md = bx * blockDim.x + threadIdx.x;
  if (md >= d.nmodes) return;
  const size_t P = d.nmodes;
  const int n = d.nr;
  const int j0 = cy * R;
  const int nrow = n - j0 < R ? n - j0 : R;
  const int m = md / d.mz;
  const int kk = md - m * d.mz;
  const bool zero = (md == d.kmax);
  auto field = [&](int f, int j) { return sf + ((size_t)f * n + j) * P + md; };
  auto wall_row = [&](int j) {
    Cd wp = {0, 0};
    if (zero && walls) {
      const double re = j == 0 ? d.re_i : d.re_o;
      wp = {0.0, re};
    }
    st(field(0, j), wp);
    st(field(1, j), Cd{-wp.x, -wp.y});
    st(field(2, j), Cd{0, 0});
  };
  if (zero) {
    for (int jj = 0; jj < nrow; ++jj) {
      const int j = j0 + jj;
      if ((j == 0 && !PIPE) || j == n - 1) {
        wall_row(j);
        continue;
      }
      const Cd h = 0.5 * (ld(field(0, j)) - ld(field(1, j)));
      st(field(0, j), h);
      st(field(1, j), Cd{-h.x, -h.y});
      // pipe: the driving pressure gradient in the axial mean flow
      if (PIPE && walls) st(field(2, j), ld(field(2, j)) + Cd{d.gp, 0.0});
    }
    return;
  }
  const double kap = (double)(kk - d.kmax) * d.kz;
  Cd dp[1][R], pc[1][R];
  stencil_rows<R, 1>(g, PIPE ? g.d1 + odd_off(g, m) : g.d1, n, j0, nrow, sp + md, 0, P, dp, pc);
#pragma unroll
  for (int jj = 0; jj < R; ++jj) {
    if (jj >= nrow) break;
    const int j = j0 + jj;
    if ((j == 0 && !PIPE) || j == n - 1) {
      wall_row(j);
      continue;
    }
    const Cd pj = pc[0][jj];
    const Cd mp = (m * g.rinv[j]) * pj;
    double2 *fp = field(0, j), *fm = field(1, j), *fz = field(2, j);
    st(fp, ld(fp) - (dp[0][jj] - mp));
    st(fm, ld(fm) - (dp[0][jj] + mp));
    st(fz, ld(fz) - kap * ci(pj));
  }
}

// Poisson right side g = mask(div f) at one (mode, row) where no divergence
// is formed: every row of mode (0,0), which takes the mean-head right side
// (D1 + 1/r) F_r inside and F_r(r_o) at the outer wall (zeros if not
// requested), and the wall rows of the other modes (zero).  Heated: the wall
// rows of f_T are replaced by the wall values (+-1/2 in (0,0), zero
// elsewhere; all zero for walls = 0) in the same pass.
__device__ __forceinline__ void div_row(const Dims &d, const Grid &g, double2 *__restrict__ sf,
                                        double2 *__restrict__ sg, const double2 *__restrict__ nn,
                                        const double2 *__restrict__ nq, double cc, int want_p,
                                        int walls, int md, int j) {
  const size_t P = d.nmodes;
  const int n = d.nr;
  if (d.heated && (j == 0 || j == n - 1)) {
    const bool mean = (md == d.kmax) && walls;
    st(sf + ((size_t)3 * n + j) * P + md, Cd{mean ? (j == 0 ? 0.5 : -0.5) : 0.0, 0.0});
  }
  if (md == d.kmax) {
    // (pipe: every row but the wall's, where p = 0; F_r odd in r)
    Cd r = {0, 0};
    if (want_p && nn && (j > 0 || d.pipe) && !(d.pipe && j == n - 1)) {
      auto Fr = [&](int t) {
        return cc * ld(nq + (size_t)t * P + md) + (1.0 - cc) * ld(nn + (size_t)t * P + md);
      };
      if (j == n - 1) {
        r = Fr(n - 1);
      } else {
        const int s0 = g.s[j];
        const double *w = g.d1 + g.podd + j * kStencil;
        r = g.rinv[j] * Fr(j);
        for (int t = 0; t < kStencil; ++t) r = fmac(w[t], Fr(s0 + t), r);
      }
    }
    st(sg + (size_t)j * P + md, r);
    return;
  }
  st(sg + (size_t)j * P + md, Cd{0, 0});  // wall rows of the other modes
}

// Poisson right side g = mask(div f) = (D1 + (1+m)/r) F_+ / 2 + (D1 + (1-m)/r)
// F_- / 2 + i kappa F_z over R consecutive rows per lane: the rows of F_+
// and F_- that the rows' nine-point windows share are read once (R + 8 rows
// for R outputs inside, fewer at the walls) instead of nine times, and each
// derivative still sums its window from the left, as a single row would.
template <int R, bool PIPE = false>
__global__ void __launch_bounds__(256)
k_div2(Dims d, Grid g, double2 *__restrict__ sf, double2 *__restrict__ sg,
       const double2 *__restrict__ nn, const double2 *__restrict__ nq, double cc, int want_p,
       int walls, int rows_first) {
  int bx, cy, unused;
  stencil_block(rows_first, bx, cy, unused);
  const int md = bx * blockDim.x + threadIdx.x;
  if (md >= d.nmodes) return;
  const size_t P = d.nmodes;
  const int n = d.nr;
  const int j0 = cy * R;
  const int nrow = n - j0 < R ? n - j0 : R;
  if (md == d.kmax) {
    for (int jj = 0; jj < nrow; ++jj) div_row(d, g, sf, sg, nn, nq, cc, want_p, walls, md, j0 + jj);
    return;
  }
  const int m = md / d.mz;
  const int kk = md - m * d.mz;
  const double kap = (double)(kk - d.kmax) * d.kz;
  const double2 *fz = sf + (size_t)2 * n * P + md;
  // D1 of F_+ and F_- (fields 0 and 1 of f)
  Cd dv[2][R], v[2][R];
  stencil_rows<R, 2>(g, PIPE ? g.d1 + odd_off(g, m + 1) : g.d1, n, j0, nrow, sf + md,
                     (size_t)n * P, P, dv, v);
#pragma unroll
  for (int jj = 0; jj < R; ++jj) {
    const int j = j0 + jj;
    if (jj >= nrow) break;
    if ((j == 0 && !PIPE) || j == n - 1) {
      div_row(d, g, sf, sg, nn, nq, cc, want_p, walls, md, j);
      continue;
    }
    const double ri = g.rinv[j];
    const Cd vz = ld(fz + (size_t)j * P);
    const Cd dp = dv[0][jj], dm = dv[1][jj], vp = v[0][jj], vm = v[1][jj];
    st(sg + (size_t)j * P + md,
       0.5 * ((dp + ((1.0 + m) * ri) * vp) + (dm + ((1.0 - m) * ri) * vm)) + kap * ci(vz));
  }
}

// lambda = -A^-1 beta(X0), beta = divergence at the two walls.
// One lane per mode, 64-lane workgroups (more of the chip for a small
// grid); the wall windows start at 0 and N-9, so all 38 loads of a lane are
// independent and issue together.
template <bool PIPE = false>
__global__ void __launch_bounds__(64) k_influence(Dims d, Grid g, Influence I,
                                                  const double2 *__restrict__ sx,
                                                  double2 *__restrict__ lam) {
  const int md = blockIdx.x * blockDim.x + threadIdx.x;
  if (md >= d.nmodes) return;
  const size_t P = d.nmodes;
  const int n = d.nr;
  const int kp1 = d.kmax + 1;
  const int m = md / d.mz;
  const int kk = md - m * d.mz;
  const int ka = kk >= d.kmax ? kk - d.kmax : d.kmax - kk;
  if (m == 0 && ka == 0) {
    st(lam + 2 * (size_t)md, Cd{0, 0});
    st(lam + 2 * (size_t)md + 1, Cd{0, 0});
    return;
  }
  const double kap = (double)(kk - d.kmax) * d.kz;
  const double mm = (double)m;
  const double2 *xp = sx + md, *xm = sx + (size_t)n * P + md, *xz = sx + (size_t)2 * n * P + md;
  Cd beta[2] = {Cd{0, 0}, Cd{0, 0}};
#pragma unroll
  for (int w = PIPE ? 1 : 0; w < 2; ++w) {  // (pipe: one wall, beta[0] = 0)
    const int j = w == 0 ? 0 : n - 1;
    const int s0 = w == 0 ? 0 : n - kStencil;  // one-sided wall window
    const double *wd = g.d1 + j * kStencil;
    if constexpr (PIPE) wd += odd_off(g, m + 1);
    const double ri = g.rinv[j];
    Cd dp = {0.0, 0.0}, dm = {0.0, 0.0};
#pragma unroll
    for (int t = 0; t < kStencil; ++t) {
      dp = fmac(wd[t], ld(xp + (size_t)(s0 + t) * P), dp);
      dm = fmac(wd[t], ld(xm + (size_t)(s0 + t) * P), dm);
    }
    beta[w] = 0.5 * ((dp + ((1.0 + mm) * ri) * ld(xp + (size_t)j * P)) +
                     (dm + ((1.0 - mm) * ri) * ld(xm + (size_t)j * P))) +
              kap * ci(ld(xz + (size_t)j * P));
  }
  const int op = m * kp1 + ka;
  const size_t ns = I.nops;
  const double a00 = I.ainv[op], a01 = I.ainv[ns + op], a10 = I.ainv[2 * ns + op], a11 = I.ainv[3 * ns + op];
  const Cd l1 = {-(a00 * beta[0].x + a01 * beta[1].x), -(a00 * beta[0].y + a01 * beta[1].y)};
  const Cd l2 = {-(a10 * beta[0].x + a11 * beta[1].x), -(a10 * beta[0].y + a11 * beta[1].y)};
  st(lam + 2 * (size_t)md, l1);
  st(lam + 2 * (size_t)md + 1, l2);
}

struct Vals {
  Cd ur, ut, uz, T, p;
};

// WITH_P: also the pressure (the step itself does not need it)
template <bool WITH_P = true>
__device__ __forceinline__ Vals final_value(const Dims &d, const Influence &I,
                                            const double2 *__restrict__ sx,
                                            const double2 *__restrict__ sp,
                                            const double2 *__restrict__ lam, int j, int md) {
  const size_t P = d.nmodes;
  const int n = d.nr;
  const int kp1 = d.kmax + 1;
  const int m = md / d.mz;
  const int kk = md - m * d.mz;
  const int ka = kk >= d.kmax ? kk - d.kmax : d.kmax - kk;
  Cd xp = ld(sx + (size_t)j * P + md);
  Cd xm = ld(sx + ((size_t)n + j) * P + md);
  Cd xz = ld(sx + ((size_t)2 * n + j) * P + md);
  Cd p = WITH_P ? ld(sp + (size_t)j * P + md) : Cd{0.0, 0.0};
  Vals v;
  if (!(m == 0 && ka == 0)) {
    const double kap = (double)(kk - d.kmax) * d.kz;
    const Cd l1 = ld(lam + 2 * (size_t)md), l2 = ld(lam + 2 * (size_t)md + 1);
    const size_t ns = I.nops;
    const int op = m * kp1 + ka;
    // the pair of responses of kind s (p, X+, X-, h) times lambda
    auto hom = [&](int s) {
      const double2 r = I.resp[((size_t)s * n + j) * ns + op];
      return r.x * l1 + r.y * l2;
    };
    if (WITH_P) p = p + hom(0);
    xp = xp + hom(1);
    xm = xm + hom(2);
    // X_z,j = -i kappa h_j
    const Cd hz = hom(3);
    xz = xz - kap * ci(hz);
  }
  v.ur = 0.5 * (xp + xm);
  const Cd dd = xp - xm;  // u_theta = (X+ - X-) / (2 i)
  v.ut = {0.5 * dd.y, -0.5 * dd.x};
  v.uz = xz;
  v.T = d.heated ? ld(sx + ((size_t)3 * n + j) * P + md) : Cd{0, 0};
  v.p = p;
  return v;
}

template <bool WITH_P>
__global__ void __launch_bounds__(256)
k_finalize(Dims d, Influence I, const double2 *__restrict__ sx, const double2 *__restrict__ sp,
           const double2 *__restrict__ lam, double2 *__restrict__ out,
           double2 *__restrict__ pout) {
  constexpr int NV = WITH_P ? 5 : 4;
  __shared__ Cd xch[NV][256];
  const int md = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y;
  const size_t P = d.nmodes;
  const int n = d.nr;
  Vals v{}, w{};
  if (d.mz <= (int)blockDim.x && blockIdx.x == 0) {
    // the whole m = 0 column lies in this workgroup: its lanes take their
    // mirror mode's values from the lane that computes them, instead of
    // computing them a second time
    if (md < d.nmodes) v = final_value<WITH_P>(d, I, sx, sp, lam, j, md);
    if (md < d.mz) {
      xch[0][md] = v.ur;
      xch[1][md] = v.ut;
      xch[2][md] = v.uz;
      xch[3][md] = v.T;
      if (WITH_P) xch[NV - 1][md] = v.p;
    }
    __syncthreads();
    if (md >= d.nmodes) return;
    if (md < d.mz) {
      const int mk = d.mz - 1 - md;
      w = Vals{xch[0][mk], xch[1][mk], xch[2][mk], xch[3][mk],
               WITH_P ? xch[NV - 1][mk] : Cd{0, 0}};
    }
  } else {
    if (md >= d.nmodes) return;
    v = final_value<WITH_P>(d, I, sx, sp, lam, j, md);
    if (md < d.mz) w = final_value<WITH_P>(d, I, sx, sp, lam, j, d.mz - 1 - md);
  }
  if (md < d.mz) {  // m = 0: Hermitian projection
    auto h = [](Cd a, Cd b) { return Cd{0.5 * (a.x + b.x), 0.5 * (a.y - b.y)}; };
    v.ur = h(v.ur, w.ur);
    v.ut = h(v.ut, w.ut);
    v.uz = h(v.uz, w.uz);
    v.T = h(v.T, w.T);
    v.p = h(v.p, w.p);
  }
  st(out + ((size_t)0 * n + j) * P + md, v.ur);
  st(out + ((size_t)1 * n + j) * P + md, v.ut);
  st(out + ((size_t)2 * n + j) * P + md, v.uz);
  if (d.heated) st(out + ((size_t)3 * n + j) * P + md, v.T);
  if (WITH_P) st(pout + (size_t)j * P + md, v.p);
}

// Perturbation energy partial sums: w_j r_j c_m |u - U_b|^2 per block.
__global__ void k_energy_part(Dims d, Grid g, const double2 *__restrict__ u, double *__restrict__ part) {
  __shared__ double red[16];
  const size_t P = d.nmodes;
  const size_t total = (size_t)d.nr * P;
  double acc = 0.0;
  for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (size_t)gridDim.x * blockDim.x) {
    const int j = (int)(idx / P);
    const int md = (int)(idx - (size_t)j * P);
    const int m = md / d.mz;
    double s = 0.0;
    for (int f = 0; f < 3; ++f) {
      double2 v = u[((size_t)f * d.nr + j) * P + md];
      if (f == 1 && md == d.kmax) v.x -= d.a_cou * g.r[j] + d.b_cou * g.rinv[j];
      s += v.x * v.x + v.y * v.y;
    }
    acc += (m == 0 ? 1.0 : 2.0) * g.ccw[j] * g.r[j] * s;
  }
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double r = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) r += red[w];
    part[blockIdx.x] = r;
  }
}

__global__ void k_energy_final(const double *__restrict__ part, int n, double scale, double *out) {
  __shared__ double red[16];
  double acc = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) acc += part[i];
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double r = 0.0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) r += red[w];
    out[0] = r * scale;
  }
}

// u~ = herm(amps) * g(r), g = 16 (r - r_i)^2 (r_o - r)^2.
__global__ void k_seed(Dims d, Grid g, const double2 *__restrict__ amps, double2 *__restrict__ out) {
  const int md = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y;
  const int f = blockIdx.z;
  if (md >= d.nmodes) return;
  const size_t P = d.nmodes;
  Cd a = ld(amps + (size_t)f * P + md);
  if (md < d.mz) {
    const Cd b = ld(amps + (size_t)f * P + (d.mz - 1 - md));
    a = {0.5 * (a.x + b.x), 0.5 * (a.y - b.y)};
  }
  if (md == d.kmax) a = {0, 0};
  const double r = g.r[j];
  if (d.pipe) {
    // u_+- = (a_r +- i a_theta) g_{m+-1}, u_z = a_z g_m, g_q = r^q (1 - r^2)^2
    // at peak one (regular at the axis); this lane writes component f
    const int m = md / d.mz;
    auto gq = [&](int q) {
      const double w = 1.0 - r * r;
      const double peak = q > 0 ? pow(q / (q + 4.0), 0.5 * q) * (16.0 / ((q + 4.0) * (q + 4.0))) : 1.0;
      return pow(r, (double)q) * w * w / peak;
    };
    Cd v;
    if (f == 2) {
      v = gq(m) * a;
    } else {
      // both in-plane amplitudes, the m = 0 column made Hermitian
      Cd ar = ld(amps + md), at = ld(amps + P + md);
      if (md < d.mz) {
        const int mm = d.mz - 1 - md;
        const Cd br = ld(amps + mm), bt = ld(amps + P + mm);
        ar = {0.5 * (ar.x + br.x), 0.5 * (ar.y - br.y)};
        at = {0.5 * (at.x + bt.x), 0.5 * (at.y - bt.y)};
      }
      if (md == d.kmax) ar = at = Cd{0, 0};
      const Cd up = gq(m + 1) * (ar + ci(at));
      const Cd um = gq(m >= 1 ? m - 1 : 1 - m) * (ar - ci(at));
      v = f == 0 ? 0.5 * (up + um) : Cd{0.5 * (up.y - um.y), -0.5 * (up.x - um.x)};
    }
    st(out + ((size_t)f * d.nr + j) * P + md, v);
    return;
  }
  const double s = 16.0 * (r - d.r_i) * (r - d.r_i) * (d.r_o - r) * (d.r_o - r);
  st(out + ((size_t)f * d.nr + j) * P + md, s * a);
}

// out += basic state; T: out_T = T_c delta_00 + u~_T (unprojected).
__global__ void k_add_base(Dims d, Grid g, const double2 *__restrict__ pert, double2 *__restrict__ out) {
  const int md = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y;
  if (md >= d.nmodes) return;
  const size_t P = d.nmodes;
  const double r = g.r[j];
  if (md == d.kmax && d.pipe) {  // Hagen--Poiseuille flow Re (1 - r^2), Re = gp / 4
    double2 *p = out + ((size_t)2 * d.nr + j) * P + md;
    p->x += 0.25 * d.gp * (1.0 - r * r);
  } else if (md == d.kmax) {
    double2 *p = out + ((size_t)1 * d.nr + j) * P + md;
    p->x += d.a_cou * r + d.b_cou * g.rinv[j];
  }
  if (d.heated) {
    Cd t = ld(pert + ((size_t)3 * d.nr + j) * P + md);
    if (md == d.kmax) t.x += 0.5 + log(r / d.r_i) / log(d.r_i / d.r_o);
    st(out + ((size_t)3 * d.nr + j) * P + md, t);
  }
}

// ---------------------------------------------------------------------------
// Vector--Jacobian product of the implicit stage (discrete adjoint).  The
// stage is affine in (X^n, N^n, N^q); its linear part per mode is, in order,
//   f = X^n/dt + (1-c) L X^n + c N^q + (1-c) N^n   (+- basis)
//   g = mask(div f), p0 = P^-1 g, X0 = H^-1 mask(f - grad p0),
//   lambda = -A^-1 beta(X0), X = X0 + sum lambda_j X_j, herm(output).
// The adjoint applies the transposes in reverse order; complex-linear maps
// are conjugate-transposed (real factors transpose, i -> -i).
// ---------------------------------------------------------------------------

// A^T x = b with A = L U in envelope storage: U^T y = b (forward), then
// L^T x = y (backward).  Rows 0..8 of the forward pass and N-9..N-1 of the
// backward pass carry the one-sided edge entries and are peeled.
template <typename V, typename RHS, typename COL>
__device__ __forceinline__ void lu_solve_t(const Factors &F, int op, int n, RHS rhs, COL col) {
  const size_t nops = F.nops;
  const RowsOf R(F, op);
  const double *__restrict__ edge = F.edge + op;
  auto Lv = [&](int row, int c) { return R.pk[(size_t)row * 8 * nops + c]; };
  auto Uv = [&](int row, int c) { return R.pk[((size_t)row * 2 + 1) * 4 * nops + c]; };
  for (int j = 0; j < 9; ++j) {
    V y = rhs(j);
    for (int t = 1; t <= 4; ++t)
      if (j - t >= 0) y = y - Uv(j - t, t - 1) * col(j - t);
    for (int c = 0; c <= 3; ++c)
      if (j - c >= 5) y = y - edge[(size_t)(edge_off(c) + j - c - 5) * nops] * col(c);
    col(j) = R.dinv(j) * y;
  }
  // the last four U rows (then L rows) stay in registers
  RowU r1 = R.u(8), r2 = R.u(7), r3 = R.u(6), r4 = R.u(5);
  V y1 = col(8), y2 = col(7), y3 = col(6), y4 = col(5);
#pragma unroll 4
  for (int j = 9; j < n; ++j) {
    const RowU r0 = R.u(j);
    V y = rhs(j);
    y = y - r1.u1 * y1;
    y = y - r2.u2 * y2;
    y = y - r3.u3 * y3;
    y = y - r4.u4 * y4;
    y = R.dinv(j) * y;
    r4 = r3;
    r3 = r2;
    r2 = r1;
    r1 = r0;
    y4 = y3;
    y3 = y2;
    y2 = y1;
    y1 = y;
    col(j) = y;
  }
  for (int j = n - 1; j >= n - 9; --j) {
    V x = col(j);
    for (int t = 1; t <= 4; ++t)
      if (j + t < n) x = x - Lv(j + t, 4 - t) * col(j + t);
    for (int c = n - 4; c <= n - 1; ++c)
      if (c - j >= 5) x = x - edge[(size_t)(10 + edge_off(n - 1 - c) + j - (n - 9)) * nops] * col(c);
    col(j) = x;
  }
  RowL q1 = R.l(n - 9), q2 = R.l(n - 8), q3 = R.l(n - 7), q4 = R.l(n - 6);
  V x1 = col(n - 9), x2 = col(n - 8), x3 = col(n - 7), x4 = col(n - 6);
#pragma unroll 4
  for (int j = n - 10; j >= 0; --j) {
    const RowL q0 = R.l(j);
    V x = col(j);
    x = x - q1.l1 * x1;
    x = x - q2.l2 * x2;
    x = x - q3.l3 * x3;
    x = x - q4.l4 * x4;
    q4 = q3;
    q3 = q2;
    q2 = q1;
    q1 = q0;
    x4 = x3;
    x3 = x2;
    x2 = x1;
    x1 = x;
    col(j) = x;
  }
}

// (W^T v)_j = sum_i W[i][j - s_i] v_i over the rows i whose window holds j.
__device__ __forceinline__ Cd wt_rowc(const Grid &g, const double *w, int n, int j,
                                      const double2 *v, size_t stride, bool scale_rinv) {
  Cd acc = {0, 0};
  const int lo = j - 8 < 0 ? 0 : j - 8;
  const int hi = j + 8 > n - 1 ? n - 1 : j + 8;
  for (int i = lo; i <= hi; ++i) {
    const int s = g.s[i];
    const int t = j - s;
    if (t >= 0 && t < kStencil) {
      double c = w[i * kStencil + t];
      if (scale_rinv) c *= g.rinv[i];
      acc = fmac(c, ld(v + (size_t)i * stride), acc);
    }
  }
  return acc;
}

// Output adjoint: Hermitian projection of u_bar, then the +- basis:
// Xbar+- = (ubar_r +- i ubar_theta)/2, Xbar_z = ubar_z, Tbar.  Mode (0,0)
// keeps ubar_theta in slot 0 (its u_theta is solved directly).
__global__ void k_adj_out(Dims d, const double2 *__restrict__ ub, double2 *__restrict__ sx) {
  const int md = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y;
  if (md >= d.nmodes) return;
  const size_t P = d.nmodes;
  const int n = d.nr;
  auto U = [&](int f, int m2) { return ld(ub + ((size_t)f * n + j) * P + m2); };
  Cd v[4];
#pragma unroll
  for (int f = 0; f < 4; ++f) {  // (constant trip count: v stays in registers)
    if (f >= d.f) {
      v[f] = Cd{0, 0};
      continue;
    }
    v[f] = U(f, md);
    if (md < d.mz) {
      const Cd w = U(f, d.mz - 1 - md);
      v[f] = {0.5 * (v[f].x + w.x), 0.5 * (v[f].y - w.y)};
    }
  }
  if (md == d.kmax) {
    st(sx + ((size_t)0 * n + j) * P + md, v[1]);
    st(sx + ((size_t)1 * n + j) * P + md, Cd{0, 0});
  } else {
    st(sx + ((size_t)0 * n + j) * P + md, 0.5 * (v[0] + ci(v[1])));
    st(sx + ((size_t)1 * n + j) * P + md, 0.5 * (v[0] - ci(v[1])));
  }
  st(sx + ((size_t)2 * n + j) * P + md, v[2]);
  if (d.heated) st(sx + ((size_t)3 * n + j) * P + md, v[3]);
}

// lambda_bar_j = sum_r (X_j+ Xbar+ + X_j- Xbar- + i kappa h_j Xbar_z);
// beta_bar = -A^-T lambda_bar.  Workgroup of 64 modes x 16 row parts (a few
// rows per lane, so each lane's loads go out in one round); the parts'
// partial sums meet in LDS (fixed order).
constexpr int kLamModes = 64, kLamParts = 16;

__global__ void __launch_bounds__(kLamModes * kLamParts)
k_adj_lambda(Dims d, Influence I, const double2 *__restrict__ sx, double2 *__restrict__ bbar) {
  __shared__ Cd part[kLamParts - 1][2][kLamModes];
  const int lane = threadIdx.x % kLamModes, q = threadIdx.x / kLamModes;
  const int md = blockIdx.x * kLamModes + lane;
  const bool live = md < d.nmodes;
  const size_t P = d.nmodes;
  const int n = d.nr;
  const int kp1 = d.kmax + 1;
  const int m = live ? md / d.mz : 0;
  const int kk = live ? md - m * d.mz : d.kmax;
  const int ka = kk >= d.kmax ? kk - d.kmax : d.kmax - kk;
  const double kap = (double)(kk - d.kmax) * d.kz;
  const int op = m * kp1 + ka;
  const size_t ns = I.nops;
  Cd l1 = {0, 0}, l2 = {0, 0};
  const int j0 = (n * q) / kLamParts, j1 = (n * (q + 1)) / kLamParts;
  if (live) {
#pragma unroll 4
    for (int j = j0; j < j1; ++j) {
      const Cd xp = ld(sx + (size_t)j * P + md);
      const Cd xm = ld(sx + ((size_t)n + j) * P + md);
      const Cd xz = kap * ci(ld(sx + ((size_t)2 * n + j) * P + md));  // i kappa Xbar_z
      auto Rv = [&](int s) { return I.resp[((size_t)s * n + j) * ns + op]; };
      const double2 r1 = Rv(1), r2 = Rv(2), r3 = Rv(3);
      l1 = l1 + (r1.x * xp + r2.x * xm + r3.x * xz);
      l2 = l2 + (r1.y * xp + r2.y * xm + r3.y * xz);
    }
  }
  if (q > 0) {
    part[q - 1][0][lane] = l1;
    part[q - 1][1][lane] = l2;
  }
  __syncthreads();
  if (q != 0 || !live) return;
#pragma unroll
  for (int t = 0; t < kLamParts - 1; ++t) {
    l1 = l1 + part[t][0][lane];
    l2 = l2 + part[t][1][lane];
  }
  if (m == 0 && ka == 0) {
    st(bbar + 2 * (size_t)md, Cd{0, 0});
    st(bbar + 2 * (size_t)md + 1, Cd{0, 0});
    return;
  }
  const double a00 = I.ainv[op], a01 = I.ainv[ns + op], a10 = I.ainv[2 * ns + op], a11 = I.ainv[3 * ns + op];
  st(bbar + 2 * (size_t)md, Cd{-(a00 * l1.x + a10 * l2.x), -(a00 * l1.y + a10 * l2.y)});
  st(bbar + 2 * (size_t)md + 1, Cd{-(a01 * l1.x + a11 * l2.x), -(a01 * l1.y + a11 * l2.y)});
}

// Transposed Helmholtz sweeps: comp 0/1/2 velocity (+, -, z), 3 temperature.
// rbar = mask(H^-T (Xbar + beta terms)) -> sf[comp]; mode (0,0) is the
// direct u_theta / u_z problem.
__global__ void __launch_bounds__(256)
k_adj_vel(Dims d, Grid g, Factors fv, Factors ft, const double2 *__restrict__ sx,
          const double2 *__restrict__ bbar, double2 *__restrict__ sf) {
  const int md = blockIdx.x * blockDim.x + threadIdx.x;
  if (md >= d.nmodes) return;
  const int comp = blockIdx.y;
  const size_t P = d.nmodes;
  const int n = d.nr;
  const int kp1 = d.kmax + 1;
  const int m = md / d.mz;
  const int kk = md - m * d.mz;
  const int ka = kk >= d.kmax ? kk - d.kmax : d.kmax - kk;
  const double kap = (double)(kk - d.kmax) * d.kz;
  const bool zero = (m == 0 && ka == 0);
  const double2 *xb = sx + (size_t)comp * n * P + md;
  double2 *out = sf + (size_t)comp * n * P + md;
  auto outr = [&](int j) -> Cd & { return *reinterpret_cast<Cd *>(out + (size_t)j * P); };
  if (comp == 3) {
    lu_solve_t<Cd>(ft, m * kp1 + ka, n, [&](int j) { return ld(xb + (size_t)j * P); }, outr);
    outr(0) = Cd{0, 0};
    outr(n - 1) = Cd{0, 0};
    return;
  }
  if (zero) {
    if (comp == 1) return;
    const int q = comp == 0 ? 1 : 0;
    lu_solve_t<Cd>(fv, q * kp1 + ka, n, [&](int j) { return ld(xb + (size_t)j * P); }, outr);
    outr(0) = Cd{0, 0};
    outr(n - 1) = Cd{0, 0};
    if (comp == 0) {  // fbar+ = (i/2) rbar_theta, fbar- = -(i/2) rbar_theta
      double2 *om = sf + (size_t)n * P + md;
      for (int j = 0; j < n; ++j) {
        const Cd r = outr(j);
        const Cd h = 0.5 * ci(r);
        outr(j) = h;
        st(om + (size_t)j * P, Cd{-h.x, -h.y});
      }
    }
    return;
  }
  const int q = comp == 0 ? m + 1 : (comp == 1 ? (m >= 1 ? m - 1 : 1 - m) : m);
  const Cd b0 = ld(bbar + 2 * (size_t)md), b1 = ld(bbar + 2 * (size_t)md + 1);
  const double sgn = comp == 0 ? 1.0 : -1.0;
  auto rhs = [&](int j) -> Cd {
    Cd v = ld(xb + (size_t)j * P);
    if (comp < 2) {
      // 1/2 (D1 + (1 +- m)/r)^T e_w beta_bar_w
      if (j <= 8) {
        double c = g.d1[0 * kStencil + j];
        if (j == 0) c += (1.0 + sgn * m) * g.rinv[0];
        v = v + (0.5 * c) * b0;
      }
      if (j >= n - 9) {
        double c = g.d1[(n - 1) * kStencil + (j - g.s[n - 1])];
        if (j == n - 1) c += (1.0 + sgn * m) * g.rinv[n - 1];
        v = v + (0.5 * c) * b1;
      }
    } else {
      if (j == 0) v = v - kap * ci(b0);
      if (j == n - 1) v = v - kap * ci(b1);
    }
    return v;
  };
  lu_solve_t<Cd>(fv, q * kp1 + ka, n, rhs, outr);
  outr(0) = Cd{0, 0};
  outr(n - 1) = Cd{0, 0};
}

// pbar0 = -D1^T (rbar+ + rbar-) + (m/r)(rbar+ - rbar-) + i kappa rbar_z.
__global__ void k_adj_pbar(Dims d, Grid g, const double2 *__restrict__ sf, double2 *__restrict__ pb) {
  const int md = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y;
  if (md >= d.nmodes) return;
  const size_t P = d.nmodes;
  const int n = d.nr;
  const int m = md / d.mz;
  const int kk = md - m * d.mz;
  if (md == d.kmax) {
    st(pb + (size_t)j * P + md, Cd{0, 0});
    return;
  }
  const double kap = (double)(kk - d.kmax) * d.kz;
  const double2 *rp = sf + md, *rm = sf + (size_t)n * P + md, *rz = sf + (size_t)2 * n * P + md;
  const Cd dp = wt_rowc(g, g.d1, n, j, rp, P, false);
  const Cd dm = wt_rowc(g, g.d1, n, j, rm, P, false);
  const Cd vp = ld(rp + (size_t)j * P), vm = ld(rm + (size_t)j * P), vz = ld(rz + (size_t)j * P);
  const Cd res = ((m * g.rinv[j]) * (vp - vm)) - (dp + dm) + kap * ci(vz);
  st(pb + (size_t)j * P + md, res);
}

// gbar = mask(P^-T pbar0).
__global__ void __launch_bounds__(256)
k_adj_poisson(Dims d, Factors fp, const double2 *__restrict__ pb, double2 *__restrict__ gb) {
  const int md = blockIdx.x * blockDim.x + threadIdx.x;
  if (md >= d.nmodes) return;
  const size_t P = d.nmodes;
  const int n = d.nr;
  const int kp1 = d.kmax + 1;
  const int m = md / d.mz;
  const int kk = md - m * d.mz;
  const int ka = kk >= d.kmax ? kk - d.kmax : d.kmax - kk;
  auto outr = [&](int j) -> Cd & { return *reinterpret_cast<Cd *>(gb + (size_t)j * P + md); };
  if (m == 0 && ka == 0) {
    for (int j = 0; j < n; ++j) outr(j) = Cd{0, 0};
    return;
  }
  lu_solve_t<Cd>(fp, m * kp1 + ka, n, [&](int j) { return ld(pb + (size_t)j * P + md); }, outr);
  outr(0) = Cd{0, 0};
  outr(n - 1) = Cd{0, 0};
}

// fbar+- = rbar+- + 1/2 (D1^T gbar + (1 +- m) gbar / r), fbar_z = rbar_z - i kappa gbar.
__global__ void k_adj_f(Dims d, Grid g, const double2 *__restrict__ sf, const double2 *__restrict__ gb,
                        double2 *__restrict__ fb) {
  const int md = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y;
  if (md >= d.nmodes) return;
  const size_t P = d.nmodes;
  const int n = d.nr;
  const int m = md / d.mz;
  const int kk = md - m * d.mz;
  const double kap = (double)(kk - d.kmax) * d.kz;
  Cd fp = ld(sf + (size_t)j * P + md), fm = ld(sf + ((size_t)n + j) * P + md);
  Cd fz = ld(sf + ((size_t)2 * n + j) * P + md);
  if (md != d.kmax) {
    const Cd dg = wt_rowc(g, g.d1, n, j, gb + md, P, false);
    const Cd gv = ld(gb + (size_t)j * P + md);
    const double ri = g.rinv[j];
    fp = fp + 0.5 * (dg + ((1.0 + m) * ri) * gv);
    fm = fm + 0.5 * (dg + ((1.0 - m) * ri) * gv);
    fz = fz - kap * ci(gv);
  }
  st(fb + (size_t)j * P + md, fp);
  st(fb + ((size_t)n + j) * P + md, fm);
  st(fb + ((size_t)2 * n + j) * P + md, fz);
  if (d.heated) st(fb + ((size_t)3 * n + j) * P + md, ld(sf + ((size_t)3 * n + j) * P + md));
}

// Input adjoints: Xbar^n = fbar/dt + (1-c) L^T fbar; Nbar^q = c fbar,
// Nbar^n = (1-c) fbar; back to (r, theta, z, T) and accumulated.
__global__ void __launch_bounds__(256)
k_adj_in(Dims d, Grid g, const int *__restrict__ trow, const int *__restrict__ tcnt,
         const double *__restrict__ twt, const double2 *__restrict__ fb, double idt, double cc,
         double2 *__restrict__ ubn, double2 *__restrict__ nbn, double2 *__restrict__ nbq,
         int overwrite) {
  const int md = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y;
  if (md >= d.nmodes) return;
  const size_t P = d.nmodes;
  const int n = d.nr;
  const int m = md / d.mz;
  const int kk = md - m * d.mz;
  const double kap = (double)(kk - d.kmax) * d.kz;
  const double ri = g.rinv[j], r2 = ri * ri, k2 = kap * kap;
  const double ce = 1.0 - cc;
  Cd xb[4], fv[4];
  const int nf = d.heated ? 4 : 3;
#pragma unroll
  for (int c = 0; c < 4; ++c) {  // (constant trip count: xb, fv stay in registers)
    if (c >= nf) {
      xb[c] = fv[c] = Cd{0, 0};
      continue;
    }
    const double2 *f = fb + (size_t)c * n * P + md;
    const double q = c == 0 ? (double)(m + 1) : (c == 1 ? (double)(m >= 1 ? m - 1 : 1 - m) : (double)m);
    const Cd v = ld(f + (size_t)j * P);
    // (D2 + D1/r)^T f at row j from the column's table (uniform per workgroup)
    Cd lt = {0, 0};
    const int cnt = tcnt[j];
    for (int e = 0; e < cnt; ++e)
      lt = fmac(twt[j * kTrans + e], ld(f + (size_t)trow[j * kTrans + e] * P), lt);
    const Cd LT = lt - (q * q * r2 + k2) * v;
    const double sc = c == 3 ? ce / d.pr : ce;
    xb[c] = idt * v + sc * LT;
    fv[c] = v;
  }
  auto acc = [&](double2 *base, int f, Cd v, int bit) {
    double2 *p = base + ((size_t)f * n + j) * P + md;
    if (overwrite & bit) {
      *p = make_double2(v.x, v.y);
    } else {
      p->x += v.x;
      p->y += v.y;
    }
  };
  // X+- = X_r +- i X_theta  =>  Xbar_r = Xbar+ + Xbar-, Xbar_theta = -i (Xbar+ - Xbar-)
  const Cd ur = xb[0] + xb[1];
  const Cd dd = xb[0] - xb[1];
  const Cd ut = {dd.y, -dd.x};
  acc(ubn, 0, ur, 1);
  acc(ubn, 1, ut, 1);
  acc(ubn, 2, xb[2], 1);
  if (d.heated) acc(ubn, 3, xb[3], 1);
  const Cd fr = fv[0] + fv[1];
  const Cd fdd = fv[0] - fv[1];
  const Cd ft = {fdd.y, -fdd.x};
  acc(nbq, 0, cc * fr, 4);
  acc(nbq, 1, cc * ft, 4);
  acc(nbq, 2, cc * fv[2], 4);
  acc(nbn, 0, ce * fr, 2);
  acc(nbn, 1, ce * ft, 2);
  acc(nbn, 2, ce * fv[2], 2);
  if (d.heated) {
    acc(nbq, 3, cc * fv[3], 4);
    acc(nbn, 3, ce * fv[3], 2);
  }
}

// dE/du = 2 pi L_z w_j r_j c_m (u - U_b) for the velocity, 0 for T.
__global__ void k_energy_grad(Dims d, Grid g, const double2 *__restrict__ u, double2 *__restrict__ gout) {
  const int md = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y;
  if (md >= d.nmodes) return;
  const size_t P = d.nmodes;
  const int m = md / d.mz;
  const double s = 2.0 * M_PI * d.lz * g.ccw[j] * g.r[j] * (m == 0 ? 1.0 : 2.0);
  for (int f = 0; f < d.f; ++f) {
    double2 v = u[((size_t)f * d.nr + j) * P + md];
    if (f == 1 && md == d.kmax) v.x -= d.a_cou * g.r[j] + d.b_cou * g.rinv[j];
    if (f == 3) v = make_double2(0.0, 0.0);
    gout[((size_t)f * d.nr + j) * P + md] = make_double2(s * v.x, s * v.y);
  }
}

// Rows per lane of a stencil kernel with `parts` workgroups per (mode tile,
// row chunk): the longest chunk, up to four rows, that still leaves
// `min_waves` wavefronts per SIMD.  Longer chunks save reads of the shared
// window rows but cost occupancy.  Measured on 64 rows x 8128 modes and 128 x
// 130816: the kernels with two stencil fields per lane (divergence, the +-
// right sides) are fastest down to four wavefronts per SIMD (two and four
// rows on the first grid, four on the second); the velocity right sides, one
// stencil field beside six streamed ones, need eight (one row on the first
// grid, four on the second).
inline int chunk_rows(const nsc_ctx *c, int parts, int min_waves) {
  const long waves_row = (long)(c->d.nmodes + 255) / 256 * 4 * parts;
  const long simds = 4L * c->cu_count;
  for (int R = 4; R > 1; R /= 2)
    if (waves_row * ((c->d.nr + R - 1) / R) >= (long)min_waves * simds) return R;
  return 1;
}

inline dim3 mode_grid(const nsc_ctx *c, int y, int z = 1) {
  return dim3((c->d.nmodes + 255) / 256, y, z);
}

}  // namespace

hipError_t launch_factor(const nsc_ctx *c, Factors *f, int kind, double alpha, double beta) {
  hipLaunchKernelGGL(k_factor, dim3((f->nops + kFacThreads - 1) / kFacThreads), dim3(kFacThreads), 0,
                     c->stream, c->d, c->g, *f, *f, kind, alpha, beta, beta);
  return hipGetLastError();
}

hipError_t launch_factor2(const nsc_ctx *c, Factors *f0, Factors *f1, int kind, double alpha,
                          double beta0, double beta1) {
  const int nmax = f0->nops > f1->nops ? f0->nops : f1->nops;
  hipLaunchKernelGGL(k_factor, dim3((nmax + kFacThreads - 1) / kFacThreads, 2),
                     dim3(kFacThreads), 0, c->stream, c->d, c->g, *f0, *f1, kind, alpha, beta0,
                     beta1);
  return hipGetLastError();
}

hipError_t launch_influence_pressure(const nsc_ctx *c) {
  hipLaunchKernelGGL(k_influence_p, dim3((c->inf.nops + 63) / 64), dim3(64), 0, c->stream, c->d,
                     c->fp, c->inf);
  return hipGetLastError();
}

hipError_t launch_influence_setup(const nsc_ctx *c) {
  const size_t shm = (size_t)4 * c->d.nr * kInfOps * sizeof(Cd);
  if (shm <= (size_t)c->lds_max) {
    hipLaunchKernelGGL(k_influence_v, dim3((c->inf.nops + kInfOps - 1) / kInfOps), dim3(kInfThreads), shm,
                       c->stream, c->d, c->g, c->fv, c->inf);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_influence_x, dim3((c->inf.nops + 63) / 64, 3), dim3(64), 0, c->stream, c->d, c->g,
                     c->fv, c->inf);
  hipLaunchKernelGGL(k_influence_a, dim3((c->inf.nops + 63) / 64), dim3(64), 0, c->stream, c->d,
                     c->g, c->inf);
  return hipGetLastError();
}

hipError_t launch_rhs(const nsc_ctx *c, const double *u, const double *nn, const double *nq,
                      double dt, double cc) {
  const int parts = c->d.heated ? 3 : 2;
  auto rhs = [&](auto rows) {
    constexpr int R = decltype(rows)::value;
    auto kern = c->d.pipe ? k_rhs<R, true> : k_rhs<R, false>;
    hipLaunchKernelGGL(kern, mode_grid(c, (c->d.nr + R - 1) / R, parts), dim3(256), 0,
                       c->stream, c->d, c->g, reinterpret_cast<const double2 *>(u),
                       reinterpret_cast<const double2 *>(nn), reinterpret_cast<const double2 *>(nq),
                       reinterpret_cast<double2 *>(c->s_f), 1.0 / dt, cc, c->rows_first);
  };
  switch (chunk_rows(c, parts, 4)) {
    case 4: rhs(std::integral_constant<int, 4>{}); break;
    case 2: rhs(std::integral_constant<int, 2>{}); break;
    default: rhs(std::integral_constant<int, 1>{}); break;
  }
  return hipGetLastError();
}

hipError_t launch_influence(const nsc_ctx *c) {
  auto kern = c->d.pipe ? k_influence<true> : k_influence<false>;
  hipLaunchKernelGGL(kern, dim3((c->d.nmodes + 63) / 64), dim3(64), 0, c->stream, c->d, c->g, c->inf,
                     reinterpret_cast<const double2 *>(c->s_x), reinterpret_cast<double2 *>(c->s_lam));
  return hipGetLastError();
}

hipError_t launch_finalize(const nsc_ctx *c, double *out, double *p_out) {
  auto fin = p_out ? k_finalize<true> : k_finalize<false>;
  hipLaunchKernelGGL(fin, mode_grid(c, c->d.nr), dim3(256), 0, c->stream, c->d, c->inf,
                     reinterpret_cast<const double2 *>(c->s_x), reinterpret_cast<const double2 *>(c->s_p),
                     reinterpret_cast<const double2 *>(c->s_lam), reinterpret_cast<double2 *>(out),
                     reinterpret_cast<double2 *>(p_out));
  return hipGetLastError();
}

hipError_t launch_energy(const nsc_ctx *c, const double *u, double *e_dev) {
  hipLaunchKernelGGL(k_energy_part, dim3(c->e_nblk), dim3(256), 0, c->stream, c->d, c->g,
                     reinterpret_cast<const double2 *>(u), c->e_part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_energy_final, dim3(1), dim3(256), 0, c->stream, c->e_part, c->e_nblk,
                     M_PI * c->d.lz, e_dev);
  return hipGetLastError();
}

hipError_t launch_seed(const nsc_ctx *c, const double *amps, double *out_pert) {
  hipLaunchKernelGGL(k_seed, mode_grid(c, c->d.nr, c->d.f), dim3(256), 0, c->stream, c->d, c->g,
                     reinterpret_cast<const double2 *>(amps), reinterpret_cast<double2 *>(out_pert));
  return hipGetLastError();
}

hipError_t launch_add_base(const nsc_ctx *c, const double *pert_tilde, double *out) {
  hipLaunchKernelGGL(k_add_base, mode_grid(c, c->d.nr), dim3(256), 0, c->stream, c->d, c->g,
                     reinterpret_cast<const double2 *>(pert_tilde), reinterpret_cast<double2 *>(out));
  return hipGetLastError();
}

hipError_t launch_solve_vjp(const nsc_ctx *c, const double *ubar_out, double *ubar_n,
                            double *nbar_n, double *nbar_q, double dt, double cc,
                            int overwrite, double *scratch) {
  if (c->fused_adj)
    return launch_stage_adj(c, ubar_out, ubar_n, nbar_n, nbar_q, dt, cc, overwrite);
  const double2 *ub = reinterpret_cast<const double2 *>(ubar_out);
  double2 *sx = reinterpret_cast<double2 *>(c->s_x);
  double2 *sf = reinterpret_cast<double2 *>(c->s_f);
  double2 *sg = reinterpret_cast<double2 *>(c->s_g);
  double2 *sp = reinterpret_cast<double2 *>(c->s_p);
  double2 *lam = reinterpret_cast<double2 *>(c->s_lam);
  double *nq = nbar_q ? nbar_q : scratch;
  if (!nbar_q) overwrite |= 4;
  hipLaunchKernelGGL(k_adj_out, mode_grid(c, c->d.nr), dim3(256), 0, c->stream, c->d, ub, sx);
  hipLaunchKernelGGL(k_adj_lambda, dim3((c->d.nmodes + kLamModes - 1) / kLamModes), dim3(kLamModes * kLamParts),
                     0, c->stream, c->d, c->inf, sx, lam);
  hipLaunchKernelGGL(k_adj_vel, mode_grid(c, c->d.heated ? 4 : 3), dim3(256), 0, c->stream, c->d,
                     c->g, c->fv, c->ft, sx, lam, sf);
  hipLaunchKernelGGL(k_adj_pbar, mode_grid(c, c->d.nr), dim3(256), 0, c->stream, c->d, c->g, sf, sp);
  hipLaunchKernelGGL(k_adj_poisson, mode_grid(c, 1), dim3(256), 0, c->stream, c->d, c->fp, sp, sg);
  hipLaunchKernelGGL(k_adj_f, mode_grid(c, c->d.nr), dim3(256), 0, c->stream, c->d, c->g, sf, sg, sx);
  hipLaunchKernelGGL(k_adj_in, mode_grid(c, c->d.nr), dim3(256), 0, c->stream, c->d, c->g,
                     c->t_row, c->t_cnt, c->t_wt, sx, 1.0 / dt, cc,
                     reinterpret_cast<double2 *>(ubar_n), reinterpret_cast<double2 *>(nbar_n),
                     reinterpret_cast<double2 *>(nq), overwrite);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || nbar_q) return e;
  return launch_add(c, nbar_n, nq, (size_t)c->d.f * c->d.nr * c->d.nmodes * 2);
}

__global__ void k_add(double *__restrict__ y, const double *__restrict__ x, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    y[i] += x[i];
}

// y += x over n doubles
hipError_t launch_add(const nsc_ctx *c, double *y, const double *x, size_t n) {
  const size_t blocks = (n + 255) / 256 < 65536 ? (n + 255) / 256 : 65536;
  hipLaunchKernelGGL(k_add, dim3((unsigned)blocks), dim3(256), 0, c->stream, y, x, n);
  return hipGetLastError();
}

hipError_t launch_energy_grad(const nsc_ctx *c, const double *u, double *gout) {
  hipLaunchKernelGGL(k_energy_grad, mode_grid(c, c->d.nr), dim3(256), 0, c->stream, c->d, c->g,
                     reinterpret_cast<const double2 *>(u), reinterpret_cast<double2 *>(gout));
  return hipGetLastError();
}

// stage 0: Poisson right side (+ temperature wall rows); 1: pressure and
// temperature sweeps; 2: velocity right sides; 3: velocity sweeps.
hipError_t launch_solve_sweeps(const nsc_ctx *c, int stage, const double *nn, const double *nq,
                               double cc, int walls, int want_p) {
  const Dims &d = c->d;
  double2 *sf = reinterpret_cast<double2 *>(c->s_f);
  double2 *sg = reinterpret_cast<double2 *>(c->s_g);
  double2 *sp = reinterpret_cast<double2 *>(c->s_p);
  double2 *sx = reinterpret_cast<double2 *>(c->s_x);
  const int wp = (want_p && nn) ? 1 : 0;
  auto launch = [&](const SweepArgs &a, int nsys, auto family) {
    dim3 gr((d.nmodes + kSweepLanes - 1) / kSweepLanes, nsys);
    hipLaunchKernelGGL((k_sweep<decltype(family)::value>), gr, dim3(kSweepLanes), 0, c->stream, d, a);
  };
  const size_t fld = (size_t)d.nr * d.nmodes;
  if (stage == 0) {
    auto div = [&](auto rows) {
      constexpr int R = decltype(rows)::value;
      auto kern = d.pipe ? k_div2<R, true> : k_div2<R, false>;
      hipLaunchKernelGGL(kern, mode_grid(c, (d.nr + R - 1) / R), dim3(256), 0, c->stream,
                         d, c->g, sf, sg, reinterpret_cast<const double2 *>(nn),
                         reinterpret_cast<const double2 *>(nq), cc, wp, walls, c->rows_first);
    };
    switch (chunk_rows(c, 1, 4)) {
      case 4: div(std::integral_constant<int, 4>{}); break;
      case 2: div(std::integral_constant<int, 2>{}); break;
      default: div(std::integral_constant<int, 1>{}); break;
    }
  } else if (stage == 1) {
    // pressure (s_g -> s_p) and temperature (s_f[3] -> s_x[3]) in one launch
    SweepArgs a{};
    a.s[0] = SweepSys{c->fp, 0, wp ? 0 : 1, sg, sp};
    if (d.heated) a.s[1] = SweepSys{c->ft, 0, 0, sf + 3 * fld, sx + 3 * fld};
    launch(a, d.heated ? 2 : 1, std::integral_constant<int, 0>{});
  } else if (stage == 2) {
    auto vel = [&](auto rows) {
      constexpr int R = decltype(rows)::value;
      auto kern = d.pipe ? k_vel_rhs<R, true> : k_vel_rhs<R, false>;
      hipLaunchKernelGGL(kern, mode_grid(c, (d.nr + R - 1) / R), dim3(256), 0,
                         c->stream, d, c->g, sf, sp, walls, c->rows_first);
    };
    switch (chunk_rows(c, 1, 8)) {
      case 4: vel(std::integral_constant<int, 4>{}); break;
      case 2: vel(std::integral_constant<int, 2>{}); break;
      default: vel(std::integral_constant<int, 1>{}); break;
    }
  } else {
    SweepArgs av{};
    av.s[0] = SweepSys{c->fv, 1, 0, sf, sx};
    av.s[1] = SweepSys{c->fv, 2, 0, sf + fld, sx + fld};
    av.s[2] = SweepSys{c->fv, 0, 0, sf + 2 * fld, sx + 2 * fld};
    launch(av, 3, std::integral_constant<int, 1>{});
  }
  return hipGetLastError();
}

}  // namespace nsc
