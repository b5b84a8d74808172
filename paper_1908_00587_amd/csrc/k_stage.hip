// The implicit stage of a predictor or corrector in one kernel (section 2.2
// of the nsCouette paper: the linear terms are independent per Fourier mode).
// All FP64; the same formulas as the kernel sequence of k_solve.hip, which
// serves the grids past kStageRows radial points.
//
// A workgroup owns the radial columns of 2 OPS modes: (m, +-k) for OPS
// consecutive |k|, which share their operators, so each factor row is read
// once for four real columns.  Everything between the reading of u^n, N^n,
// N^q and the writing of the new state stays on chip:
//   right sides f -> divergence -> pressure (and temperature) sweeps ->
//   velocity right sides -> velocity sweeps -> influence coefficients ->
//   superposition, +- -> (r, theta).
// The stencil phases run over (row, mode) items, RPT consecutive rows per
// thread, from columns in LDS; the sweeps run on one lane per real column,
// four lanes ((+-k) x (Re, Im)) per operator, with the factor rows staged
// through LDS: every thread fetches its share of the factors into registers
// a phase ahead and hands them over in chunks of rows.
//
// The kernel sequence wrote and read eight intermediate fields (right sides,
// divergence, p0, X0, each through HBM or the last-level cache) and read each
// factor row twice, once per sign of k; this reads 2.5 to 3.5 states and the
// factors and writes one state.  Measured per stage, sequence -> this:
// 32 points x 16 x 31 modes 34 -> 14 us, heated 64 x 64 x 127 109 -> 70 us,
// pipe 64 x 64 x 127 97 -> 47 us, 128 x 256 x 511 2840 -> 1740 us (6.6 GB of
// counted traffic, 3.8 TB/s).  What bounds it: on the large grid the fetched
// bytes and, with two workgroups' columns filling a compute unit's LDS, the
// latency of the recurrences (two workgroups of eight modes take turns in
// loading and sweeping); on the small ones the latency alone.  The registers
// of the phases are kept below 256 by hand (loads issued one phase ahead, not
// two; scheduling barriers), because spills cost more than the latency they
// hide: 65 spilled registers wrote 1.1 GB per launch on 128 x 256 x 511.
#include <cfloat>
#include <type_traits>

#include "solve_common.h"

namespace nsc {
namespace {

constexpr int kStageThreads = 256;
constexpr int kBlock = 12;          // rows per unrolled block of a recurrence
constexpr int kRing = 6;            // factor rows in registers (kBlock is a multiple)
constexpr int kPad = 8;             // complex values between fields: next field on the other banks

// (a native vector: arrays of HIP's double2 class do not stay in registers)
typedef double Dbl2 __attribute__((ext_vector_type(2)));

// 16 or 8 bytes at a uniform base plus a 32-bit byte offset (one scalar pair
// and one vector register per address; stage_fused keeps the arrays below
// 4 GiB)
template <class V>
__device__ __forceinline__ V at(const void *base, unsigned off) {
  return *reinterpret_cast<const V *>(reinterpret_cast<const char *>(base) + off);
}
__device__ __forceinline__ Cd ldc(const double2 *base, unsigned off) {
  const Dbl2 v = at<Dbl2>(base, off);
  return Cd{v.x, v.y};
}
__device__ __forceinline__ void stc(double2 *base, unsigned off, Cd v) {
  *reinterpret_cast<Dbl2 *>(reinterpret_cast<char *>(base) + off) = Dbl2{v.x, v.y};
}

struct StageArgs {
  Factors fp, fv, ft;
  Influence inf;
  const double2 *u, *nn, *nq;
  double2 *out, *pout;
  double idt, cc, cq, cn;
  int walls, head;
};

// LDS layout in doubles: three fields, the edge entries E, then one region
// for the weight tables T1 and T2 and the factor chunks: T2 and the chunks of
// the pressure and temperature sweeps behind T1, those of the velocity sweeps
// from its start.  kc_*: rows per chunk (multiples of kBlock; the last chunk
// brings the four rows past the band rows along).
struct StageLds {
  int fs;  // field stride, complex
  int e, t1, t2, total, kc_pt, kc_v;
};

// rows n, RPT rows per thread, npt pressure and temperature systems; budget in
// doubles.  total > budget if even the smallest chunks do not fit.
template <int OPS>
StageLds stage_lds(int n, int rpt, int npt, int budget) {
  StageLds l;
  const int nw = ((n + rpt - 1) / rpt * rpt * (rpt + 8) + 1) & ~1;  // one table of padded weights
  l.fs = n * 2 * OPS + kPad;
  l.e = 2 * 3 * l.fs;
  l.t1 = l.e + 3 * kEdge * OPS;
  l.t2 = l.t1 + nw;
  const int most = (n - 4 + kBlock - 1) / kBlock * kBlock;
  auto rows = [&](int room, int ns) {
    int kc = (room / (ns * OPS * 5) - 4) / kBlock * kBlock;
    if (kc > most) kc = most;
    return kc < kBlock ? kBlock : kc;
  };
  l.kc_pt = rows(budget - l.t2, npt);
  l.kc_v = rows(budget - l.t1, 3);
  const int a = l.t2 + nw, b = l.t2 + (l.kc_pt + 4) * npt * OPS * 5, c = l.t1 + (l.kc_v + 4) * 3 * OPS * 5;
  l.total = a > b ? a : b;
  if (c > l.total) l.total = c;
  return l;
}

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// First row of the window that holds the nine-point windows of all RPT rows
// from j0 on (RPT + 8 rows).
template <int RPT>
__device__ __forceinline__ int win_base(int j0, int n) { return clampi(j0 - 4, 0, n - (RPT + 8)); }

// Weight table with each row's nine weights placed in its group's window and
// zeros elsewhere (also in the rows past n - 1 of the last group):
// dst[j][RPT + 8].
template <int RPT>
__device__ __forceinline__ void fill_weights(double *dst, const double *__restrict__ w, int n, int t) {
  constexpr int W = RPT + 8;
  const int rows = (n + RPT - 1) / RPT * RPT;
  for (int i = t; i < rows * W; i += kStageThreads) {
    const int j = i / W, e = i - j * W;
    const int tt = e + win_base<RPT>(j / RPT * RPT, n) - clampi(j - 4, 0, n - kStencil);
    dst[i] = j < n && tt >= 0 && tt < kStencil ? w[j * kStencil + tt] : 0.0;
  }
}

// Stencil sums of NF fields over the thread's RPT rows: acc[f][jj] =
// sum_e w[j0 + jj][e] x_f[base + e], from the left.
template <int OPS, int RPT, int NF>
__device__ __forceinline__ void stencil(const double *w, const Cd *x, int fs, Cd (&acc)[NF][RPT]) {
  constexpr int W = RPT + 8;
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int jj = 0; jj < RPT; ++jj) acc[f][jj] = Cd{0.0, 0.0};
  // one window row read ahead; the scheduling barriers keep the compiler from
  // hoisting every read (and spilling)
  Cd v[2][NF];
  double wt[2][RPT];
  auto load = [&](int e) {
#pragma unroll
    for (int f = 0; f < NF; ++f) v[e & 1][f] = x[f * fs + e * 2 * OPS];
#pragma unroll
    for (int jj = 0; jj < RPT; ++jj) wt[e & 1][jj] = w[jj * W + e];
  };
  load(0);
#pragma unroll
  for (int e = 0; e < W; ++e) {
    if (e + 1 < W) load(e + 1);
#pragma unroll
    for (int jj = 0; jj < RPT; ++jj)
#pragma unroll
      for (int f = 0; f < NF; ++f) acc[f][jj] = fmac(wt[e & 1][jj], v[e & 1][f], acc[f][jj]);
    __builtin_amdgcn_sched_barrier(0);
  }
  // the sums are taken here: sunk past the branches of later phases, they
  // would keep every operand in registers
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int jj = 0; jj < RPT; ++jj) asm volatile("" : "+v"(acc[f][jj].x), "+v"(acc[f][jj].y));
}

// The factors of NS systems on the way from HBM to the sweeps: this thread's
// share of the L or U rows, the inverse diagonals, and the edge entries, in
// registers.
template <int OPS, int NS, int RPT>
struct FactorRegs {
  static constexpr int DQ = (RPT + 1) / 2;
  Dbl2 q[NS][RPT];  // L or U quarters: flat index t + i T over [row][op][2]
  double dg[NS][DQ];   // diagonals: flat index over [row][op]
  double ed[NS];

  // system s: op0 the tile's first operator (ops past the last live one
  // repeat it).  Rows in sweep order: the L rows upwards, the U rows
  // (BACK) downwards from n - 1.
  template <bool BACK>
  __device__ __forceinline__ void load(int s, const Factors &F, int op0, int nlive, int n, int t) {
    {
      const int o = (t / 2) % OPS;
      const unsigned col = (unsigned)(o < nlive ? o : nlive - 1) * 32 + 16 * (t & 1);
      const double *p = F.pk + ((size_t)(BACK ? 1 : 0) * F.nops + op0) * 4;
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        int row = t / (2 * OPS) + i * (kStageThreads / (2 * OPS));
        row = row < n ? row : n - 1;
        if (BACK) row = n - 1 - row;
        q[s][i] = at<Dbl2>(p, (unsigned)row * ((unsigned)F.nops * 64) + col);
      }
    }
    if (BACK) {
      const int o = t % OPS;
      const unsigned col = (unsigned)(o < nlive ? o : nlive - 1) * 8;
      const double *p = F.vals + 4 * (size_t)F.nops + op0;
#pragma unroll
      for (int i = 0; i < DQ; ++i) {
        int row = t / OPS + i * (kStageThreads / OPS);
        row = row < n ? row : n - 1;
        dg[s][i] = at<double>(p, (unsigned)(n - 1 - row) * ((unsigned)F.nops * (8 * kSlots)) + col);
      }
    }
  }
  __device__ __forceinline__ void load_edges(int s, const Factors &F, int op0, int nlive, int t) {
    const int o = t % OPS;
    if (t < kEdge * OPS)
      ed[s] = F.edge[(size_t)(t / OPS) * F.nops + op0 + (o < nlive ? o : nlive - 1)];
  }
  __device__ __forceinline__ void store_edges(double *E, int t) const {
#pragma unroll
    for (int s = 0; s < NS; ++s)
      if (t < kEdge * OPS) E[s * kEdge * OPS + t] = ed[s];
  }
  // rows [r0, r1) of the sweep order to B[row - r0][system][op][4], the
  // diagonals (BACK) to D[row - r0][system][op]
  template <bool BACK>
  __device__ __forceinline__ void store_rows(double *B, double *D, int r0, int r1, int t) const {
    constexpr int RQ = kStageThreads / (2 * OPS), RD = kStageThreads / OPS;  // rows per register
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int row = t / (2 * OPS) + i * RQ;
      if (row >= r0 && row < r1)
#pragma unroll
        for (int s = 0; s < NS; ++s)
          *reinterpret_cast<Dbl2 *>(B + ((row - r0) * NS + s) * (4 * OPS) + 2 * (t % (2 * OPS))) = q[s][i];
    }
    if (BACK) {
#pragma unroll
      for (int i = 0; i < DQ; ++i) {
        const int row = t / OPS + i * RD;
        if (row >= r0 && row < r1)
#pragma unroll
          for (int s = 0; s < NS; ++s) D[((row - r0) * NS + s) * OPS + t % OPS] = dg[s][i];
      }
    }
  }
};

// One real column's recurrence: the last four values, newest first.
struct Carry {
  double y1, y2, y3, y4;
};

// One factor row and right side of a sweeping lane.
struct Row {
  Dbl2 qa, qb;
  double b, dg;
};

// A sweeping lane's recurrence, rows in sweep order: forward y = b - L y,
// backward x = (y - U x) / U_jj.
template <int OPS, bool BACK, int NS>
struct Recur {
  static constexpr int cs = BACK ? -4 * OPS : 4 * OPS;    // column step per row
  static constexpr int qs = NS * 4 * OPS, ds = NS * OPS;  // factor steps per row
  __device__ __forceinline__ static Row row(const double *c, const double *S, const double *D, int i) {
    Row r;
    r.qa = *reinterpret_cast<const Dbl2 *>(S + i * qs);
    r.qb = *reinterpret_cast<const Dbl2 *>(S + i * qs + 2);
    r.b = c[i * cs];
    r.dg = BACK ? D[i * ds] : 0.0;
    return r;
  }
  // entry at distance d = 1..4: L(j, j-d) or U(j, j+d)
  __device__ __forceinline__ static double e(const Row &r, int d) {
    return BACK ? (d == 1 ? r.qa.x : d == 2 ? r.qa.y : d == 3 ? r.qb.x : r.qb.y)
                : (d == 1 ? r.qb.y : d == 2 ? r.qb.x : d == 3 ? r.qa.y : r.qa.x);
  }
  // LEN rows (a multiple of kRing, or one ring's part) from the ring's rows;
  // the rows past LEN - kRing are replaced by the next block's if `more`.
  // Each new value is subtracted from the rows it enters at once (independent
  // multiply-adds), so that one of them and the diagonal's product lie
  // between a row and the next; every row takes its terms from the farthest
  // to the nearest.
  template <int LEN, int R>
  __device__ __forceinline__ static void rows(Row (&w)[R], Carry &k, double *c, const double *S,
                                              const double *D, bool more) {
    static_assert(R >= 4 && LEN % R == 0, "the ring holds the rows a value enters");
    double s0 = fma(-e(w[0], 2), k.y2, fma(-e(w[0], 3), k.y3, fma(-e(w[0], 4), k.y4, w[0].b)));
    double s1 = fma(-e(w[1], 3), k.y2, fma(-e(w[1], 4), k.y3, w[1].b));
    double s2 = fma(-e(w[2], 4), k.y2, w[2].b);
#pragma unroll
    for (int i = 0; i < LEN; ++i) {
      const double yp = k.y1;
      double y = fma(-e(w[i % R], 1), yp, s0);
      if (BACK) y *= w[i % R].dg;
      if (i + 1 < LEN) s0 = fma(-e(w[(i + 1) % R], 2), yp, s1);
      if (i + 2 < LEN) s1 = fma(-e(w[(i + 2) % R], 3), yp, s2);
      if (i + 3 < LEN) s2 = fma(-e(w[(i + 3) % R], 4), yp, w[(i + 3) % R].b);
      k = Carry{y, k.y1, k.y2, k.y3};
      c[i * cs] = y;
      if (i + R < LEN || more) w[i % R] = row(c, S, D, i + R);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // One row on its own.
  __device__ __forceinline__ static void one(Carry &k, double *c, const double *S, const double *D) {
    const Row r = row(c, S, D, 0);
    double y = fma(-e(r, 4), k.y4, r.b);
    y = fma(-e(r, 3), k.y3, y);
    y = fma(-e(r, 2), k.y2, y);
    y = fma(-e(r, 1), k.y1, y);
    if (BACK) y *= r.dg;
    c[0] = y;
    k = Carry{y, k.y1, k.y2, k.y3};
  }
  // The four rows with the envelope entries E (stride OPS) of the one-sided
  // wall rows: row n-4+q (backward 3-q) has q + 1 entries past the band,
  // entry t at edge_off(3 - q) + t of the wall's list, by ascending column:
  // n-9.. forward, ..8 backward.  Everything is read before the first row.
  __device__ __forceinline__ static void tail(Carry k, double *c, const double *S, const double *D,
                                              const double *E) {
    Row w[4];
    double ed[10];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = row(c, S, D, i);
#pragma unroll
    for (int t = 0; t < 10; ++t) ed[t] = E[((BACK ? 0 : 10) + t) * OPS];
    // the values five to two rows before the four rows
    const double far[4] = {c[-5 * cs], k.y4, k.y3, k.y2};
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      double y = w[q].b;
      y = fma(-e(w[q], 1), k.y1, y);
      y = fma(-e(w[q], 2), k.y2, y);
      y = fma(-e(w[q], 3), k.y3, y);
      y = fma(-e(w[q], 4), k.y4, y);
#pragma unroll
      for (int t = 0; t <= q; ++t)  // forward column n-9+t; backward column 8-q+t
        y = fma(-ed[edge_off(3 - q) + t], far[BACK ? q - t : t], y);
      if (BACK) y *= w[q].dg;
      c[q * cs] = y;
      k = Carry{y, k.y1, k.y2, k.y3};
    }
  }
};

// One direction of the sweeps of NS systems, fields 0..NS-1 in place: the
// workgroup hands the factor rows over in chunks of kc rows, the first
// 4 OPS NS threads run one real column each.
template <bool BACK, int OPS, int NS, int RPT>
__device__ __forceinline__ void sweep_dir(const FactorRegs<OPS, NS, RPT> &R, double *fld, int fs, double *S,
                                          int kc, const double *E, int n, int t) {
  using Q = Recur<OPS, BACK, NS>;
  constexpr int kCols = 4 * OPS;  // real columns per field
  const int nb = n - 4;           // band rows; the last four follow in the last chunk
  const int sys = t / kCols, col = t % kCols, o = (col >> 1) % OPS;
  const bool lane = t < NS * kCols;
  double *c0 = fld + (size_t)sys * 2 * fs + col + (BACK ? (n - 1) * kCols : 0);
  double *D = S + (kc + 4) * Q::qs;
  const double *Sl = S + sys * 4 * OPS + o * 4, *Dl = D + sys * OPS + o;
  const double *El = E + sys * kEdge * OPS + o;
  Carry k{0.0, 0.0, 0.0, 0.0};
  for (int i0 = 0; i0 < nb; i0 += kc) {
    const bool last = i0 + kc >= nb;
    const int i1 = last ? n : i0 + kc;
    R.template store_rows<BACK>(S, D, i0, i1, t);
    __syncthreads();
    if (lane) {
      const int len = last ? nb - i0 : kc;
      double *c = c0 + i0 * Q::cs;
      int i = 0;
      if (len >= kBlock) {
        Row w[kRing];
#pragma unroll
        for (int r = 0; r < kRing; ++r) w[r] = Q::row(c, Sl, Dl, r);
        __builtin_amdgcn_sched_barrier(0);
        for (; i + kBlock <= len; i += kBlock)
          Q::template rows<kBlock>(w, k, c + i * Q::cs, Sl + i * Q::qs, Dl + i * Q::ds,
                                   i + 2 * kBlock <= len);
      }
      for (; i + 4 <= len; i += 4) {
        Row w[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] = Q::row(c + i * Q::cs, Sl + i * Q::qs, Dl + i * Q::ds, r);
        Q::template rows<4>(w, k, c + i * Q::cs, Sl + i * Q::qs, Dl + i * Q::ds, false);
      }
      for (; i < len; ++i) Q::one(k, c + i * Q::cs, Sl + i * Q::qs, Dl + i * Q::ds);
      if (last) Q::tail(k, c + i * Q::cs, Sl + i * Q::qs, Dl + i * Q::ds, El);
    }
    __syncthreads();
  }
}

__device__ __forceinline__ double xor_lane(double v, int mask) { return __shfl_xor(v, mask, 64); }
template <int OPS>
__device__ __forceinline__ Cd herm_pair(Cd v) {  // (v + conj(v of the -k lane)) / 2
  return Cd{0.5 * (v.x + xor_lane(v.x, OPS)), 0.5 * (v.y - xor_lane(v.y, OPS))};
}

template <int OPS, int RPT, bool HEATED, bool PIPE, bool WITH_P>
__global__ void __launch_bounds__(kStageThreads, 2) k_stage(Dims d, Grid g, StageArgs a, StageLds lay) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int W = RPT + 8;
  constexpr int kModes = 2 * OPS;
  constexpr int NPT = HEATED ? 2 : 1;
  const int n = d.nr, K = d.kmax, kp1 = K + 1;
  double *base = reinterpret_cast<double *>(smem);
  Cd *fA = reinterpret_cast<Cd *>(smem), *fB = fA + lay.fs, *fC = fB + lay.fs;
  double *T1 = base + lay.t1, *S = base + lay.t2, *E = base + lay.e;
  const int t = threadIdx.x;
  // neighbouring |k| tiles share cache lines: contiguous tiles per XCD
  // (spans of 16 |k| with m next, for the factors that q = m, m + 1 share,
  // fetched as much and ran 4 % longer on 128 x 256 x 511)
  const int kt = (kp1 + OPS - 1) / OPS;
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  const int m = L / kt, ka0 = (L - m * kt) * OPS;
  const int nlive = kp1 - ka0 < OPS ? kp1 - ka0 : OPS;
  const int ml = t % kModes, rg = t / kModes;
  const int o = ml % OPS, sg = ml / OPS;
  const int ka = ka0 + (o < nlive ? o : nlive - 1);
  const int kk = sg ? K - ka : K + ka;
  const bool live = o < nlive && !(sg && ka == 0);  // the other lanes repeat a live one
  const bool zero = m == 0 && ka == 0;
  const int md = m * d.mz + kk;
  const size_t fst = (size_t)n * d.nmodes;
  const double kap = (double)(kk - K) * d.kz;
  const double k2 = kap * kap, mm = (double)m;
  const double ce = 1.0 - a.cc;
  const int j0 = rg * RPT;
  const int wb = win_base<RPT>(j0 < n ? j0 : n - 1, n);
  const Cd *win = fA + wb * kModes + ml;           // window of field A
  // (threads past the last row repeat row 0's weights and store nothing)
  const int jw = j0 < n ? j0 : 0;
  auto rowc = [&](int jj) { return j0 + jj < n ? j0 + jj : n - 1; };
  auto ok = [&](int jj) { return j0 + jj < n; };
  auto inner = [&](int j) { return (PIPE || j > 0) && j < n - 1; };
  // this lane's entries of a field, at byte offset row * 16 P + 16 md
  const unsigned row16 = (unsigned)d.nmodes * 16, md16 = (unsigned)md * 16;
  auto off = [&](int jj) { return (unsigned)rowc(jj) * row16 + md16; };
  // c N^q + (1-c) N^n (no branches on what is given: the host passes u^n with
  // coefficients zero for no nonlinear term)
  auto Nv = [&](int f, unsigned at) -> Cd {
    return a.cq * ldc(a.nq + f * fst, at) + a.cn * ldc(a.nn + f * fst, at);
  };
  const double *wl = g.lw, *wd = g.d1;
  // ---- u^n and its stencils: f = X^n/dt + (1-c) L X^n + c N^q + (1-c) N^n
  // (the scheduling barriers bound what is in flight at once: left alone, the
  // compiler hoists the loads of later phases and spills)
  Cd n0[RPT], n1[RPT];
  {
    Cd v[3][RPT];
#pragma unroll
    for (int f = 0; f < 3; ++f)
#pragma unroll
      for (int jj = 0; jj < RPT; ++jj) v[f][jj] = ldc(a.u + f * fst, off(jj));
#pragma unroll
    for (int jj = 0; jj < RPT; ++jj) {
      n0[jj] = Nv(0, off(jj));
      n1[jj] = Nv(1, off(jj));
    }
    __builtin_amdgcn_sched_barrier(0);
    fill_weights<RPT>(S, wl + (PIPE ? odd_off(g, m + 1) : 0), n, t);
    if (PIPE) fill_weights<RPT>(T1, wl + odd_off(g, m), n, t);
#pragma unroll
    for (int jj = 0; jj < RPT; ++jj)
      if (ok(jj)) {
        const int pos = (j0 + jj) * kModes + ml;
        fA[pos] = v[0][jj];
        fB[pos] = v[1][jj];
        fC[pos] = v[2][jj];
      }
  }
  __syncthreads();
  Cd fp[RPT], fm[RPT], fz[RPT];
  {
    Cd l[2][RPT];
    stencil<OPS, RPT, 2>(S + jw * W, win, lay.fs, l);
    const double qp = mm + 1.0, qm = m >= 1 ? mm - 1.0 : 1.0;
#pragma unroll
    for (int jj = 0; jj < RPT; ++jj) {
      const int pos = rowc(jj) * kModes + ml;
      const double ri = g.rinv[rowc(jj)];
      const double r2 = ri * ri;
      const Cd ur = fA[pos], ut = fB[pos];
      const Cd xp = ur + ci(ut), xm = ur - ci(ut);
      const Cd lp = l[0][jj] + ci(l[1][jj]), lm = l[0][jj] - ci(l[1][jj]);
      const Cd Lp = lp - (qp * qp * r2 + k2) * xp;
      const Cd Lm = lm - (qm * qm * r2 + k2) * xm;
      fp[jj] = a.idt * xp + ce * Lp + (n0[jj] + ci(n1[jj]));
      fm[jj] = a.idt * xm + ce * Lm + (n0[jj] - ci(n1[jj]));
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  {
    Cd l[1][RPT], n2[RPT];
#pragma unroll
    for (int jj = 0; jj < RPT; ++jj) n2[jj] = Nv(2, off(jj));
    __builtin_amdgcn_sched_barrier(0);
    stencil<OPS, RPT, 1>((PIPE ? T1 : S) + jw * W, win + 2 * lay.fs, lay.fs, l);
#pragma unroll
    for (int jj = 0; jj < RPT; ++jj) {
      const double ri = g.rinv[rowc(jj)];
      const double r2 = ri * ri;
      const Cd uz = fC[rowc(jj) * kModes + ml];
      const Cd Lz = l[0][jj] - (mm * mm * r2 + k2) * uz;
      fz[jj] = a.idt * uz + ce * Lz + n2[jj];
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  Cd nT[RPT];
  {
    Cd tT[RPT];
    if constexpr (HEATED) {
#pragma unroll
      for (int jj = 0; jj < RPT; ++jj) {
        tT[jj] = ldc(a.u + 3 * fst, off(jj));
        nT[jj] = Nv(3, off(jj));
      }
    }
    __syncthreads();
#pragma unroll
    for (int jj = 0; jj < RPT; ++jj)
      if (ok(jj)) {
        const int pos = (j0 + jj) * kModes + ml;
        fA[pos] = fp[jj];
        fB[pos] = fm[jj];
        if (HEATED) fC[pos] = tT[jj];
      }
  }
  __builtin_amdgcn_sched_barrier(0);
  fill_weights<RPT>(T1, wd + (PIPE ? odd_off(g, m + 1) : 0), n, t);
  // the pressure and temperature factors come next
  FactorRegs<OPS, NPT, RPT> L1, U1;
  const int opm = m * kp1 + ka0;
  L1.template load<false>(0, a.fp, opm, nlive, n, t);
  L1.load_edges(0, a.fp, opm, nlive, t);
  if constexpr (HEATED) {
    L1.template load<false>(NPT - 1, a.ft, opm, nlive, n, t);
    L1.load_edges(NPT - 1, a.ft, opm, nlive, t);
  }
  __syncthreads();
  // ---- Poisson right side g = mask(div f), temperature right side
  {
    Cd dv[2][RPT], lT[1][RPT];
    stencil<OPS, RPT, 2>(T1 + jw * W, win, lay.fs, dv);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (HEATED) {
      stencil<OPS, RPT, 1>(S + jw * W, win + 2 * lay.fs, lay.fs, lT);
#pragma unroll
      for (int jj = 0; jj < RPT; ++jj) {
        const int j = rowc(jj);
        const double ri = g.rinv[j], r2 = ri * ri;
        const Cd T = fC[j * kModes + ml];
        const Cd Lx = lT[0][jj] - (mm * mm * r2 + k2) * T;
        nT[jj] = a.idt * T + (ce / d.pr) * Lx + nT[jj];
        if (j == 0 || j == n - 1) nT[jj] = Cd{zero && a.walls ? (j == 0 ? 0.5 : -0.5) : 0.0, 0.0};
      }
    }
    __syncthreads();
#pragma unroll
    for (int jj = 0; jj < RPT; ++jj) {
      const int j = rowc(jj);
      const double ri = g.rinv[j];
      Cd gv = 0.5 * ((dv[0][jj] + ((1.0 + mm) * ri) * fp[jj]) + (dv[1][jj] + ((1.0 - mm) * ri) * fm[jj])) +
              kap * ci(fz[jj]);
      if (!inner(j)) gv = Cd{0.0, 0.0};
      gv = Cd{zero ? 0.0 : gv.x, zero ? 0.0 : gv.y};
      // (f+, and f- of a heated run, wait in registers; the rest in LDS)
      const int pos = j * kModes + ml;
      if (ok(jj)) {
        fA[pos] = gv;
        if constexpr (HEATED) fB[pos] = nT[jj];
        fC[pos] = fz[jj];
      }
    }
  }
  if (a.head && m == 0 && ka0 == 0 && zero) {
    // mode (0,0) where the pressure is asked for: the mean head's right side
    // (D1 + 1/r) F_r, F_r(r_o) at the outer wall (pipe: every row but the
    // wall's, where p = 0)
#pragma unroll 1
    for (int j = j0; j < j0 + RPT && j < n; ++j) {
      if (PIPE ? j == n - 1 : j == 0) continue;
      auto Fr = [&](int row) { return Nv(0, (unsigned)row * row16 + md16); };
      Cd gv = Fr(j);
      if (j < n - 1) {
        gv = g.rinv[j] * gv;
        const int s0 = clampi(j - 4, 0, n - kStencil);
        const double *w = g.d1 + g.podd + j * kStencil;
#pragma unroll 1
        for (int e = 0; e < kStencil; ++e) gv = fmac(w[e], Fr(s0 + e), gv);
      }
      fA[j * kModes + ml] = gv;
    }
  }
  L1.store_edges(E, t);
  if (PIPE) fill_weights<RPT>(T1, wd + odd_off(g, m), n, t);
  // ---- pressure and temperature sweeps (their U rows on their way)
  const int op_v[3] = {(m + 1) * kp1 + ka0, (m >= 1 ? m - 1 : 1) * kp1 + ka0, opm};
  U1.template load<true>(0, a.fp, opm, nlive, n, t);
  if constexpr (HEATED) {
    U1.template load<true>(NPT - 1, a.ft, opm, nlive, n, t);
  }
  sweep_dir<false, OPS, NPT, RPT>(L1, base, lay.fs, S, lay.kc_pt, E, n, t);
  sweep_dir<true, OPS, NPT, RPT>(U1, base, lay.fs, S, lay.kc_pt, E, n, t);
  // ---- temperature out; velocity right sides f - grad p0 (the velocity L
  // rows on their way)
  FactorRegs<OPS, 3, RPT> L2;
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    L2.template load<false>(s, a.fv, op_v[s], nlive, n, t);
    L2.load_edges(s, a.fv, op_v[s], nlive, t);
  }
  Cd p0[RPT];
  {
    Cd dp[1][RPT];
    stencil<OPS, RPT, 1>(T1 + jw * W, win, lay.fs, dp);
#pragma unroll
    for (int jj = 0; jj < RPT; ++jj) {
      const int j = rowc(jj);
      const Cd p = fA[j * kModes + ml];
      p0[jj] = p;
      fz[jj] = fC[j * kModes + ml];
      if constexpr (!HEATED) fm[jj] = fB[j * kModes + ml];
      if constexpr (HEATED) {
        Cd T = fB[j * kModes + ml];
        if (m == 0) T = herm_pair<OPS>(T);
        if (live && ok(jj)) stc(a.out + 3 * fst, off(jj), T);
      }
      // inside f - grad p0, zero at the walls; mode (0,0) solves u_theta
      // directly (X+- = +-i u_theta) under the wall speeds, and u_z (pipe:
      // with the driving gradient)
      const bool in = inner(j);
      const Cd mp = (mm * g.rinv[j]) * p;
      const Cd h = 0.5 * (fp[jj] - fm[jj]);
      const double wall = a.walls ? (j == 0 ? d.re_i : d.re_o) : 0.0;
      const Cd gp = fp[jj] - (dp[0][jj] - mp), gm = fm[jj] - (dp[0][jj] + mp);
      const Cd gz = fz[jj] - kap * ci(p);
      const double drive = PIPE && a.walls ? d.gp : 0.0;
      fp[jj].x = in ? (zero ? h.x : gp.x) : 0.0;
      fp[jj].y = in ? (zero ? h.y : gp.y) : (zero ? wall : 0.0);
      fm[jj].x = in ? (zero ? -h.x : gm.x) : 0.0;
      fm[jj].y = in ? (zero ? -h.y : gm.y) : (zero ? -wall : 0.0);
      fz[jj].x = in ? (zero ? fz[jj].x + drive : gz.x) : 0.0;
      fz[jj].y = in ? (zero ? fz[jj].y : gz.y) : 0.0;
    }
  }
  __syncthreads();
#pragma unroll
  for (int jj = 0; jj < RPT; ++jj)
    if (ok(jj)) {
      const int pos = (j0 + jj) * kModes + ml;
      fA[pos] = fp[jj];
      fB[pos] = fm[jj];
      fC[pos] = fz[jj];
    }
  L2.store_edges(E, t);
  // ---- velocity sweeps; the U rows, then the responses follow
  FactorRegs<OPS, 3, RPT> U2;
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    U2.template load<true>(s, a.fv, op_v[s], nlive, n, t);
  }
  sweep_dir<false, OPS, 3, RPT>(L2, base, lay.fs, T1, lay.kc_v, E, n, t);
  Dbl2 rs[WITH_P ? 4 : 3][RPT];
  const int opi = m * kp1 + ka;
#pragma unroll
  for (int jj = 0; jj < RPT; ++jj) {
    auto R = [&](int kind) {
      return at<Dbl2>(a.inf.resp + (size_t)kind * n * a.inf.nops,
                      ((unsigned)rowc(jj) * (unsigned)a.inf.nops + (unsigned)opi) * 16);
    };
    rs[0][jj] = R(1);
    rs[1][jj] = R(2);
    rs[2][jj] = R(3);
    if constexpr (WITH_P) rs[WITH_P ? 3 : 0][jj] = R(0);
  }
  sweep_dir<true, OPS, 3, RPT>(U2, base, lay.fs, T1, lay.kc_v, E, n, t);
  // ---- lambda = -A^-1 beta(X0), beta the wall divergences: one lane per
  // (wall, mode); S is free again
  Cd *lam = reinterpret_cast<Cd *>(S);
  if (t < 2 * kModes) {
    const int w = t / kModes;
    const int j = w == 0 ? 0 : n - 1;
    const int s0 = w == 0 ? 0 : n - kStencil;
    Cd beta = {0.0, 0.0};
    if (!(PIPE && w == 0)) {  // pipe: one wall, beta[0] = 0
      const double *wr = g.d1 + (PIPE ? odd_off(g, m + 1) : 0) + j * kStencil;
      const double ri = g.rinv[j];
      Cd dp = {0.0, 0.0}, dm = {0.0, 0.0};
#pragma unroll
      for (int e = 0; e < kStencil; ++e) {
        dp = fmac(wr[e], fA[(s0 + e) * kModes + ml], dp);
        dm = fmac(wr[e], fB[(s0 + e) * kModes + ml], dm);
      }
      beta = 0.5 * ((dp + ((1.0 + mm) * ri) * fA[j * kModes + ml]) +
                    (dm + ((1.0 - mm) * ri) * fB[j * kModes + ml])) +
             kap * ci(fC[j * kModes + ml]);
    }
    const Cd other = {xor_lane(beta.x, kModes), xor_lane(beta.y, kModes)};
    const Cd b0 = w == 0 ? beta : other, b1 = w == 0 ? other : beta;
    const size_t ns = a.inf.nops;
    const double a0 = a.inf.ainv[(size_t)(2 * w) * ns + opi], a1 = a.inf.ainv[(size_t)(2 * w + 1) * ns + opi];
    Cd l = {-(a0 * b0.x + a1 * b1.x), -(a0 * b0.y + a1 * b1.y)};
    if (zero) l = Cd{0.0, 0.0};
    lam[w * kModes + ml] = l;
  }
  __syncthreads();
  // ---- X = X0 + sum lambda_j X_j, back to (r, theta), m = 0 Hermitian
  const Cd l1 = lam[ml], l2 = lam[kModes + ml];
#pragma unroll
  for (int jj = 0; jj < RPT; ++jj) {
    const int j = rowc(jj);
    auto hom = [&](Dbl2 r) { return r.x * l1 + r.y * l2; };
    Cd xp = fA[j * kModes + ml], xm = fB[j * kModes + ml], xz = fC[j * kModes + ml];
    Cd p = p0[jj];
    if (!zero) {
      xp = xp + hom(rs[0][jj]);
      xm = xm + hom(rs[1][jj]);
      xz = xz - kap * ci(hom(rs[2][jj]));  // X_z,j = -i kappa h_j
      if constexpr (WITH_P) p = p + hom(rs[WITH_P ? 3 : 0][jj]);
    }
    Cd vr = 0.5 * (xp + xm);
    const Cd dd = xp - xm;  // u_theta = (X+ - X-) / (2 i)
    Cd vt = {0.5 * dd.y, -0.5 * dd.x};
    if (m == 0) {
      vr = herm_pair<OPS>(vr);
      vt = herm_pair<OPS>(vt);
      xz = herm_pair<OPS>(xz);
      if constexpr (WITH_P) p = herm_pair<OPS>(p);
    }
    if (live && ok(jj)) {
      stc(a.out, off(jj), vr);
      stc(a.out + fst, off(jj), vt);
      stc(a.out + 2 * fst, off(jj), xz);
      if constexpr (WITH_P) stc(a.pout, off(jj), p);
    }
  }
}

// Launch shape: |k| values per workgroup, rows per thread, LDS layout (within
// half a compute unit's LDS where the grid fits, so that two workgroups share
// one).
struct StageShape {
  int ops, rpt;
  StageLds lds;
};

template <int OPS>
StageShape shape_for(const nsc_ctx *c) {
  const int groups = kStageThreads / (2 * OPS), n = c->d.nr;
  const int rpt = (n + groups - 1) / groups, npt = c->d.heated ? 2 : 1;
  StageShape sh{OPS, rpt, stage_lds<OPS>(n, rpt, npt, c->lds_cu / 2 / 8)};
  return sh;
}

StageShape stage_shape(const nsc_ctx *c) {
  const long tiles = (long)c->d.mt * ((c->d.kmax + 8) / 8);
  return c->d.nr <= 64 && tiles >= c->cu_count ? shape_for<8>(c) : shape_for<4>(c);
}

}  // namespace

bool stage_fused(const nsc_ctx *c) {
  const Dims &d = c->d;
  if (d.nr > kStageRows) return false;
  // 32-bit byte offsets: fields, factor rows (72 bytes per operator and
  // row), responses
  const size_t nops = (size_t)(d.mt + 1) * (d.kmax + 1);
  if ((size_t)d.nr * d.nmodes * 16 >> 32 || (size_t)d.nr * nops * 72 >> 32) return false;
  return (size_t)stage_shape(c).lds.total * sizeof(double) <= (size_t)c->lds_max;
}

hipError_t launch_stage(const nsc_ctx *c, const double *u, const double *nn, const double *nq,
                        double *out, double *pout, double dt, double cc, int walls) {
  const Dims &d = c->d;
  StageArgs a{c->fp, c->fv, c->ft, c->inf, reinterpret_cast<const double2 *>(u),
              reinterpret_cast<const double2 *>(nn ? nn : u),
              reinterpret_cast<const double2 *>(nn ? nq : u), reinterpret_cast<double2 *>(out),
              reinterpret_cast<double2 *>(pout), 1.0 / dt, cc, nn ? cc : 0.0, nn ? 1.0 - cc : 0.0,
              walls, pout && nn ? 1 : 0};
  const StageShape sh = stage_shape(c);
  const int kt = (d.kmax + sh.ops) / sh.ops;
  auto go = [&](auto ops, auto rows) {
    constexpr int OPS = decltype(ops)::value, RPT = decltype(rows)::value;
    auto kern = d.pipe ? (pout ? k_stage<OPS, RPT, false, true, true> : k_stage<OPS, RPT, false, true, false>)
              : d.heated ? (pout ? k_stage<OPS, RPT, true, false, true> : k_stage<OPS, RPT, true, false, false>)
                         : (pout ? k_stage<OPS, RPT, false, false, true> : k_stage<OPS, RPT, false, false, false>);
    hipLaunchKernelGGL(kern, dim3(d.mt * kt), dim3(kStageThreads),
                       (size_t)sh.lds.total * sizeof(double), c->stream, d, c->g, a, sh.lds);
    return hipGetLastError();
  };
  auto rows = [&](auto ops) {
    switch (sh.rpt) {
      case 1: return go(ops, std::integral_constant<int, 1>{});
      case 2: return go(ops, std::integral_constant<int, 2>{});
      case 3: return go(ops, std::integral_constant<int, 3>{});
      default: return go(ops, std::integral_constant<int, 4>{});
    }
  };
  return sh.ops == 8 ? rows(std::integral_constant<int, 8>{}) : rows(std::integral_constant<int, 4>{});
}

}  // namespace nsc
