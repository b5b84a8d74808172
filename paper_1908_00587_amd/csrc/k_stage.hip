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
// The new state may replace u^n (nsc_step does): no other workgroup touches
// these columns, and every read of u^n, N^n, N^q lies before the barrier ahead
// of the pressure sweeps, every store behind it.
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
// 32 points x 16 x 31 modes 34 -> 14 us, heated 64 x 64 x 127 109 -> 73 us,
// pipe 64 x 64 x 127 97 -> 47 us, 128 x 256 x 511 2840 -> 1840 us (6.4 GB of
// counted traffic, 3.5 TB/s).  What bounds it: on the large grid the fetched
// bytes and, with two workgroups' columns filling a compute unit's LDS, the
// latency of the recurrences (two workgroups of eight modes take turns in
// loading and sweeping); on the small ones the latency alone.  The registers
// of the phases are kept below 256 by hand (loads issued one phase ahead, not
// two; scheduling barriers), because spills cost more than the latency they
// hide: 65 spilled registers wrote 1.1 GB per launch on 128 x 256 x 511.  Four
// rows per thread still spill 11, with the temperature 79.
#include <cfloat>
#include <type_traits>

#include "solve_common.h"

namespace nsc {
namespace {

constexpr int kStageThreads = 256;
constexpr int kBlock = 12;          // rows per unrolled block of a recurrence
constexpr int kRing = 6;            // factor rows in registers (kBlock is a multiple)
constexpr int kPad = 8;             // complex values between fields: next field on the other banks

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

// LDS layout in doubles: the edge entries E, three fields, then one region
// for the weight tables T1 and T2 and the factor chunks: T2 and the chunks of
// the pressure and temperature sweeps behind T1, those of the velocity sweeps
// from its start.  kc_*: rows per chunk (multiples of kBlock; the last chunk
// brings the four rows past the band rows along).
struct StageLds {
  int fs;  // field stride, complex
  int f, t1, t2, total, kc_pt, kc_v;
};

// rows n, rpt rows per thread, npt pressure and temperature systems, stencil
// windows of rpt + extra rows, one weight table or two; budget in doubles.  total > budget if even the smallest chunks do not fit.
template <int OPS>
StageLds stage_lds(int n, int rpt, int npt, int extra, bool two, int budget) {
  StageLds l;
  // one table of padded weights (windows of rpt + extra rows)
  const int nw = ((n + rpt - 1) / rpt * rpt * (rpt + extra) + 1) & ~1;
  l.fs = n * 2 * OPS + kPad;
  l.f = 3 * kEdge * OPS;
  l.t1 = l.f + 2 * 3 * l.fs;
  l.t2 = l.t1 + nw;
  const int most = (n - 4 + kBlock - 1) / kBlock * kBlock;
  auto rows = [&](int room, int ns) {
    int kc = (room / (ns * OPS * 5) - 4) / kBlock * kBlock;
    if (kc > most) kc = most;
    return kc < kBlock ? kBlock : kc;
  };
  l.kc_pt = rows(budget - l.t2, npt);
  l.kc_v = rows(budget - l.t1, 3);
  const int a = l.t2 + (two ? nw : 0), b = l.t2 + (l.kc_pt + 4) * npt * OPS * 5, c = l.t1 + (l.kc_v + 4) * 3 * OPS * 5;
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
// (last: the window's last row inside the column, for the transposed windows
// of single rows, which a short column does not fill)
template <int OPS, int RPT, int NF, int EXTRA = 8>
__device__ __forceinline__ void stencil(const double *w, const Cd *x, int fs, Cd (&acc)[NF][RPT],
                                        int last = 0) {
  constexpr int W = RPT + EXTRA;
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
    for (int f = 0; f < NF; ++f)
      v[e & 1][f] = x[f * fs + (EXTRA == 16 && e > last ? last : e) * 2 * OPS];
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

// Row of the matrix at sweep index i (indices past the last repeat it), and
// the lowest row of the indices [i rows, (i + 1) rows): a scalar base from
// which the lanes' rows are a 32-bit byte offset away.
template <bool DOWN>
__device__ __forceinline__ int lane_row(int i, int n) {
  i = i < n ? i : n - 1;
  return DOWN ? n - 1 - i : i;
}
template <bool DOWN>
__device__ __forceinline__ int first_row(int i, int rows, int n) {
  const int r = DOWN ? n - (i + 1) * rows : i * rows;
  return r < 0 ? 0 : (r < n ? r : n - 1);
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
  // repeat it).  The L rows (or, UP, the U rows with the inverse diagonals) in
  // sweep order: upwards, or DOWN from n - 1.
  template <bool UP, bool DOWN>
  __device__ __forceinline__ void load(int s, const Factors &F, int op0, int nlive, int n, int t) {
    {
      const int o = (t / 2) % OPS;
      const unsigned col = (unsigned)(o < nlive ? o : nlive - 1) * 32 + 16 * (t & 1);
      constexpr int RQ = kStageThreads / (2 * OPS);  // rows per register
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        const int r0 = first_row<DOWN>(i, RQ, n);
        const double *p = F.pk + (((size_t)r0 * 2 + (UP ? 1 : 0)) * F.nops + op0) * 4;
        q[s][i] = at<Dbl2>(p, (unsigned)(lane_row<DOWN>(t / (2 * OPS) + i * RQ, n) - r0) *
                                  ((unsigned)F.nops * 64) + col);
      }
    }
    if (UP) {
      constexpr int RD = kStageThreads / OPS;
      const int o = t % OPS;
      const unsigned col = (unsigned)(o < nlive ? o : nlive - 1) * 8;
#pragma unroll
      for (int i = 0; i < DQ; ++i) {
        const int r0 = first_row<DOWN>(i, RD, n);
        const double *p = F.di + (size_t)r0 * F.nops + op0;
        dg[s][i] = at<double>(p, (unsigned)(lane_row<DOWN>(t / OPS + i * RD, n) - r0) *
                                     ((unsigned)F.nops * 8) + col);
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
  // diagonals (UP) to D[row - r0][system][op]
  template <bool UP>
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
    if (UP) {
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
  double *E = base, *fld = base + lay.f, *T1 = base + lay.t1, *S = base + lay.t2;
  Cd *fA = reinterpret_cast<Cd *>(fld), *fB = fA + lay.fs, *fC = fB + lay.fs;
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
  L1.template load<false, false>(0, a.fp, opm, nlive, n, t);
  L1.load_edges(0, a.fp, opm, nlive, t);
  if constexpr (HEATED) {
    L1.template load<false, false>(NPT - 1, a.ft, opm, nlive, n, t);
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
  U1.template load<true, true>(0, a.fp, opm, nlive, n, t);
  if constexpr (HEATED) {
    U1.template load<true, true>(NPT - 1, a.ft, opm, nlive, n, t);
  }
  sweep_dir<false, OPS, NPT, RPT>(L1, fld, lay.fs, S, lay.kc_pt, E, n, t);
  sweep_dir<true, OPS, NPT, RPT>(U1, fld, lay.fs, S, lay.kc_pt, E, n, t);
  // ---- temperature out; velocity right sides f - grad p0 (the velocity L
  // rows on their way)
  FactorRegs<OPS, 3, RPT> L2;
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    L2.template load<false, false>(s, a.fv, op_v[s], nlive, n, t);
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
    U2.template load<true, true>(s, a.fv, op_v[s], nlive, n, t);
  }
  sweep_dir<false, OPS, 3, RPT>(L2, fld, lay.fs, T1, lay.kc_v, E, n, t);
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
  sweep_dir<true, OPS, 3, RPT>(U2, fld, lay.fs, T1, lay.kc_v, E, n, t);
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

// ---------------------------------------------------------------------------
// Vector--Jacobian product of the implicit stage in one kernel: the
// conjugate transposes of the steps above in reverse order (formulas at the
// kernel sequence in k_solve.hip), on the same tiles. What bounds it is what
// bounds k_stage, the serial sweeps (here in axpy form: the rows of the packed
// factors are the columns of their transposes, so no second copy of the factors
// is kept) between barriers. It replaces eight to ten launches that passed the
// fields through memory. Per call, sequence -> this kernel: 32x16x15 61 -> 24 us,
// 64x32x63 98 -> 49, 64x64x127 heated 211 -> 146, 128x64x127 653 -> 279,
// 128x64x127 heated 725 -> 368.
// ---------------------------------------------------------------------------

// Rows past RPT of the window that holds, for every column of a group of RPT
// rows, the rows whose nine-point windows contain it: nine inside, up to
// thirteen next to the one-sided wall windows, and up to all of them in
// columns of up to 18 points, where the two walls' windows overlap (taken
// with one row per thread there: stage_shape).
constexpr int win_extra_t(int rpt) { return rpt == 1 ? 16 : 12; }

// First row of that window for the group from j0 on.
template <int RPT>
__device__ __forceinline__ int win_base_t(int j0, int n) {
  const int hi = n - (RPT + win_extra_t(RPT));
  return clampi(j0 <= 8 ? 0 : j0 - 4, 0, hi > 0 ? hi : 0);
}

// Transposed weight table: dst[j][RPT + win_extra_t], entry e the weight of row
// base + e in column j.
template <int RPT>
__device__ __forceinline__ void fill_weights_t(double *dst, const double *__restrict__ w, int n, int t) {
  constexpr int W = RPT + win_extra_t(RPT);
  const int rows = (n + RPT - 1) / RPT * RPT;
  for (int i = t; i < rows * W; i += kStageThreads) {
    const int j = i / W, e = i - j * W;
    const int r = e + win_base_t<RPT>(j / RPT * RPT, n);
    const int tt = j - clampi(r - 4, 0, n - kStencil);
    dst[i] = j < n && r < n && tt >= 0 && tt < kStencil ? w[r * kStencil + tt] : 0.0;
  }
}

// Partial sums of the next four rows of a transposed recurrence.
struct CarryT {
  double s0, s1, s2, s3;
};

// A transposed recurrence, rows in sweep order: U^T y = b upwards (UP), L^T x
// = y downwards.  Row j's entries update the following rows as soon as its
// value is known (four independent multiply-adds), so the factors are read by
// rows here too; every row still takes its terms from the farthest to the
// nearest.
template <int OPS, bool UP, int NS>
struct RecurT {
  static constexpr int cs = UP ? 4 * OPS : -4 * OPS;
  static constexpr int qs = NS * 4 * OPS, ds = NS * OPS;
  // (b: the right side four rows on; past the last row it is never used)
  __device__ __forceinline__ static Row row(const double *c, const double *S, const double *D, int i) {
    Row r;
    r.qa = *reinterpret_cast<const Dbl2 *>(S + i * qs);
    r.qb = *reinterpret_cast<const Dbl2 *>(S + i * qs + 2);
    r.b = c[(i + 4) * cs];
    r.dg = UP ? D[i * ds] : 0.0;
    return r;
  }
  __device__ __forceinline__ static double e(const Row &r, int d) {
    return UP ? (d == 1 ? r.qa.x : d == 2 ? r.qa.y : d == 3 ? r.qb.x : r.qb.y)
              : (d == 1 ? r.qb.y : d == 2 ? r.qb.x : d == 3 ? r.qa.y : r.qa.x);
  }
  __device__ __forceinline__ static void step(const Row &r, CarryT &k, double *c) {
    const double y = UP ? k.s0 * r.dg : k.s0;
    k.s0 = fma(-e(r, 1), y, k.s1);
    k.s1 = fma(-e(r, 2), y, k.s2);
    k.s2 = fma(-e(r, 3), y, k.s3);
    k.s3 = fma(-e(r, 4), y, r.b);
    *c = y;
  }
  template <int LEN, int R>
  __device__ __forceinline__ static void rows(Row (&w)[R], CarryT &k, double *c, const double *S,
                                              const double *D, bool more) {
    static_assert(LEN % R == 0, "whole rings");
#pragma unroll
    for (int i = 0; i < LEN; ++i) {
      step(w[i % R], k, c + i * cs);
      if (i + R < LEN || more) w[i % R] = row(c, S, D, i + R);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // The first four rows, whose envelope entries (E, stride OPS) reach past
  // the band: row 0 + q (UP) to columns up to 8, row n-1-q down to n-9.
  __device__ __forceinline__ static CarryT head(double *c, const double *S, const double *D,
                                                const double *E) {
    Row w[4];
    double ed[10], b[9];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = row(c, S, D, i);
#pragma unroll
    for (int t = 0; t < 10; ++t) ed[t] = E[((UP ? 0 : 10) + t) * OPS];
#pragma unroll
    for (int i = 0; i < 9; ++i) b[i] = c[i * cs];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double y = UP ? b[q] * w[q].dg : b[q];
#pragma unroll
      for (int d = 1; d <= 4; ++d) b[q + d] = fma(-e(w[q], d), y, b[q + d]);
#pragma unroll
      for (int t = 0; t < 4 - q; ++t) {  // entry t: column q+5+t upwards, n-9+t downwards
        const int i = UP ? q + 5 + t : 8 - t;
        b[i] = fma(-ed[edge_off(q) + t], y, b[i]);
      }
      c[q * cs] = y;
    }
    c[8 * cs] = b[8];
    return CarryT{b[4], b[5], b[6], b[7]};
  }
};

// One direction of the transposed sweeps of NS systems (see sweep_dir).
template <bool UP, int OPS, int NS, int RPT>
__device__ __forceinline__ void sweep_dir_t(const FactorRegs<OPS, NS, RPT> &R, double *fld, int fs,
                                            double *S, int kc, const double *E, int n, int t) {
  using Q = RecurT<OPS, UP, NS>;
  constexpr int kCols = 4 * OPS;
  const int nb = n - 4;  // rows after the first four, which the first chunk brings along
  const int sys = t / kCols, col = t % kCols, o = (col >> 1) % OPS;
  const bool lane = t < NS * kCols;
  double *c0 = fld + (size_t)sys * 2 * fs + col + (UP ? 0 : (n - 1) * kCols);
  double *D = S + (kc + 4) * Q::qs;
  const double *Sl = S + sys * 4 * OPS + o * 4, *Dl = D + sys * OPS + o;
  const double *El = E + sys * kEdge * OPS + o;
  CarryT k{0.0, 0.0, 0.0, 0.0};
  for (int i0 = 0; i0 < nb; i0 += kc) {
    const int first = i0 == 0 ? 0 : i0 + 4;  // chunk's first row
    const int len = nb - i0 < kc ? nb - i0 : kc;
    R.template store_rows<UP>(S, D, first, i0 + 4 + len, t);
    __syncthreads();
    if (lane) {
      const double *Sc = Sl, *Dc = Dl;
      if (i0 == 0) {
        k = Q::head(c0, Sl, Dl, El);
        Sc += 4 * Q::qs;
        Dc += 4 * Q::ds;
      }
      double *c = c0 + (i0 + 4) * Q::cs;
      int i = 0;
      if (len >= kBlock) {
        Row w[kRing];
#pragma unroll
        for (int r = 0; r < kRing; ++r) w[r] = Q::row(c, Sc, Dc, r);
        __builtin_amdgcn_sched_barrier(0);
        for (; i + kBlock <= len; i += kBlock)
          Q::template rows<kBlock>(w, k, c + i * Q::cs, Sc + i * Q::qs, Dc + i * Q::ds,
                                   i + 2 * kBlock <= len);
      }
      for (; i + 4 <= len; i += 4) {
        Row w[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] = Q::row(c + i * Q::cs, Sc + i * Q::qs, Dc + i * Q::ds, r);
        Q::template rows<4>(w, k, c + i * Q::cs, Sc + i * Q::qs, Dc + i * Q::ds, false);
      }
      for (; i < len; ++i) {
        const Row w = Q::row(c + i * Q::cs, Sc + i * Q::qs, Dc + i * Q::ds, 0);
        Q::step(w, k, c + i * Q::cs);
      }
    }
    __syncthreads();
  }
}

struct StageAdjArgs {
  Factors fp, fv, ft;
  Influence inf;
  const double2 *ub;            // output adjoint
  double2 *ubn, *nbn, *nbq;     // input adjoints (nbq null: its part is added to nbn)
  double idt, cc;
  int overwrite;                // bit 1 ubn, 2 nbn, 4 nbq written instead of accumulated
};

template <int OPS, int RPT, bool HEATED>
__global__ void __launch_bounds__(kStageThreads, 2) k_stage_adj(Dims d, Grid g, StageAdjArgs a, StageLds lay) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int X = win_extra_t(RPT), W = RPT + X;
  constexpr int kModes = 2 * OPS;
  constexpr int NPT = HEATED ? 2 : 1;
  const int n = d.nr, K = d.kmax, kp1 = K + 1;
  double *base = reinterpret_cast<double *>(smem);
  double *E = base, *fld = base + lay.f, *T1 = base + lay.t1, *S = base + lay.t2;
  Cd *fA = reinterpret_cast<Cd *>(fld), *fB = fA + lay.fs, *fC = fB + lay.fs;
  const int t = threadIdx.x;
  const int kt = (kp1 + OPS - 1) / OPS;
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  const int m = L / kt, ka0 = (L - m * kt) * OPS;
  const int nlive = kp1 - ka0 < OPS ? kp1 - ka0 : OPS;
  const int ml = t % kModes, rg = t / kModes;
  const int o = ml % OPS, sg = ml / OPS;
  const int ka = ka0 + (o < nlive ? o : nlive - 1);
  const int kk = sg ? K - ka : K + ka;
  const bool live = o < nlive && !(sg && ka == 0);
  const bool zero = m == 0 && ka == 0;
  const int md = m * d.mz + kk;
  const size_t fst = (size_t)n * d.nmodes;
  const double kap = (double)(kk - K) * d.kz;
  const double k2 = kap * kap, mm = (double)m;
  const double ce = 1.0 - a.cc;
  const int j0 = rg * RPT;
  const int wb = win_base_t<RPT>(j0 < n ? j0 : n - 1, n);
  const Cd *win = fA + wb * kModes + ml;
  const int jw = j0 < n ? j0 : 0;
  auto rowc = [&](int jj) { return j0 + jj < n ? j0 + jj : n - 1; };
  auto ok = [&](int jj) { return j0 + jj < n; };
  auto inner = [&](int j) { return j > 0 && j < n - 1; };
  const unsigned row16 = (unsigned)d.nmodes * 16, md16 = (unsigned)md * 16;
  auto off = [&](int jj) { return (unsigned)rowc(jj) * row16 + md16; };
  const int opm = m * kp1 + ka0, opi = m * kp1 + ka;
  const int op_v[3] = {(m + 1) * kp1 + ka0, (m >= 1 ? m - 1 : 1) * kp1 + ka0, opm};
  // ---- output adjoint: m = 0 Hermitian, +- basis (mode (0,0): u_theta in
  // the first slot)
  Cd xp[RPT], xm[RPT], xz[RPT];
#pragma unroll
  for (int jj = 0; jj < RPT; ++jj) {
    xp[jj] = ldc(a.ub, off(jj));
    xm[jj] = ldc(a.ub + fst, off(jj));
    xz[jj] = ldc(a.ub + 2 * fst, off(jj));
  }
  // ---- lambda_bar_w = sum_j (X_w+ Xbar+ + X_w- Xbar- + i kappa h_w Xbar_z)
  Cd l1 = {0.0, 0.0}, l2 = {0.0, 0.0};
#pragma unroll
  for (int jj = 0; jj < RPT; ++jj) {
    if (m == 0) {
      xp[jj] = herm_pair<OPS>(xp[jj]);
      xm[jj] = herm_pair<OPS>(xm[jj]);
      xz[jj] = herm_pair<OPS>(xz[jj]);
    }
    const Cd r = xp[jj], th = xm[jj];
    const Cd p = 0.5 * (r + ci(th)), q = 0.5 * (r - ci(th));
    xp[jj] = Cd{zero ? th.x : p.x, zero ? th.y : p.y};
    xm[jj] = Cd{zero ? 0.0 : q.x, zero ? 0.0 : q.y};
    auto R = [&](int kind) {
      return at<Dbl2>(a.inf.resp + (size_t)kind * n * a.inf.nops,
                      ((unsigned)rowc(jj) * (unsigned)a.inf.nops + (unsigned)opi) * 16);
    };
    const Dbl2 r1 = R(1), r2 = R(2), r3 = R(3);
    const Cd iz = kap * ci(xz[jj]);
    const double on = ok(jj) ? 1.0 : 0.0;
    l1 = l1 + on * (r1.x * xp[jj] + r2.x * xm[jj] + r3.x * iz);
    l2 = l2 + on * (r1.y * xp[jj] + r2.y * xm[jj] + r3.y * iz);
  }
  FactorRegs<OPS, 3, RPT> U2;
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    U2.template load<true, false>(s, a.fv, op_v[s], nlive, n, t);
    U2.load_edges(s, a.fv, op_v[s], nlive, t);
  }
  // over the row groups of a wavefront, then over the four wavefronts
#pragma unroll
  for (int msk = kModes; msk < 64; msk *= 2) {
    l1 = l1 + Cd{xor_lane(l1.x, msk), xor_lane(l1.y, msk)};
    l2 = l2 + Cd{xor_lane(l2.x, msk), xor_lane(l2.y, msk)};
  }
  Cd *red = reinterpret_cast<Cd *>(S);
  if ((t & 63) < kModes) {
    red[(t >> 6) * 2 * kModes + ml] = l1;
    red[((t >> 6) * 2 + 1) * kModes + ml] = l2;
  }
  U2.store_edges(E, t);
  __syncthreads();
  l1 = red[ml];
  l2 = red[kModes + ml];
#pragma unroll
  for (int w = 1; w < kStageThreads / 64; ++w) {
    l1 = l1 + red[2 * w * kModes + ml];
    l2 = l2 + red[(2 * w + 1) * kModes + ml];
  }
  // ---- right sides of the transposed Helmholtz problems: Xbar + the wall
  // divergences' transposes times beta_bar = -A^-T lambda_bar
  {
    const size_t ns = a.inf.nops;
    const double a00 = a.inf.ainv[opi], a01 = a.inf.ainv[ns + opi], a10 = a.inf.ainv[2 * ns + opi],
                 a11 = a.inf.ainv[3 * ns + opi];
    const double on = zero ? 0.0 : 1.0;
    const Cd b0 = on * Cd{-(a00 * l1.x + a10 * l2.x), -(a00 * l1.y + a10 * l2.y)};
    const Cd b1 = on * Cd{-(a01 * l1.x + a11 * l2.x), -(a01 * l1.y + a11 * l2.y)};
    const double ri0 = g.rinv[0], ri1 = g.rinv[n - 1];
#pragma unroll
    for (int jj = 0; jj < RPT; ++jj) {
      const int j = rowc(jj);
      const double c0 = j <= 8 ? g.d1[j] : 0.0;
      const double c1 = j >= n - 9 ? g.d1[(n - 1) * kStencil + (j - (n - 9))] : 0.0;
      const double e0 = j == 0 ? ri0 : 0.0, e1 = j == n - 1 ? ri1 : 0.0;
      const double z0 = j == 0 ? kap : 0.0, z1 = j == n - 1 ? kap : 0.0;
      const Cd vp = xp[jj] + (0.5 * (c0 + (1.0 + mm) * e0)) * b0 + (0.5 * (c1 + (1.0 + mm) * e1)) * b1;
      const Cd vm = xm[jj] + (0.5 * (c0 + (1.0 - mm) * e0)) * b0 + (0.5 * (c1 + (1.0 - mm) * e1)) * b1;
      const Cd vz = xz[jj] - z0 * ci(b0) - z1 * ci(b1);
      if (ok(jj)) {
        const int pos = j * kModes + ml;
        fA[pos] = vp;
        fB[pos] = vm;
        fC[pos] = vz;
      }
    }
  }
  __syncthreads();  // (the partial sums in S are read)
  // ---- transposed velocity sweeps; their L rows on their way
  FactorRegs<OPS, 3, RPT> L2;
#pragma unroll
  for (int s = 0; s < 3; ++s) L2.template load<false, true>(s, a.fv, op_v[s], nlive, n, t);
  sweep_dir_t<true, OPS, 3, RPT>(U2, fld, lay.fs, T1, lay.kc_v, E, n, t);
  FactorRegs<OPS, NPT, RPT> U1;
  U1.template load<true, false>(0, a.fp, opm, nlive, n, t);
  U1.load_edges(0, a.fp, opm, nlive, t);
  if constexpr (HEATED) {
    U1.template load<true, false>(NPT - 1, a.ft, opm, nlive, n, t);
    U1.load_edges(NPT - 1, a.ft, opm, nlive, t);
  }
  sweep_dir_t<false, OPS, 3, RPT>(L2, fld, lay.fs, T1, lay.kc_v, E, n, t);
  // ---- wall rows masked; mode (0,0): fbar+- = +-(i/2) rbar_theta
  Cd rp[RPT], rm[RPT];
#pragma unroll
  for (int jj = 0; jj < RPT; ++jj) {
    const int j = rowc(jj), pos = j * kModes + ml;
    const Cd h = 0.5 * ci(fA[pos]);
    Cd vp = fA[pos], vm = fB[pos], vz = fC[pos];
    vp = Cd{zero ? h.x : vp.x, zero ? h.y : vp.y};
    vm = Cd{zero ? -h.x : vm.x, zero ? -h.y : vm.y};
    rp[jj] = Cd{inner(j) ? vp.x : 0.0, inner(j) ? vp.y : 0.0};
    rm[jj] = Cd{inner(j) ? vm.x : 0.0, inner(j) ? vm.y : 0.0};
    vz = Cd{inner(j) ? vz.x : 0.0, inner(j) ? vz.y : 0.0};
    if (ok(jj)) {  // (this thread's own entries)
      fA[pos] = rp[jj];
      fB[pos] = rm[jj];
      fC[pos] = vz;
    }
  }
  fill_weights_t<RPT>(T1, g.d1, n, t);
  U1.store_edges(E, t);
  __syncthreads();
  // ---- pbar0 = -D1^T (rbar+ + rbar-) + (m/r)(rbar+ - rbar-) + i kappa rbar_z
  Cd tT[RPT];
  {
    Cd dv[2][RPT];
    if constexpr (HEATED)
#pragma unroll
      for (int jj = 0; jj < RPT; ++jj) tT[jj] = ldc(a.ub + 3 * fst, off(jj));
    stencil<OPS, RPT, 2, X>(T1 + jw * W, win, lay.fs, dv, n - 1 - wb);
    __syncthreads();
#pragma unroll
    for (int jj = 0; jj < RPT; ++jj) {
      const int j = rowc(jj), pos = j * kModes + ml;
      Cd pb = ((mm * g.rinv[j]) * (rp[jj] - rm[jj])) - (dv[0][jj] + dv[1][jj]) + kap * ci(fC[pos]);
      pb = Cd{zero ? 0.0 : pb.x, zero ? 0.0 : pb.y};
      if (HEATED && m == 0) tT[jj] = herm_pair<OPS>(tT[jj]);
      if (ok(jj)) {
        fA[pos] = pb;
        if (HEATED) fB[pos] = tT[jj];
      }
    }
  }
  // ---- transposed pressure and temperature sweeps
  FactorRegs<OPS, NPT, RPT> L1;
  L1.template load<false, true>(0, a.fp, opm, nlive, n, t);
  if constexpr (HEATED) L1.template load<false, true>(NPT - 1, a.ft, opm, nlive, n, t);
  sweep_dir_t<true, OPS, NPT, RPT>(U1, fld, lay.fs, S, lay.kc_pt, E, n, t);
  sweep_dir_t<false, OPS, NPT, RPT>(L1, fld, lay.fs, S, lay.kc_pt, E, n, t);
  // ---- gbar and the temperature masked; fbar+- = rbar+- + (D1^T gbar +
  // (1 +- m) gbar / r) / 2, fbar_z = rbar_z - i kappa gbar
  Cd fz[RPT];
#pragma unroll
  for (int jj = 0; jj < RPT; ++jj) {
    const int j = rowc(jj), pos = j * kModes + ml;
    const bool keep = inner(j) && !zero;
    if (ok(jj)) fA[pos] = Cd{keep ? fA[pos].x : 0.0, keep ? fA[pos].y : 0.0};
    if constexpr (HEATED) tT[jj] = Cd{inner(j) ? fB[pos].x : 0.0, inner(j) ? fB[pos].y : 0.0};
  }
  __syncthreads();
  {
    Cd dg[1][RPT];
    stencil<OPS, RPT, 1, X>(T1 + jw * W, win, lay.fs, dg, n - 1 - wb);
#pragma unroll
    for (int jj = 0; jj < RPT; ++jj) {
      const int j = rowc(jj), pos = j * kModes + ml;
      const double ri = g.rinv[j];
      const Cd gv = fA[pos];
      rp[jj] = rp[jj] + 0.5 * (dg[0][jj] + ((1.0 + mm) * ri) * gv);
      rm[jj] = rm[jj] + 0.5 * (dg[0][jj] + ((1.0 - mm) * ri) * gv);
      fz[jj] = fC[pos] - kap * ci(gv);
    }
  }
  __syncthreads();
#pragma unroll
  for (int jj = 0; jj < RPT; ++jj)
    if (ok(jj)) {
      const int pos = (j0 + jj) * kModes + ml;
      fA[pos] = rp[jj];
      fB[pos] = rm[jj];
      fC[pos] = fz[jj];
    }
  fill_weights_t<RPT>(T1, g.lw, n, t);
  __syncthreads();
  // ---- input adjoints: Xbar^n = fbar/dt + (1-c) L^T fbar, Nbar^q = c fbar,
  // Nbar^n = (1-c) fbar, back to (r, theta, z, T)
  auto put = [&](double2 *p, int jj, Cd v, int bit) {
    if (!(live && ok(jj))) return;
    if (!(a.overwrite & bit)) v = ldc(p, off(jj)) + v;
    stc(p, off(jj), v);
  };
  auto put_n = [&](int f, int jj, Cd v) {
    if (a.nbq) {
      put(a.nbn + f * fst, jj, ce * v, 2);
      put(a.nbq + f * fst, jj, a.cc * v, 4);
    } else if (live && ok(jj)) {  // N^n and N^q are the same array
      double2 *p = a.nbn + f * fst;
      const Cd old = a.overwrite & 2 ? Cd{0.0, 0.0} : ldc(p, off(jj));
      stc(p, off(jj), (old + ce * v) + a.cc * v);
    }
  };
  {
    Cd l[2][RPT];
    stencil<OPS, RPT, 2, X>(T1 + jw * W, win, lay.fs, l, n - 1 - wb);
    const double qp = mm + 1.0, qm = m >= 1 ? mm - 1.0 : 1.0;
#pragma unroll
    for (int jj = 0; jj < RPT; ++jj) {
      const double ri = g.rinv[rowc(jj)], r2 = ri * ri;
      const Cd x0 = a.idt * rp[jj] + ce * (l[0][jj] - (qp * qp * r2 + k2) * rp[jj]);
      const Cd x1 = a.idt * rm[jj] + ce * (l[1][jj] - (qm * qm * r2 + k2) * rm[jj]);
      // X+- = X_r +- i X_theta => Xbar_r = Xbar+ + Xbar-, Xbar_theta = -i (Xbar+ - Xbar-)
      const Cd dx = x0 - x1, df = rp[jj] - rm[jj];
      put(a.ubn, jj, x0 + x1, 1);
      put(a.ubn + fst, jj, Cd{dx.y, -dx.x}, 1);
      put_n(0, jj, rp[jj] + rm[jj]);
      put_n(1, jj, Cd{df.y, -df.x});
    }
  }
  {
    Cd l[1][RPT];
    stencil<OPS, RPT, 1, X>(T1 + jw * W, win + 2 * lay.fs, lay.fs, l, n - 1 - wb);
#pragma unroll
    for (int jj = 0; jj < RPT; ++jj) {
      const double ri = g.rinv[rowc(jj)], r2 = ri * ri;
      put(a.ubn + 2 * fst, jj, a.idt * fz[jj] + ce * (l[0][jj] - (mm * mm * r2 + k2) * fz[jj]), 1);
      put_n(2, jj, fz[jj]);
    }
  }
  if constexpr (HEATED) {
    __syncthreads();
#pragma unroll
    for (int jj = 0; jj < RPT; ++jj)
      if (ok(jj)) fA[(j0 + jj) * kModes + ml] = tT[jj];
    __syncthreads();
    Cd l[1][RPT];
    stencil<OPS, RPT, 1, X>(T1 + jw * W, win, lay.fs, l, n - 1 - wb);
#pragma unroll
    for (int jj = 0; jj < RPT; ++jj) {
      const double ri = g.rinv[rowc(jj)], r2 = ri * ri;
      put(a.ubn + 3 * fst, jj,
          a.idt * tT[jj] + (ce / d.pr) * (l[0][jj] - (mm * mm * r2 + k2) * tT[jj]), 1);
      put_n(3, jj, tT[jj]);
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
StageShape shape_for(const nsc_ctx *c, bool adjoint) {
  const int groups = kStageThreads / (2 * OPS), n = c->d.nr;
  const int rpt = (n + groups - 1) / groups, npt = c->d.heated ? 2 : 1;
  return StageShape{OPS, rpt, stage_lds<OPS>(n, rpt, npt, adjoint ? win_extra_t(rpt) : 8, !adjoint, c->lds_cu / 2 / 8)};
}

// Eight |k| per workgroup (whole 128-byte lines of sixteen modes, half the
// workgroups) once that leaves a workgroup per compute unit; four otherwise,
// past 64 points, where a thread would hold more than four rows, and for the
// adjoint at 17 and 18 points, where a pair of rows has every row of the column
// in its transposed windows.  us with four / eight |k|, isothermal:
//                        stage          adjoint
//   48 x 40 x 79  (200 tiles of eight)  22.8 / 23.0    33.4 / 35.7
//   48 x 45 x 89  (270)                 37.8 / 30.4    54.8 / 44.1
//   48 x 64 x 127 (512)                 43.9 / 34.0    63.8 / 48.1
//   64 x 40 x 79  (200)                 27.5 / 32.1    38.9 / 56.6
//   64 x 64 x 127 (512)                 53.6 / 46.2    76.2 / 78.8
// On 32 points the two meet at the line (16.4 / 16.3 at 200 tiles, 20.0 / 21.1
// at 270), on 16 a little below it.  From 49 points on, four rows per thread
// spill with the temperature (79 registers; 11 without) and in the adjoint (92 and
// 56): there the line is not the best one (64 x 64 x 127 heated 60.3 / 71.0,
// adjoint 86.1 / 110.7).
StageShape stage_shape(const nsc_ctx *c, bool adjoint) {
  const int n = c->d.nr;
  const long tiles = (long)c->d.mt * ((c->d.kmax + 8) / 8);
  return n <= 64 && !(adjoint && (n == 17 || n == 18)) && tiles >= c->cu_count ? shape_for<8>(c, adjoint) : shape_for<4>(c, adjoint);
}

// f(ops, rows) with the shape's |k| count and rows per thread as constants
template <class F>
hipError_t with_shape(const StageShape &sh, F f) {
  auto rows = [&](auto ops) {
    switch (sh.rpt) {
      case 1: return f(ops, std::integral_constant<int, 1>{});
      case 2: return f(ops, std::integral_constant<int, 2>{});
      case 3: return f(ops, std::integral_constant<int, 3>{});
      default: return f(ops, std::integral_constant<int, 4>{});
    }
  };
  return sh.ops == 8 ? rows(std::integral_constant<int, 8>{}) : rows(std::integral_constant<int, 4>{});
}

}  // namespace

bool stage_fused(const nsc_ctx *c) {
  const Dims &d = c->d;
  if (d.nr > kStageRows) return false;
  // 32-bit byte offsets of the fields and responses (always within reach up
  // to 64 radial points: the transform lengths bound the modes to 3.8 million)
  if ((size_t)d.nr * d.nmodes * 16 >> 32) return false;
  return (size_t)stage_shape(c, false).lds.total * sizeof(double) <= (size_t)c->lds_max;
}

bool stage_adj_fused(const nsc_ctx *c) {
  return stage_fused(c) && (size_t)stage_shape(c, true).lds.total * sizeof(double) <= (size_t)c->lds_max;
}

hipError_t launch_stage(const nsc_ctx *c, const double *u, const double *nn, const double *nq,
                        double *out, double *pout, double dt, double cc, int walls) {
  const Dims &d = c->d;
  StageArgs a{c->fp, c->fv, c->ft, c->inf, reinterpret_cast<const double2 *>(u),
              reinterpret_cast<const double2 *>(nn ? nn : u),
              reinterpret_cast<const double2 *>(nn ? nq : u), reinterpret_cast<double2 *>(out),
              reinterpret_cast<double2 *>(pout), 1.0 / dt, cc, nn ? cc : 0.0, nn ? 1.0 - cc : 0.0,
              walls, pout && nn ? 1 : 0};
  const StageShape sh = stage_shape(c, false);
  const int kt = (d.kmax + sh.ops) / sh.ops;
  return with_shape(sh, [&](auto ops, auto rows) {
    constexpr int OPS = decltype(ops)::value, RPT = decltype(rows)::value;
    auto kern = d.pipe ? (pout ? k_stage<OPS, RPT, false, true, true> : k_stage<OPS, RPT, false, true, false>)
              : d.heated ? (pout ? k_stage<OPS, RPT, true, false, true> : k_stage<OPS, RPT, true, false, false>)
                         : (pout ? k_stage<OPS, RPT, false, false, true> : k_stage<OPS, RPT, false, false, false>);
    hipLaunchKernelGGL(kern, dim3(d.mt * kt), dim3(kStageThreads),
                       (size_t)sh.lds.total * sizeof(double), c->stream, d, c->g, a, sh.lds);
    return hipGetLastError();
  });
}

hipError_t launch_stage_adj(const nsc_ctx *c, const double *ubar_out, double *ubar_n, double *nbar_n,
                            double *nbar_q, double dt, double cc, int overwrite) {
  const Dims &d = c->d;
  StageAdjArgs a{c->fp, c->fv, c->ft, c->inf, reinterpret_cast<const double2 *>(ubar_out),
                 reinterpret_cast<double2 *>(ubar_n), reinterpret_cast<double2 *>(nbar_n),
                 reinterpret_cast<double2 *>(nbar_q), 1.0 / dt, cc, overwrite};
  const StageShape sh = stage_shape(c, true);
  const int kt = (d.kmax + sh.ops) / sh.ops;
  return with_shape(sh, [&](auto ops, auto rows) {
    constexpr int OPS = decltype(ops)::value, RPT = decltype(rows)::value;
    auto kern = d.heated ? k_stage_adj<OPS, RPT, true> : k_stage_adj<OPS, RPT, false>;
    hipLaunchKernelGGL(kern, dim3(d.mt * kt), dim3(kStageThreads),
                       (size_t)sh.lds.total * sizeof(double), c->stream, d, c->g, a, sh.lds);
    return hipGetLastError();
  });
}

}  // namespace nsc
