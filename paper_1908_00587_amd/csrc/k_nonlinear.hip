// Dispatch of the pseudospectral nonlinear term and its adjoint (kernels in
// nl_kernels.h): compile-time transform lengths where nl_lengths.h has them,
// the runtime-length passes otherwise.
#include "nl_kernels.h"

namespace nsc {
namespace {

// ubar += D(u)^T dbar (transposes of the spectral curl/gradient) + buoyancy.
// (WRITE: ubar = instead of +=; tables: the transposed rows of D1)
// On the smaller grids its time is the latency of the stencil's loads: nine are
// requested together (a loop over the rows 7.8 and 7.1 us on 32 x 16 x 31 modes and
// 9.8 and 8.6 on 64 x 32 x 63 adding and writing, now 5.2, 5.0, 8.2 and 7.0).
template <bool WRITE>
__global__ void __launch_bounds__(256)
k_derived_adj(Dims d, Grid g, const int *__restrict__ trow, const int *__restrict__ tcnt,
              const double *__restrict__ twd, const double2 *__restrict__ db,
              const double2 *__restrict__ nb, double2 *__restrict__ ub) {
  const int md = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y;
  if (md >= d.nmodes) return;
  const size_t P = d.nmodes;
  const int n = d.nr;
  const int m = md / d.mz;
  const int kk = md - m * d.mz;
  const double kap = (double)(kk - d.kmax) * d.kz;
  const double ri = g.rinv[j];
  const double mr = (double)m * ri;
  auto D = [&](int f) { return db[((size_t)f * n + j) * P + md]; };
  // (D1^T v)_j over the rows whose window holds j (uniform per workgroup)
  const int cnt = tcnt[j];
  auto D1T = [&](int f) {
    double2 acc = make_double2(0.0, 0.0), v9[kStencil];
    // (past the last row: that row again, with weight zero)
#pragma unroll
    for (int e = 0; e < kStencil; ++e)
      v9[e] = db[((size_t)f * n + trow[j * kTrans + (e < cnt ? e : cnt - 1)]) * P + md];
#pragma unroll
    for (int e = 0; e < kStencil; ++e) {
      const double w = e < cnt ? twd[j * kTrans + e] : 0.0;
      acc.x = fma(w, v9[e].x, acc.x);
      acc.y = fma(w, v9[e].y, acc.y);
    }
    for (int e = kStencil; e < cnt; ++e) {
      const double w = twd[j * kTrans + e];
      const double2 v = db[((size_t)f * n + trow[j * kTrans + e]) * P + md];
      acc.x = fma(w, v.x, acc.x);
      acc.y = fma(w, v.y, acc.y);
    }
    return acc;
  };
  auto mul_i = [](double s, double2 v) { return make_double2(-s * v.y, s * v.x); };  // i s v
  auto add = [&](int f, double2 v) {
    double2 *p = ub + ((size_t)f * n + j) * P + md;
    if (WRITE) {
      *p = v;
    } else {
      p->x += v.x;
      p->y += v.y;
    }
  };
  const double2 d0 = D(0), d1 = D(1), d2 = D(2), d3 = D(3), d4 = D(4), d5 = D(5);
  const double2 a4 = mul_i(-kap, d4), a5 = mul_i(mr, d5);
  add(0, make_double2(d0.x + a4.x + a5.x, d0.y + a4.y + a5.y));
  const double2 b3 = mul_i(kap, d3), t5 = D1T(5);
  add(1, make_double2(d1.x + b3.x + t5.x + ri * d5.x, d1.y + b3.y + t5.y + ri * d5.y));
  const double2 c3 = mul_i(-mr, d3), t4 = D1T(4);
  add(2, make_double2(d2.x + c3.x - t4.x, d2.y + c3.y - t4.y));
  if (d.heated) {
    const double2 t6 = D1T(6), e7 = mul_i(-mr, D(7)), e8 = mul_i(-kap, D(8));
    auto NB = [&](int fo) {
      double2 a = nb[((size_t)fo * n + j) * P + md];
      if (md < d.mz) {
        const double2 w = nb[((size_t)fo * n + j) * P + (d.mz - 1 - md)];
        a = make_double2(0.5 * (a.x + w.x), 0.5 * (a.y - w.y));
      }
      return a;
    };
    const double2 nz = NB(2);
    add(3, make_double2(t6.x + e7.x + e8.x + d.gr * nz.x, t6.y + e7.y + e8.y + d.gr * nz.y));
  }
}

// Theta-pass launch shape: wavefront-scope sets when a wavefront can carry
// at least two lines per stage and a set's lines fit a modest LDS share,
// else one set per workgroup.
struct ThetaLaunch {
  bool wave;
  int waves;      // sets per workgroup (wave mode)
  dim3 grid;
  int threads;
  size_t shm;
};

ThetaLaunch theta_launch(const nsc_ctx *c, int nlines, size_t esize, bool one_line = false) {
  ThetaLaunch L;
  const size_t line = (size_t)line_len(c->d.nt, esize) * esize;
  const size_t tws = (size_t)c->d.nt * 16;  // 16-byte twiddle entries in both precisions
  const int nsets = c->d.nz * c->d.nr;
  // wavefront scope: lines that fit a wavefront's registers two at a time
  // and a line set of at most 24 KB; one_line: also one line at a time and
  // any line set the LDS holds (768-point lines: measured faster than the
  // workgroup-scope stages)
  L.wave = one_line ? (c->plan_t.wave_lines >= 1 && (size_t)nlines * line + tws <= (size_t)c->lds_max)
                    : (c->plan_t.wave_lines >= 2 && (size_t)nlines * line <= 24 * 1024);
  if (L.wave) {
    int w = (int)(((size_t)c->lds_max - tws) / ((size_t)nlines * line));
    if (w > 4) w = 4;
    if (w < 1) w = 1;
    L.waves = w;
    L.grid = dim3((nsets + w - 1) / w);
    L.threads = 64 * w;
    L.shm = tws + (size_t)w * nlines * line;
  } else {
    L.waves = 1;
    L.grid = dim3(c->d.nz, c->d.nr);
    L.threads = block_for(c->plan_t, nlines, 256);
    L.shm = tws + (size_t)nlines * line;
  }
  return L;
}


template <typename T>
LenOps len_ops(int n) {
  constexpr bool F32 = sizeof(T) == 4;
  switch (n) {
#define NSC_LEN_CASE(N) case N: return F32 ? len32_##N() : len64_##N();
    NSC_LENGTHS(NSC_LEN_CASE)
#undef NSC_LEN_CASE
    case 1536: return F32 ? len32_1536() : LenOps{};
    default: return LenOps{};
  }
}

// the z passes of the context's z length
template <typename T>
LenOps z_ops(const nsc_ctx *c) {
  const LenOps o = len_ops<T>(c->d.nz);
  return o.zinv ? o : LenPass<T, 0>::z_ops();
}

template <typename T>
hipError_t theta_any(const nsc_ctx *c, int want_cfl) {
  if (const LenOps o = len_ops<T>(c->d.nt); o.theta) return o.theta(c, want_cfl);
  const ThetaLaunch L = theta_launch(c, (c->n_in + 1) / 2, sizeof(C2<T>), true);
  auto kern = L.wave ? k_theta<T, true> : k_theta<T, false>;
  hipLaunchKernelGGL(kern, L.grid, dim3(L.threads), L.shm, c->stream, c->d, c->g, c->plan_t,
                     reinterpret_cast<const C2<T> *>(c->zbuf), reinterpret_cast<C2<T> *>(c->wbuf),
                     tw_t<T>(c), c->n_in, 2.0 * M_PI / c->d.nt, c->d.lz / c->d.nz, c->cfl_part,
                     want_cfl, c->s_mean);
  return hipGetLastError();
}

template <typename T>
hipError_t theta_adj_any(const nsc_ctx *c) {
  if (const LenOps o = len_ops<T>(c->d.nt); o.theta_adj) return o.theta_adj(c);
  const ThetaLaunch L = theta_launch(c, (c->n_in + 1) / 2 + 2, sizeof(C2<T>));
  auto kern = L.wave ? k_theta_adj<T, true> : k_theta_adj<T, false>;
  hipLaunchKernelGGL(kern, L.grid, dim3(L.threads), L.shm, c->stream, c->d, c->plan_t,
                     reinterpret_cast<C2<T> *>(c->zbuf), reinterpret_cast<const C2<T> *>(c->wbuf),
                     tw_t<T>(c), c->n_in, c->n_out);
  return hipGetLastError();
}

template <typename T>
hipError_t nonlinear_vjp_impl(const nsc_ctx *c, const double *u, const double *nbar, double *ubar,
                              int overwrite) {
  const LenOps o = z_ops<T>(c);
  // forward fields and output adjoints on the (r, theta-spectral, z-physical)
  // grid, pointwise adjoint, input adjoints back
  hipError_t e = o.zinv(c, u, 0);
  if (e == hipSuccess) e = o.zinv_adj(c, nbar);
  if (e == hipSuccess) e = theta_adj_any<T>(c);
  if (e == hipSuccess) e = o.zfwd_adj(c);
  if (e != hipSuccess) return e;
  auto kern = overwrite ? k_derived_adj<true> : k_derived_adj<false>;
  hipLaunchKernelGGL(kern, dim3((c->d.nmodes + 255) / 256, c->d.nr), dim3(256), 0, c->stream,
                     c->d, c->g, c->t_row, c->t_cnt, c->t_wd, reinterpret_cast<const double2 *>(c->s_adj),
                     reinterpret_cast<const double2 *>(nbar), reinterpret_cast<double2 *>(ubar));
  return hipGetLastError();
}

template <typename T>
bool theta_fits_impl(const nsc_ctx *c, int adjoint) {
  if (const LenOps o = len_ops<T>(c->d.nt); o.theta_sets) return o.theta_sets(c, adjoint) > 0;
  const int npi = (c->n_in + 1) / 2;
  return theta_launch(c, adjoint ? npi + 2 : npi, sizeof(C2<T>), !adjoint).shm <= (size_t)c->lds_max;
}

}  // namespace

hipError_t launch_zinv(const nsc_ctx *c, int prec, const double *u) {
  return (prec == NSC_MIXED ? z_ops<float>(c) : z_ops<double>(c)).zinv(c, u, 1);
}

bool theta_fits(const nsc_ctx *c, int prec, int adjoint) {
  return prec == NSC_MIXED ? theta_fits_impl<float>(c, adjoint) : theta_fits_impl<double>(c, adjoint);
}

hipError_t launch_theta(const nsc_ctx *c, int prec, int want_cfl) {
  return prec == NSC_MIXED ? theta_any<float>(c, want_cfl) : theta_any<double>(c, want_cfl);
}

hipError_t launch_zfwd(const nsc_ctx *c, int prec, const double *u, double *n_hat, double *cfl_out,
                       double *cfl_host) {
  return (prec == NSC_MIXED ? z_ops<float>(c) : z_ops<double>(c)).zfwd(c, u, n_hat, cfl_out, cfl_host);
}

hipError_t launch_nonlinear_vjp(const nsc_ctx *c, int prec, const double *u, const double *nbar,
                                double *ubar, int overwrite) {
  if (prec == NSC_MIXED) return nonlinear_vjp_impl<float>(c, u, nbar, ubar, overwrite);
  return nonlinear_vjp_impl<double>(c, u, nbar, ubar, overwrite);
}

}  // namespace nsc
