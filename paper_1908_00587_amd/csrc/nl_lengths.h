// Transform lengths with compile-time kernels: every multiple of 12 with no
// prime factor above 5 up to 768 (three times a multiple of four modes), in
// both precisions, and 1536 in FP32.  Other lengths run the runtime-length
// stages, about half as fast (theta pass of FP64 384-point lines 990 against
// 370 us, of 120-point lines 46 against 27 us).
#pragma once
#include "nsc_internal.h"

namespace nsc {

struct LenOps {  // (all null: no compile-time kernels)
  hipError_t (*zinv)(const nsc_ctx *, const double *u, int drop_mean);
  hipError_t (*zfwd)(const nsc_ctx *, const double *u, double *nh, double *cfl_out, double *cfl_host);
  hipError_t (*zinv_adj)(const nsc_ctx *, const double *nbar);
  hipError_t (*zfwd_adj)(const nsc_ctx *);
  hipError_t (*theta)(const nsc_ctx *, int want_cfl);
  hipError_t (*theta_adj)(const nsc_ctx *);
  int (*theta_sets)(const nsc_ctx *, int adjoint);  // line sets per workgroup, 0: none fits
};

// (one line per file of instantiations, k_len1.hip ...)
#define NSC_LENGTHS(X)                \
  X(12) X(24) X(36) X(48)             \
  X(60) X(72) X(96) X(108)            \
  X(120) X(144) X(180) X(192)         \
  X(216) X(240) X(288) X(300)         \
  X(324) X(360) X(384) X(432)         \
  X(480) X(540) X(576) X(600)         \
  X(648) X(720) X(768)

#define NSC_LEN_DECL(N) LenOps len64_##N(), len32_##N();
NSC_LENGTHS(NSC_LEN_DECL)
#undef NSC_LEN_DECL
LenOps len32_1536();

}  // namespace nsc
