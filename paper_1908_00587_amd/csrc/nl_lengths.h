// Transform lengths with compile-time kernels: three times every count of modes
// with no prime factor above 5 from 4 to 150, three times every such multiple
// of 4 up to 256, in both precisions, and 1536 in FP32.  Other lengths run the
// runtime-length stages, about half as fast (all three passes in FP64: 64 rows of
// 81 x 81 points 76 against 48 us, 24 rows of 405 x 405 points 602 against 286).
// What bounds the list is the build: the last eighteen lengths took it from 60 to
// 95 s on eight cores and the library from 11.6 to 17.2 MiB.  486, 675, 729 and
// 750, the counts past 150 that are no multiples of 4, are left out on that
// account alone.
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
#define NSC_LENGTHS(X)                        \
  X(12) X(24) X(36) X(48)                     \
  X(60) X(72) X(96) X(108)                    \
  X(120) X(144) X(180) X(192)                 \
  X(216) X(240) X(288) X(300)                 \
  X(324) X(360) X(384) X(432)                 \
  X(480) X(540) X(576) X(600)                 \
  X(648) X(720) X(768)                        \
  X(15) X(18) X(27) X(30) X(45) X(54)         \
  X(75) X(81) X(90) X(135) X(150)             \
  X(162) X(225) X(243)                        \
  X(270) X(375)                               \
  X(405) X(450)

#define NSC_LEN_DECL(N) LenOps len64_##N(), len32_##N();
NSC_LENGTHS(NSC_LEN_DECL)
#undef NSC_LEN_DECL
LenOps len32_1536();

}  // namespace nsc
