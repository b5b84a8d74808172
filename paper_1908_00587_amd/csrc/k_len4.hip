// Fixed-length transform passes (nl_lengths.h).
#include "nl_kernels.h"

namespace nsc {
NSC_LEN(216)
NSC_LEN(240)
NSC_LEN(288)
NSC_LEN(300)
}  // namespace nsc
