// Fixed-length transform passes (nl_lengths.h).
#include "nl_kernels.h"

namespace nsc {
NSC_LEN(12)
NSC_LEN(24)
NSC_LEN(36)
NSC_LEN(48)
}  // namespace nsc
