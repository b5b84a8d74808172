// Fixed-length transform passes (nl_lengths.h).
#include "nl_kernels.h"

namespace nsc {
NSC_LEN(270)
NSC_LEN(375)
}  // namespace nsc
