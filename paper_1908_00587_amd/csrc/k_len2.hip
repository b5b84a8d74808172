// Fixed-length transform passes (nl_lengths.h).
#include "nl_kernels.h"

namespace nsc {
NSC_LEN(60)
NSC_LEN(72)
NSC_LEN(96)
NSC_LEN(108)
}  // namespace nsc
