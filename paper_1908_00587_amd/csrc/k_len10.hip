// Fixed-length transform passes (nl_lengths.h).
#include "nl_kernels.h"

namespace nsc {
NSC_LEN(162)
NSC_LEN(225)
NSC_LEN(243)
}  // namespace nsc
