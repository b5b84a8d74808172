// Fixed-length transform passes (nl_lengths.h).
#include "nl_kernels.h"

namespace nsc {
NSC_LEN(480)
NSC_LEN(540)
NSC_LEN(576)
NSC_LEN(600)
}  // namespace nsc
