// Fixed-length transform passes (nl_lengths.h).
#include "nl_kernels.h"

namespace nsc {
NSC_LEN(75)
NSC_LEN(81)
NSC_LEN(90)
NSC_LEN(135)
NSC_LEN(150)
}  // namespace nsc
