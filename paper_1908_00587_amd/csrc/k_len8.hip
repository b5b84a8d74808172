// Fixed-length transform passes (nl_lengths.h).
#include "nl_kernels.h"

namespace nsc {
NSC_LEN(15)
NSC_LEN(18)
NSC_LEN(27)
NSC_LEN(30)
NSC_LEN(45)
NSC_LEN(54)
}  // namespace nsc
