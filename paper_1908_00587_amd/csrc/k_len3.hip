// Fixed-length transform passes (nl_lengths.h).
#include "nl_kernels.h"

namespace nsc {
NSC_LEN(120)
NSC_LEN(144)
NSC_LEN(180)
NSC_LEN(192)
}  // namespace nsc
