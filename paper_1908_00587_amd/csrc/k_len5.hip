// Fixed-length transform passes (nl_lengths.h).
#include "nl_kernels.h"

namespace nsc {
NSC_LEN(324)
NSC_LEN(360)
NSC_LEN(384)
NSC_LEN(432)
}  // namespace nsc
