// Fixed-length transform passes (nl_lengths.h).
#include "nl_kernels.h"

namespace nsc {
NSC_LEN(405)
NSC_LEN(450)
}  // namespace nsc
