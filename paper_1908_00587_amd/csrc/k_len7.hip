// Fixed-length transform passes (nl_lengths.h).
#include "nl_kernels.h"

namespace nsc {
NSC_LEN(648)
NSC_LEN(720)
NSC_LEN(768)
NSC_LEN32(1536)
}  // namespace nsc
