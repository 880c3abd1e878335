// The large-M kernel for 4-bit codes, several matrices in a launch (see lords_prefill_b4.hip).
#include "lords_prefill_kernel.h"

namespace lords {

hipError_t launch_prefill_4bit(const PrefillArgsT<kMaxBatch> &a, const PfShape &d, dim3 grid, hipStream_t st) { return launch_pf_bits<4, true>(a, d, grid, st); }

}  // namespace lords
