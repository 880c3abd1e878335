// The large-M kernel for 3-bit codes, several matrices in a launch (see lords_prefill_b3.hip).
#include "lords_prefill_kernel.h"

namespace lords {

hipError_t launch_prefill_3bit(const PrefillArgsT<kMaxBatch> &a, const PfShape &d, dim3 grid, hipStream_t st) { return launch_pf_bits<3, true>(a, d, grid, st); }

}  // namespace lords
