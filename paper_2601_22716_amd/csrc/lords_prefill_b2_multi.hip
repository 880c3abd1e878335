// The large-M kernel for 2-bit codes, several matrices in a launch (see lords_prefill_b2.hip).
#include "lords_prefill_kernel.h"

namespace lords {

hipError_t launch_prefill_2bit(const PrefillArgsT<kMaxBatch> &a, const PfShape &d, dim3 grid, hipStream_t st) { return launch_pf_bits<2, true>(a, d, grid, st); }

}  // namespace lords
