// The large-M kernel for 4-bit codes, one matrix (the kernel template lives in lords_prefill_kernel.h; a translation unit for
// each code width, and one for several matrices, keep the build parallel).
#include "lords_prefill_kernel.h"

namespace lords {

hipError_t launch_prefill_4bit(const PrefillArgsT<1> &a, const PfShape &d, dim3 grid, hipStream_t st) { return launch_pf_bits<4, false>(a, d, grid, st); }

}  // namespace lords
