// The large-M kernel for 4-bit codes (the kernel template lives in lords_prefill_kernel.h; one translation unit per code
// width keeps the build parallel).
#include "lords_prefill_kernel.h"

namespace lords {

hipError_t launch_prefill_4bit(const PrefillArgsT<1> &a, const PfShape &d, dim3 grid, hipStream_t st) { return launch_pf_bits<4, false>(a, d, grid, st); }
hipError_t launch_prefill_4bit(const PrefillArgsT<kMaxBatch> &a, const PfShape &d, dim3 grid, hipStream_t st) { return launch_pf_bits<4, true>(a, d, grid, st); }

}  // namespace lords
