// Test shim: a term-parallel walk kernel and a learned one, for a look at the
// code that is generated for them (test_kernarg.py).
#include "../paper_2511_20317_amd/csrc/walk_kernel.h"

namespace tsfk {
template __global__ void walk_kernel<64, 1, uint32_t, false, false, false>(KArgs);
template __global__ void walk_learned_kernel<8, 1, uint32_t, false>(KArgs);
}  // namespace tsfk
