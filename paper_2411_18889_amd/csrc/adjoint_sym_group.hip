// The symmetric adjoint's one-wave-per-group kernels of the plain FP32 and
// FP64 policies (adjoint_group_kernel in adjoint_sym_pairs.h), in a
// translation unit of their own so that they can be built with their own
// instruction schedule: the build compiles this file with the maximum-ILP
// strategy (-mllvm -amdgpu-sched-strategy=max-ilp). FP32 at 16384 particles:
// 120 against 132 us with the default strategy (entry pass), 147 against 165
// (with the force sums); FP64 is the same either way. The tile-compensated
// kernels are faster as the files around them are built (165 against 170).
#include "adjoint_sym_pairs.h"

namespace nb {
namespace asym {

hipError_t launch_group_own(const ASymArgs<PolF32>& a, bool force_sums, hipStream_t stream) {
    return force_sums ? launch_group<PolF32, true>(a, stream) : launch_group<PolF32, false>(a, stream);
}
hipError_t launch_group_own(const ASymArgs<PolF64>& a, bool force_sums, hipStream_t stream) {
    return force_sums ? launch_group<PolF64, true>(a, stream) : launch_group<PolF64, false>(a, stream);
}

}  // namespace asym
}  // namespace nb
