// The symmetric adjoint's one-wave-per-group kernels of the plain FP32 policy
// (adjoint_group_kernel in adjoint_sym_pairs.h), in a translation unit of their
// own so that they can be built with their own instruction schedule: the build
// compiles this file with the maximum-ILP strategy (-mllvm
// -amdgpu-sched-strategy=max-ilp). 16384 particles: 111 against 121 us with the
// default strategy (entry pass), 136.6 against 137.9 (with the force sums). The
// FP64 kernels are faster with the default (entry pass 191 against 196), the
// tile-compensated ones as the files around them are built (165 against 170).
#include "adjoint_sym_pairs.h"

namespace nb {
namespace asym {

hipError_t launch_group_own(const ASymArgs<PolF32>& a, bool force_sums, hipStream_t stream) {
    return force_sums ? launch_group<PolF32, true>(a, stream) : launch_group<PolF32, false>(a, stream);
}

}  // namespace asym
}  // namespace nb
