// executor_generic.hip -- the generic executor kernel: every fold, operator and type mix, and the
// only one that records traces.
#include "executor_device.h"

namespace hccl {

hipError_t launch_generic(const LaunchArgs& a, uint32_t blocks, hipStream_t stream) {
    hipLaunchKernelGGL(hccl_executor<kKindGeneric>, dim3(blocks), dim3(kBlockThreads), 0, stream, a);
    return hipGetLastError();
}

hipError_t generic_occupancy(int* blocks_per_cu) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, hccl_executor<kKindGeneric>, kBlockThreads, 0);
}

}  // namespace hccl
