// executor.hip -- launchers of the executor kernels, and the static workspace. The kernels are in
// executor_device.h; the generic and the resident one have files of their own.
#include <hip/hip_runtime.h>

#include <stddef.h>

#include <mutex>

#include "executor_device.h"

namespace hccl {

// Workspace of the allocation-free entry point: the program image, the dependency counters and
// the FP32 partials of one call live here instead of in memory the library allocates. Every
// device the library runs on holds its own copy, from the loading of this code object until
// the process ends. In host code `scratch` only names the symbol: its device address comes
// from workspace_address(), and only that address is ever handed to a kernel or a copy.
constexpr size_t kWorkspaceBytes = size_t(64) << 20;
static __device__ __align__(256) unsigned char scratch[kWorkspaceBytes];

namespace {

// The completion word of a triggered collective, launched right behind the executor on its
// stream (the paper's dedicated subgraph for the set, Section IV-B-3): the executor's results
// are visible device-wide once it has ended, which costs nothing extra, whereas a write-back
// of the L2 by every workgroup before a word set from inside the executor measured 15-20 us.
// Nothing is written if the launch recorded an error.
__global__ void hccl_signal(uint64_t* word, uint64_t value, const ErrorRecord* err) {
    if (threadIdx.x == 0 && blockIdx.x == 0 &&
        __hip_atomic_load(&err->code, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u)
        __hip_atomic_store(word, value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ void hccl_fill_u32(uint32_t* p, uint64_t n, uint32_t v) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i < n; i += (uint64_t)gridDim.x * blockDim.x) p[i] = v;
}

}  // namespace

// the generic kernel (executor_generic.hip)
hipError_t launch_generic(const LaunchArgs& a, uint32_t blocks, hipStream_t stream);
hipError_t generic_occupancy(int* blocks_per_cu);

int executor_block_threads() { return kBlockThreads; }

size_t workspace_bytes() { return kWorkspaceBytes; }

// Device address of the static workspace on the current device, looked up once per device
// and kept for the rest of the process.
hipError_t workspace_address(void** ptr) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}
int executor_waves_per_block() { return kWavesPerBlock; }

// kind: a plain signature (SIG_BF16 .. SIG_INT32) for SUM-only programs of that signature,
// kKindCopyOnly, or anything else for the generic kernel.
hipError_t launch_executor(const LaunchArgs& a, uint32_t blocks, int kind, hipStream_t stream) {
    switch (kind) {
        case SIG_BF16: hipLaunchKernelGGL(hccl_executor<SIG_BF16>, dim3(blocks), dim3(kBlockThreads), 0, stream, a); break;
        case SIG_FP16: hipLaunchKernelGGL(hccl_executor<SIG_FP16>, dim3(blocks), dim3(kBlockThreads), 0, stream, a); break;
        case SIG_FP32: hipLaunchKernelGGL(hccl_executor<SIG_FP32>, dim3(blocks), dim3(kBlockThreads), 0, stream, a); break;
        case SIG_INT32: hipLaunchKernelGGL(hccl_executor<SIG_INT32>, dim3(blocks), dim3(kBlockThreads), 0, stream, a); break;
        case kKindCopyOnly:
            hipLaunchKernelGGL(hccl_executor<kKindCopyOnly>, dim3(blocks), dim3(kBlockThreads), 0, stream, a);
            break;
        case kKindCopyAligned:
            hipLaunchKernelGGL(hccl_executor<kKindCopyAligned>, dim3(blocks), dim3(kBlockThreads), 0, stream, a);
            break;
        case kKindDynamic:
            hipLaunchKernelGGL(hccl_executor<kKindDynamic>, dim3(blocks), dim3(kBlockThreads), 0, stream, a);
            break;
        default: return launch_generic(a, blocks, stream);
    }
    return hipGetLastError();
}

hipError_t launch_signal(uint64_t* word, uint64_t value, const ErrorRecord* err, hipStream_t stream) {
    hipLaunchKernelGGL(hccl_signal, dim3(1), dim3(64), 0, stream, word, value, err);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, uint64_t n, uint32_t v, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    uint64_t blocks = (n + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(hccl_fill_u32, dim3((uint32_t)blocks), dim3(256), 0, stream, p, n, v);
    return hipGetLastError();
}

// Resident blocks per CU of the kernel of one kind.
hipError_t executor_occupancy(int kind, int* blocks_per_cu) {
    switch (kind) {
        case SIG_BF16: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, hccl_executor<SIG_BF16>, kBlockThreads, 0);
        case SIG_FP16: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, hccl_executor<SIG_FP16>, kBlockThreads, 0);
        case SIG_FP32: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, hccl_executor<SIG_FP32>, kBlockThreads, 0);
        case SIG_INT32: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, hccl_executor<SIG_INT32>, kBlockThreads, 0);
        case kKindCopyOnly: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, hccl_executor<kKindCopyOnly>, kBlockThreads, 0);
        case kKindCopyAligned: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, hccl_executor<kKindCopyAligned>, kBlockThreads, 0);
        case kKindDynamic: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, hccl_executor<kKindDynamic>, kBlockThreads, 0);
        default: return generic_occupancy(blocks_per_cu);
    }
}

}  // namespace hccl
