// executor_runs.h -- tiles and copies of the kernels that find their work without a program image.
#pragma once

#include "executor_device.h"

namespace hccl {
namespace {

// Entry `lane` of the 64-entry list at byte `off` of the kernel arguments.
__device__ __forceinline__ uint64_t lane_entry(size_t off, uint32_t lane) {
    return ((const uint64_t*)((const char*)__builtin_amdgcn_kernarg_segment_ptr() + off))[lane];
}

// Elements that tile 0 of a segment takes beyond its tile size, so that every other tile begins on a
// 128-byte line of its (first) destination: a non-temporal store of part of a line costs a line.
__device__ __forceinline__ uint32_t line_pad(uint64_t dst, uint32_t es) {
    return (uint32_t)((128u - (dst & 127u)) & 127u) / es;
}

// Elements [e0, e0 + n) of a segment of `total` that its tile k covers; false if there are none.
__device__ __forceinline__ bool tile_range(uint32_t k, uint32_t te, uint32_t pad, uint64_t total, uint64_t& e0, uint32_t& n) {
    e0 = k ? (uint64_t)k * te + pad : 0;
    if (e0 >= total) return false;
    const uint64_t left = total - e0, most = k ? te : te + pad;
    n = (uint32_t)(left < most ? left : most);
    return true;
}

template <int ES, int U, bool ONCE>
__device__ __forceinline__ uint32_t copy_steps(const char* src, char* dst, uint32_t at, uint32_t nvec, uint32_t lane) {
    for (; at + U * kWaveSize <= nvec; at += U * kWaveSize) {
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = ONCE ? vld(src + 16u * (at + u * kWaveSize + lane)) : vld_shifted<ES>(src + 16u * (at + u * kWaveSize + lane));
#pragma unroll
        for (int u = 0; u < U; ++u) vst_copy(dst + 16u * (at + u * kWaveSize + lane), v[u]);
    }
    return at;
}

// n elements from src to dst: 16-byte stores to dst's own alignment, after fewer than 16 bytes of
// single elements, of 16-byte loads at whatever alignment that leaves the source. ONCE: no other
// wavefront reads the source, and it is 16-byte aligned where dst is: non-temporal loads.
template <int ES, bool ONCE = false>
__device__ __forceinline__ void copy_run(const char* src, char* dst, uint32_t n, uint32_t lane) {
    typedef typename std::conditional<ES == 2, uint16_t, uint32_t>::type W;
    uint32_t head = (uint32_t)(16u - ((uint64_t)dst & 15u)) % 16u / ES;
    if (head > n) head = n;
    const uint32_t nvec = (n - head) * ES / 16u, rest = n - head - nvec * (16u / ES);
    // the single elements before and after the vectors, one per lane
    if (lane < head + rest) {
        const uint32_t e = lane < head ? lane : n - rest + (lane - head);
        *gp<W>(dst + (uint64_t)e * ES) = *gp<W>(src + (uint64_t)e * ES);
    }
    const char* s = src + head * ES;
    char* d = dst + head * ES;
    uint32_t at = copy_steps<ES, 8, ONCE>(s, d, 0, nvec, lane);
    at = copy_steps<ES, 4, ONCE>(s, d, at, nvec, lane);
    for (at += lane; at < nvec; at += kWaveSize) vst_copy(d + 16u * at, ONCE ? vld(s + 16u * at) : vld_shifted<ES>(s + 16u * at));
}

}  // namespace
}  // namespace hccl
