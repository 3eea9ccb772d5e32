// executor_dynamic.hip -- kernels of a lone AllToAllvDynamic, described by the launch packet alone.
//
// The layout is worked out from the count matrix when the kernel runs, by rules that are those of
// dyn_slot (executor_device.h). There every wavefront reads the whole matrix by itself, a few
// rows at a time. Here a wavefront plans in registers up to 8 ranks (one load brings the matrix),
// and above that a workgroup of 16 wavefronts plans together, once, in LDS: every row is read by one
// wavefront, all rows at the same time, and each tile is then found with two ballots.
#include "executor_runs.h"

namespace hccl {

namespace {

// Inclusive prefix sum over the lanes of a wavefront.
__device__ __forceinline__ uint32_t scan32(uint32_t v, uint32_t lane) {
#pragma unroll
    for (uint32_t d = 1; d < (uint32_t)kWaveSize; d <<= 1) {
        const uint32_t t = __shfl_up(v, d);
        if (lane >= d) v += t;
    }
    return v;
}

__device__ __forceinline__ uint32_t lane32(uint32_t v, uint32_t j) { return __builtin_amdgcn_readlane(v, j); }

// The first error of a communicator is kept until it is read.
__device__ __forceinline__ void reject(ErrorRecord* err) {
    uint32_t zero = 0;
    if (__hip_atomic_compare_exchange_strong(&err->code, &zero, 2u, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT)) {
        __hip_atomic_store(&err->desc, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&err->tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Whether a non-empty range [x, x + c) leaves a buffer of `cap` rows.
__device__ __forceinline__ bool outside(uint32_t c, int64_t x, uint32_t cap) {
    return c && (x < 0 || (uint64_t)x > cap || c > cap - (uint64_t)x);
}

// Tile t of a pair of c rows, rows [so, so + c) of `src` to rows [ro, ro + c) of `dst`.
template <int ES>
__device__ __forceinline__ void copy_pair_tile(const DynamicArgs& a, const char* src, char* dst, uint32_t so, uint32_t ro,
                                               uint32_t c, uint32_t t, uint32_t lane) {
    src += (uint64_t)so * a.row_elems * ES;
    dst += (uint64_t)ro * a.row_elems * ES;
    uint64_t e0;
    uint32_t n;
    if (!tile_range(t, 1u << a.tile_shift, line_pad((uint64_t)dst, ES), (uint64_t)c * a.row_elems, e0, n)) return;
    src += e0 * ES;
    dst += e0 * ES;
    if ((((uint64_t)src ^ (uint64_t)dst) & 15u) == 0) copy_run<ES, true>(src, dst, n, lane);
    else copy_run<ES>(src, dst, n, lane);
}

// Up to 8 ranks: lane l stands for the pair (source, destination) = (l % P, l / P).
template <int ES>
__global__ void __launch_bounds__(kBlockThreads) hccl_dynamic_small(DynamicArgs a) {
    const uint32_t lane = __lane_id();
    const uint32_t wave = uni(blockIdx.x * kWavesPerBlock + threadIdx.x / kWaveSize);
    const uint64_t send = lane_entry(offsetof(DynamicArgs, send), lane), recv = lane_entry(offsetof(DynamicArgs, recv), lane);
    const uint32_t P = a.P, PP = P * P;
    const bool on = lane < PP;
    const uint32_t d = on ? lane / P : 0u, s = on ? lane - d * P : 0u;
    const uint32_t most = a.send_cap < a.recv_cap ? a.send_cap : a.recv_cap;
    const int64_t cx = on ? a.counts[s * P + d] : 0;
    const int64_t sx = on && a.sdispls ? a.sdispls[s * P + d] : 0;
    const int64_t rx = on && a.rdispls ? a.rdispls[d * P + s] : 0;
    bool bad = cx < 0 || (uint64_t)cx > most;
    const uint32_t c = bad ? 0u : (uint32_t)cx;
    uint32_t row = 0, col = 0, so = 0, ro = 0;
    for (uint32_t j = 0; j < P; ++j) {
        const uint32_t cr = __shfl(c, (int)(j * P + s)), cc = __shfl(c, (int)(d * P + j));  // pairs (s, j), (j, d)
        row += cr;
        col += cc;
        if (j < d) so += cr;
        if (j < s) ro += cc;
    }
    if (a.sdispls) {
        bad |= outside(c, sx, a.send_cap);
        so = (uint32_t)sx;
    } else {
        bad |= on && row > a.send_cap;
    }
    if (a.rdispls) {
        bad |= outside(c, rx, a.recv_cap);
        ro = (uint32_t)rx;
        const uint64_t r = (uint64_t)rx;  // (a range out of bounds has already failed)
        for (uint32_t j = 0; j < P; ++j) {
            const uint32_t cj = __shfl(c, (int)(d * P + j));
            const uint64_t rj = __shfl(r, (int)(d * P + j));
            bad |= j != s && c && cj && r < rj + cj && rj < r + c;
        }
    } else {
        bad |= on && col > a.recv_cap;
    }
    const bool rejected = __ballot(bad) != 0ull;
    if (wave == 0) {
        if (a.recvcounts && on) a.recvcounts[d * P + s] = cx;
        if (rejected && lane == 0) reject(a.error);
    }
    if (rejected) return;  // move nothing
    const uint32_t tiles = (uint32_t)(((uint64_t)c * a.row_elems + (1u << a.tile_shift) - 1) >> a.tile_shift);
    const uint32_t incl = scan32(tiles, lane), J = lane32(incl, kWaveSize - 1);
    for (uint32_t j = wave; j < J; j += a.nworkers) {
        const uint32_t p = (uint32_t)__popcll(__ballot(incl <= j));
        const uint32_t pd = p / P, ps = p - pd * P;
        copy_pair_tile<ES>(a, (const char*)from_lane(send, ps), (char*)from_lane(recv, pd), lane32(so, p), lane32(ro, p), lane32(c, p),
                           j - (p ? lane32(incl, p - 1) : 0u), lane);
    }
}

// Up to 64 ranks: the workgroup plans in LDS. Wavefront w owns rows (sources) w * R ... of the matrix,
// lane d standing for destination d.
constexpr int kPlanWaves = 16;
constexpr int kPlanRows = kMaxRanks / kPlanWaves;  // rows of one wavefront, at most
constexpr int kPlanStride = kMaxRanks + 1;         // words of a row: a column then touches every bank

template <int ES>
__global__ void __launch_bounds__(kPlanWaves * kWaveSize) hccl_dynamic_wide(DynamicArgs a) {
    __shared__ uint32_t l_count[kMaxRanks * kPlanStride];  // rows of the pair
    __shared__ uint32_t l_send[kMaxRanks * kPlanStride];   // its first row in the send buffer
    __shared__ uint32_t l_recv[kMaxRanks * kPlanStride];   // ... and in the receive buffer
    __shared__ uint32_t l_tiles[kMaxRanks * kPlanStride];  // tiles of its row up to and with it
    __shared__ uint32_t l_part[kPlanWaves * kMaxRanks];    // rows that each wavefront's sources send to each destination
    __shared__ uint32_t l_row[kMaxRanks];                  // tiles of a row
    __shared__ uint32_t l_bad;
    const uint32_t lane = __lane_id(), w = uni(threadIdx.x / kWaveSize);
    const uint64_t send = lane_entry(offsetof(DynamicArgs, send), lane), recv = lane_entry(offsetof(DynamicArgs, recv), lane);
    const uint32_t P = a.P, rows = (P + kPlanWaves - 1) / kPlanWaves;
    const uint32_t most = a.send_cap < a.recv_cap ? a.send_cap : a.recv_cap;
    if (threadIdx.x == 0) l_bad = 0;

    int64_t cx[kPlanRows], sx[kPlanRows], rx[kPlanRows];
    bool in[kPlanRows];
#pragma unroll
    for (int i = 0; i < kPlanRows; ++i) {
        const uint32_t s = w * rows + i;
        in[i] = (uint32_t)i < rows && s < P && lane < P;
        cx[i] = in[i] ? a.counts[s * P + lane] : 0;
        sx[i] = in[i] && a.sdispls ? a.sdispls[s * P + lane] : 0;
        rx[i] = in[i] && a.rdispls ? a.rdispls[lane * P + s] : 0;
    }
    bool bad = false;
    uint32_t c[kPlanRows], part = 0;
#pragma unroll
    for (int i = 0; i < kPlanRows; ++i) {
        const uint32_t s = w * rows + i;
        const bool wrong = cx[i] < 0 || (uint64_t)cx[i] > most;
        bad |= wrong;
        c[i] = wrong ? 0u : (uint32_t)cx[i];
        part += c[i];
        const uint32_t before = scan32(c[i], lane) - c[i];
        const uint32_t tiles = scan32((uint32_t)(((uint64_t)c[i] * a.row_elems + (1u << a.tile_shift) - 1) >> a.tile_shift), lane);
        if (a.sdispls) bad |= outside(c[i], sx[i], a.send_cap);
        else bad |= before + c[i] > a.send_cap;  // a packed source fits iff its total fits
        if (in[i]) {
            l_count[s * kPlanStride + lane] = c[i];
            l_send[s * kPlanStride + lane] = a.sdispls ? (uint32_t)sx[i] : before;
            l_tiles[s * kPlanStride + lane] = tiles;
            if (lane == P - 1) l_row[s] = tiles;
            if (a.recvcounts && blockIdx.x == 0) a.recvcounts[lane * P + s] = cx[i];
        }
    }
    l_part[w * kMaxRanks + lane] = part;
    __syncthreads();
    uint32_t col = 0, all = 0;  // rows that destination `lane` gets from the wavefronts before this one; from all
#pragma unroll
    for (int q = 0; q < kPlanWaves; ++q) {
        const uint32_t v = l_part[q * kMaxRanks + lane];
        all += v;
        if ((uint32_t)q < w) col += v;
    }
    if (!a.rdispls) bad |= all > a.recv_cap;
#pragma unroll
    for (int i = 0; i < kPlanRows; ++i) {
        if (a.rdispls) bad |= outside(c[i], rx[i], a.recv_cap);
        if (in[i]) l_recv[(w * rows + i) * kPlanStride + lane] = a.rdispls ? (uint32_t)rx[i] : col;
        col += c[i];
    }
    if (a.rdispls) {
        // Receive ranges of one destination must not overlap (lane = source; the ranges that leave
        // their buffer have already failed, so the others' sums are below 2^32).
        __syncthreads();
        for (uint32_t d = w; d < P; d += kPlanWaves) {
            const uint32_t cs = lane < P ? l_count[lane * kPlanStride + d] : 0u;
            const uint32_t r = lane < P ? l_recv[lane * kPlanStride + d] : 0u;
            for (uint32_t j = 0; j < P; ++j) {
                const uint32_t cj = lane32(cs, j), rj = lane32(r, j);
                bad |= j != lane && cs && cj && r < rj + cj && rj < r + cs;
            }
        }
    }
    if (__ballot(bad) != 0ull && lane == 0) l_bad = 1;
    __syncthreads();
    if (l_bad) {  // move nothing
        if (blockIdx.x == 0 && threadIdx.x == 0) reject(a.error);
        return;
    }
    const uint32_t incl = scan32(lane < P ? l_row[lane] : 0u, lane), J = lane32(incl, kWaveSize - 1);
    for (uint32_t j = uni(blockIdx.x * kPlanWaves + w); j < J; j += a.nworkers) {
        const uint32_t s = (uint32_t)__popcll(__ballot(incl <= j));
        const uint32_t jr = j - (s ? lane32(incl, s - 1) : 0u);
        const uint32_t mine = lane < P ? l_tiles[s * kPlanStride + lane] : ~0u;
        const uint32_t d = (uint32_t)__popcll(__ballot(mine <= jr));
        const uint32_t at = s * kPlanStride + d;
        copy_pair_tile<ES>(a, (const char*)from_lane(send, s), (char*)from_lane(recv, d), uni(l_send[at]), uni(l_recv[at]), uni(l_count[at]),
                           jr - (d ? lane32(mine, d - 1) : 0u), lane);
    }
}

}  // namespace

uint32_t dynamic_waves_per_block(uint32_t P) { return P <= 8 ? kWavesPerBlock : kPlanWaves; }

hipError_t launch_dynamic(const DynamicArgs& a, uint32_t elem_bytes, uint32_t blocks, hipStream_t s) {
    const bool small = a.P <= 8;
    const dim3 threads(dynamic_waves_per_block(a.P) * kWaveSize);
    if (small && elem_bytes == 2) hipLaunchKernelGGL(hccl_dynamic_small<2>, dim3(blocks), threads, 0, s, a);
    else if (small) hipLaunchKernelGGL(hccl_dynamic_small<4>, dim3(blocks), threads, 0, s, a);
    else if (elem_bytes == 2) hipLaunchKernelGGL(hccl_dynamic_wide<2>, dim3(blocks), threads, 0, s, a);
    else hipLaunchKernelGGL(hccl_dynamic_wide<4>, dim3(blocks), threads, 0, s, a);
    return hipGetLastError();
}

}  // namespace hccl
