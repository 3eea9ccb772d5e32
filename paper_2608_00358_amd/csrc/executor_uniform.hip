// executor_uniform.hip -- kernels of the uniform phases (UniformArgs): one fold or one copy over
// equal segments, described by the launch packet alone.
//
// A wavefront of the descriptor executor finds its tile through the program image: header, tile
// table, descriptor, operands, buffer table, each a dependent read of memory. Here tile number and
// kernel arguments give every address by arithmetic. Every kernel
// is compiled for one type, one operator and one fold, with as many loads in flight as that allows.
#include "executor_runs.h"

namespace hccl {

namespace {

enum Mode { M_SUM, M_MINMAX, M_REQ };  // M_REQ: SUM, every partial rounded to the element type

constexpr int kBatch = 8;   // sources whose loads are in flight together
constexpr int kUnroll = 2;  // 16-byte vectors per lane and source in flight

template <int T> constexpr int kVec = 16 / DtInfo<T>::size;  // elements of a 16-byte vector

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Two fp32 -> bf16 in one instruction (v_cvt_pk_bf16_f32): the same bits as bf16_bits for all 2^32
// inputs, NaNs included.
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
    const f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

template <int T, typename A>
__device__ __forceinline__ void widen(const u32x4& r, A (&x)[kVec<T>]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (T == DT_BF16) {
            x[2 * i] = bf16_lo(r[i]);
            x[2 * i + 1] = bf16_hi(r[i]);
        } else if constexpr (T == DT_FP16) {
            x[2 * i] = f16_lo(r[i]);
            x[2 * i + 1] = f16_hi(r[i]);
        } else if constexpr (T == DT_FP32) {
            x[i] = __uint_as_float(r[i]);
        } else {
            x[i] = (int32_t)r[i];
        }
    }
}

template <int T, typename A>
__device__ __forceinline__ u32x4 narrow(const A (&x)[kVec<T>]) {
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (T == DT_BF16) w[i] = bf16_pair(x[2 * i], x[2 * i + 1]);
        else if constexpr (T == DT_FP16) w[i] = f16_bits(x[2 * i]) | (f16_bits(x[2 * i + 1]) << 16);
        else if constexpr (T == DT_FP32) w[i] = __float_as_uint(x[i]);
        else w[i] = (uint32_t)x[i];
    }
    return w;
}

// a = a op x, element by element; OPR is RO_SUM, RO_MAX or RO_MIN.
template <int T, int OPR, bool REQ, typename A>
__device__ __forceinline__ void combine(A (&a)[kVec<T>], const A (&x)[kVec<T>]) {
#pragma unroll
    for (int i = 0; i < kVec<T>; ++i) a[i] = comb<OPR>(a[i], x[i]);
    if constexpr (REQ) widen<T, A>(narrow<T, A>(a), a);
}

// The fold of one tile's segment: where its sources and destinations are. Lane j holds entry j of
// the operand lists: one vector load brings a list of 64, where scalar loads of the entries in
// turn would wait for eight cache lines one after the other.
struct Fold1 {
    uint64_t src, dst;
    uint64_t src_off, dst_off;  // bytes from a list entry to element 0 of the tile
    uint32_t nsrc, ndst, group;
    uint32_t rot, flip;         // source i of the fold is entry (i + rot) mod nsrc, or i ^ flip
    uint32_t first;             // entry of destination 0
    __device__ __forceinline__ const char* source(uint32_t i) const {
        uint32_t k = i + rot;
        if (k >= nsrc) k -= nsrc;
        return (const char*)(from_lane(src, k ^ flip) + src_off);
    }
    __device__ __forceinline__ char* dest(uint32_t j) const { return (char*)(from_lane(dst, first + j) + dst_off); }
};

// MEM: which accesses are ordinary (MemFlags); the others are non-temporal. SHIFT: addresses aligned only to the element.
template <int T, bool SHIFT, int MEM>
__device__ __forceinline__ u32x4 load_vec(const char* p) {
    if constexpr (SHIFT) return vld_shifted<DtInfo<T>::size>(p);
    else if constexpr (MEM & MEM_LOAD) return *gp<u32x4>(p);
    else return __builtin_nontemporal_load(gp<u32x4>(p));
}
template <int T, bool SHIFT, int MEM>
__device__ __forceinline__ void store_vec(char* p, u32x4 v) {
    typedef typename std::conditional<DtInfo<T>::size == 2, u32x4_a2, u32x4_a4>::type VU;
    typedef typename std::conditional<SHIFT, VU, u32x4>::type V;
    if constexpr (MEM & MEM_STORE) *gp<V>(p) = (V)v;
    else __builtin_nontemporal_store((V)v, gp<V>(p));
}

// Fold in list order of U vectors per lane, the first at byte `at` of the tile, 1 KiB apart.
// The loads of kBatch sources are all issued before the first of them is folded: one memory round
// trip for 8 sources.
template <int T, int OPR, bool REQ, int U, bool SHIFT, int MEM, bool GROUPED>
__device__ __forceinline__ void fold_list(const Fold1& f, uint32_t at) {
    typedef typename DtInfo<T>::acc A;
    A acc[U][kVec<T>], tot[GROUPED ? U : 1][kVec<T>];
    const uint32_t L = GROUPED ? f.group : f.nsrc;
    for (uint32_t g0 = 0; g0 < f.nsrc; g0 += L) {
        const uint32_t end = (!GROUPED || g0 + L > f.nsrc) ? f.nsrc : g0 + L;
        for (uint32_t s = g0; s < end; s += kBatch) {
            u32x4 r[kBatch][U];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                if (s + j < end) {
                    const char* b = f.source(s + j);
#pragma unroll
                    for (int u = 0; u < U; ++u) r[j][u] = load_vec<T, SHIFT, MEM>(b + (at + u * 1024u));
                }
            }
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                if (s + j < end) {
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        A x[kVec<T>];
                        widen<T, A>(r[j][u], x);
                        if (j == 0 && s == g0) {
#pragma unroll
                            for (int i = 0; i < kVec<T>; ++i) acc[u][i] = x[i];
                        } else {
                            combine<T, OPR, REQ, A>(acc[u], x);
                        }
                    }
                }
            }
        }
        if constexpr (GROUPED) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (g0 == 0) {
#pragma unroll
                    for (int i = 0; i < kVec<T>; ++i) tot[u][i] = acc[u][i];
                } else {
                    combine<T, OPR, REQ, A>(tot[u], acc[u]);
                }
            }
        }
    }
    u32x4 w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) w[u] = narrow<T, A>(GROUPED ? tot[GROUPED ? u : 0] : acc[u]);
    for (uint32_t d = 0; d < f.ndst; ++d) {
        char* b = f.dest(d);
#pragma unroll
        for (int u = 0; u < U; ++u) store_vec<T, SHIFT, MEM>(b + (at + u * 1024u), w[u]);
    }
}

// Fold as a complete binary tree over the list: eight sources at a time make one subtree, and the
// subtrees before the current one wait on a stack of three levels (64 sources).
template <int T, bool REQ, bool SHIFT, int MEM>
__device__ __forceinline__ void fold_tree(const Fold1& f, uint32_t at) {
    typedef float A;
    constexpr int V = kVec<T>;
    A stk[3][V], v[V];
    const uint32_t nb = (f.nsrc + 7) / 8;
    for (uint32_t b = 0; b < nb; ++b) {
        u32x4 r[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (8 * b + j < f.nsrc) r[j] = load_vec<T, SHIFT, MEM>(f.source(8 * b + j) + at);
        A p[3][V], x[V];
        // pairs, pairs of pairs, and those two, as far as there are sources
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if ((uint32_t)(2 * q) < f.nsrc) {
                A(&t)[V] = (q & 1) ? p[2] : p[q / 2];
                widen<T, A>(r[2 * q], t);
                if ((uint32_t)(2 * q + 1) < f.nsrc) {
                    widen<T, A>(r[2 * q + 1], x);
                    combine<T, RO_SUM, REQ, A>(t, x);
                }
                if (q & 1) combine<T, RO_SUM, REQ, A>(p[q / 2], p[2]);
            }
        }
        if (f.nsrc > 4) combine<T, RO_SUM, REQ, A>(p[0], p[1]);
#pragma unroll
        for (int i = 0; i < V; ++i) v[i] = p[0][i];
        bool open = true;
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            if (open && (2u << l) <= nb) {
                if ((b >> l) & 1u) {
                    combine<T, RO_SUM, REQ, A>(stk[l], v);
#pragma unroll
                    for (int i = 0; i < V; ++i) v[i] = stk[l][i];
                } else {
#pragma unroll
                    for (int i = 0; i < V; ++i) stk[l][i] = v[i];
                    open = false;
                }
            }
        }
    }
    const u32x4 w = narrow<T, A>(v);
    for (uint32_t d = 0; d < f.ndst; ++d) store_vec<T, SHIFT, MEM>(f.dest(d) + at, w);
}

// Elements [first, first + count) of the tile, one per lane: what is left after whole wavefront steps
// if it is less than a vector. The tree's stack has six levels here.
template <int T, int OPR, bool REQ, bool TREE>
__device__ __forceinline__ void fold_elems(const Fold1& f, uint32_t first, uint32_t count, uint32_t lane) {
    typedef typename DtInfo<T>::acc A;
    constexpr uint32_t S = DtInfo<T>::size;
    auto round = [](A v) { return requant<T, REQ>(v); };
    for (uint32_t e = first + lane; e < first + count; e += kWaveSize) {
        A acc = A(0), tot = A(0), stk[TREE ? 6 : 1];
        const uint32_t L = f.group ? f.group : f.nsrc;
        uint32_t left = 0;  // sources of the group still to come
        for (uint32_t s = 0; s < f.nsrc; s += kBatch) {
            A x[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j)
                if (s + j < f.nsrc) x[j] = load1<T, A>(f.source(s + j) + (uint64_t)e * S);
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                if (s + j >= f.nsrc) continue;
                if constexpr (TREE) {
                    bool open = true;
                    acc = x[j];
#pragma unroll
                    for (int l = 0; l < 6; ++l) {
                        if (open && (2u << l) <= f.nsrc) {
                            if (((s + j) >> l) & 1u) acc = round(comb<OPR>(stk[l], acc));
                            else stk[l] = acc, open = false;
                        }
                    }
                } else if (left == 0) {  // the first of a group: what was folded so far joins the total
                    if (s + j == L) tot = acc;
                    else if (s + j > L) tot = round(comb<OPR>(tot, acc));
                    acc = x[j];
                    left = L - 1;
                } else {
                    acc = round(comb<OPR>(acc, x[j]));
                    --left;
                }
            }
        }
        if (!TREE && L < f.nsrc) acc = round(comb<OPR>(tot, acc));
        for (uint32_t d = 0; d < f.ndst; ++d) store1<T, A>(f.dest(d) + (uint64_t)e * S, acc);
    }
}

// The n elements of a tile. The last step takes what is left over whole wavefront steps: the lanes
// whose vector is whole, and one lane more that takes the last vector's worth of elements, some of
// them a second time (in the same step, so that in place every source is read before any result
// is stored). SHIFT: addresses aligned only to the element.
template <int T, int OPR, bool REQ, bool TREE, bool SHIFT, int MEM, bool GROUPED>
__device__ __forceinline__ void fold_vectors(const Fold1& f, uint32_t n, uint32_t lane) {
    constexpr uint32_t S = DtInfo<T>::size, V = kVec<T>, kStep = kWaveSize * V;
    uint32_t e = 0;
    if constexpr (!TREE) {
        for (; e + kUnroll * kStep <= n; e += kUnroll * kStep)
            fold_list<T, OPR, REQ, kUnroll, SHIFT, MEM, GROUPED>(f, (e + lane * V) * S);
    }
    for (; e + kStep <= n; e += kStep) {
        if constexpr (TREE) fold_tree<T, REQ, SHIFT, MEM>(f, (e + lane * V) * S);
        else fold_list<T, OPR, REQ, 1, SHIFT, MEM, GROUPED>(f, (e + lane * V) * S);
    }
    if (e == n) return;
    const uint32_t whole = (n - e) / V;
    if (whole == 0) {
        fold_elems<T, OPR, REQ, TREE>(f, e, n - e, lane);
    } else if (lane * V < n - e) {
        const uint32_t at = (lane < whole ? e + lane * V : n - V) * S;
        if constexpr (TREE) fold_tree<T, REQ, true, MEM>(f, at);
        else fold_list<T, OPR, REQ, 1, true, MEM, GROUPED>(f, at);
    }
}

template <int T, int OPR, bool REQ, bool TREE, int MEM>
__device__ __forceinline__ void fold_tile(const Fold1& f, uint32_t n, bool aligned, uint32_t lane) {
    if constexpr (!TREE && OPR == RO_SUM && T != DT_INT32) {
        if (f.group) {
            if (aligned) fold_vectors<T, OPR, REQ, TREE, false, MEM, true>(f, n, lane);
            else fold_vectors<T, OPR, REQ, TREE, true, MEM, true>(f, n, lane);
            return;
        }
    }
    if (aligned) fold_vectors<T, OPR, REQ, TREE, false, MEM, false>(f, n, lane);
    else fold_vectors<T, OPR, REQ, TREE, true, MEM, false>(f, n, lane);
}

// Number of this wavefront in the launch (see hccl_executor for the XCD order).
__device__ __forceinline__ uint32_t wave_number(bool xcd_order) {
    uint32_t block = blockIdx.x;
    if (xcd_order) {
        const uint32_t B = gridDim.x, x = block % kXcds, j = block / kXcds;
        block = x * (B / kXcds) + (x < B % kXcds ? x : B % kXcds) + j;
    }
    return uni(block * kWavesPerBlock + (threadIdx.x / kWaveSize));
}

template <int T, int MODE, bool TREE, int MEM>
__global__ void __launch_bounds__(kBlockThreads) hccl_uniform_reduce(UniformArgs a, uint32_t redop) {
    const uint32_t lane = __lane_id();
    Fold1 f;
    f.src = lane_entry(offsetof(UniformArgs, src), lane);
    f.dst = lane_entry(offsetof(UniformArgs, dst), lane);
    f.nsrc = a.nsrc;
    f.ndst = a.ndst;
    f.group = a.group;
    for (uint32_t t = wave_number(a.flags & UF_XCD); t < a.ntiles; t += a.nworkers) {
        const uint32_t g = a.nseg > 1 ? t / a.tiles_per_seg : 0u;
        const uint32_t k = t - g * a.tiles_per_seg;
        f.first = a.flags & UF_DST_PER_SEG ? g : 0u;
        const uint32_t pad = a.flags & UF_ALIGNED ? 0u : line_pad(from_lane(f.dst, f.first) + g * a.dst_step, DtInfo<T>::size);
        uint64_t e0;
        uint32_t n;
        if (!tile_range(k, a.tile_elems, pad, g + 1 < a.nseg ? a.seg_elems : a.last_elems, e0, n)) continue;
        f.src_off = g * a.src_step + e0 * DtInfo<T>::size;
        f.dst_off = g * a.dst_step + e0 * DtInfo<T>::size;
        f.rot = a.flags & UF_ROTATE ? (g + 1 < a.nsrc ? g + 1 : 0u) : 0u;
        f.flip = a.flags & UF_FLIP ? __brev(g) >> (__clz(a.nsrc) + 1) : 0u;
        if constexpr (MODE == M_SUM) fold_tile<T, RO_SUM, false, TREE, MEM>(f, n, a.flags & UF_ALIGNED, lane);
        else if constexpr (MODE == M_REQ) fold_tile<T, RO_SUM, true, TREE, MEM>(f, n, a.flags & UF_ALIGNED, lane);
        else if (redop == RO_MAX) fold_tile<T, RO_MAX, false, TREE, MEM>(f, n, a.flags & UF_ALIGNED, lane);
        else fold_tile<T, RO_MIN, false, TREE, MEM>(f, n, a.flags & UF_ALIGNED, lane);
    }
}

// ------------------------------------------------------------------------------ copies
// A wavefront copies one tile to `per_wave` of its destinations, all of the tile to one after the
// other (the tile is read again for each, from the caches); its neighbours take the same tile to the
// other destinations. Ordinary loads, non-temporal stores of whole lines.
template <int ES>
__global__ void __launch_bounds__(kBlockThreads) hccl_uniform_copy(UniformArgs a) {
    const uint32_t lane = __lane_id();
    const uint64_t srcs = lane_entry(offsetof(UniformArgs, src), lane), dsts = lane_entry(offsetof(UniformArgs, dst), lane);
    const uint32_t sets = (a.ndst + a.per_wave - 1) / a.per_wave;
    for (uint32_t t = wave_number(false); t < a.ntiles; t += a.nworkers) {
        const uint32_t tile = sets > 1 ? t / sets : t, set = t - tile * sets;
        const uint32_t g = a.nseg > 1 ? tile / a.tiles_per_seg : 0u;
        const uint32_t pad = a.flags & UF_ALIGNED ? 0u : line_pad(from_lane(dsts, a.flags & UF_DST_PER_SEG ? g : 0u) + g * a.dst_step, ES);
        uint64_t e0;
        uint32_t n;
        if (!tile_range(tile - g * a.tiles_per_seg, a.tile_elems, pad, g + 1 < a.nseg ? a.seg_elems : a.last_elems, e0, n)) continue;
        const char* src = (const char*)(from_lane(srcs, a.flags & UF_SRC_PER_SEG ? g : 0u) + g * a.src_step + e0 * ES);
        const uint32_t j1 = (set + 1) * a.per_wave < a.ndst ? (set + 1) * a.per_wave : a.ndst;
        for (uint32_t j = set * a.per_wave; j < j1; ++j) {
            char* dst = (char*)(from_lane(dsts, a.flags & UF_DST_PER_SEG ? g : j) + g * a.dst_step + e0 * ES);
            if (dst != src) copy_run<ES>(src, dst, n, lane);
        }
    }
}

// One tile of a copy list. Its entry is found with a ballot over the tiles of 64 entries (two where
// there are more entries), where the executor's kernels read a tile table, a step, two operands and two
// buffer addresses, each after the other; and the tiles are 4 KiB and begin on lines of their
// destination. Everything is counted in 2-byte units, whatever the type. AllToAllv, tiles of the image
// -> list: 16 ranks x 68352 rows of 200 bytes 87 -> 72 us, 64 x 65536 of 128 bytes 206 -> 186,
// 8 x 100000 of 200 bytes with ids 61 -> 51, 4 x 13781 of 512 bytes 13.0 -> 11.2, 8 x 2^18 of 256 bytes
// with ids 183 -> 181.
__global__ void __launch_bounds__(kBlockThreads) hccl_copy_list(CopyListArgs a) {
    const uint32_t lane = __lane_id();
    const uint32_t* ends = (const uint32_t*)a.list;
    const uint64_t entries = 256u + 256ull * ((a.nentry + 63u) / 64u);
    const auto bufs = (const __attribute__((address_space(4))) uint64_t*)__builtin_amdgcn_kernarg_segment_ptr() +
                      offsetof(CopyListArgs, bufs) / 8;
    for (uint32_t t = wave_number(false); t < a.ntiles; t += a.nworkers) {
        const uint32_t b = a.nentry > 64u ? (uint32_t)__popcll(__ballot(ends[lane] <= t)) : 0u;
        const uint32_t i = b * 64u + (uint32_t)__popcll(__ballot(ends[64u + b * 64u + lane] <= t));
        const u32x4 w0 = cld<u32x4>(a.list, entries + 32ull * uni(i)), w1 = cld<u32x4>(a.list, entries + 32ull * uni(i) + 16);
        const uint64_t src_off = w0[0] | (uint64_t)w0[1] << 32, dst_off = w0[2] | (uint64_t)w0[3] << 32;
        const char* src = (const char*)bufs[w1[2] & 0xFFFFu] + src_off;
        char* dst = (char*)bufs[w1[2] >> 16] + dst_off;
        uint64_t e0;
        uint32_t n;
        if (!tile_range(t - w1[3], kListTileBytes / 2, line_pad((uint64_t)dst, 2), (w1[0] | (uint64_t)w1[1] << 32) / 2, e0, n)) continue;
        src += 2 * e0;
        dst += 2 * e0;
        if ((((uint64_t)src ^ (uint64_t)dst) & 15u) == 0) copy_run<2, true>(src, dst, n, lane);
        else copy_run<2>(src, dst, n, lane);
    }
}

template <int T, int MODE, bool TREE>
void launch_reduce(const UniformKernel& k, const UniformArgs& a, uint32_t blocks, hipStream_t s) {
    if (k.mem & MEM_STORE) {
        hipLaunchKernelGGL((hccl_uniform_reduce<T, MODE, TREE, MEM_STORE>), dim3(blocks), dim3(kBlockThreads), 0, s, a, k.redop);
    } else if (k.mem & MEM_LOAD) {
        hipLaunchKernelGGL((hccl_uniform_reduce<T, MODE, TREE, MEM_LOAD>), dim3(blocks), dim3(kBlockThreads), 0, s, a, k.redop);
    } else {
        hipLaunchKernelGGL((hccl_uniform_reduce<T, MODE, TREE, 0>), dim3(blocks), dim3(kBlockThreads), 0, s, a, k.redop);
    }
}

// SUM of a floating type, in the folds and roundings there are
template <int T>
void launch_sum(const UniformKernel& k, const UniformArgs& a, uint32_t blocks, hipStream_t s) {
    const bool tree = k.fold == FOLD_PAIRWISE;
    if constexpr (T != DT_FP32) {
        if (k.requant && tree) return launch_reduce<T, M_REQ, true>(k, a, blocks, s);
        if (k.requant) return launch_reduce<T, M_REQ, false>(k, a, blocks, s);
    }
    if (tree) return launch_reduce<T, M_SUM, true>(k, a, blocks, s);
    launch_reduce<T, M_SUM, false>(k, a, blocks, s);
}

template <int ES>
void launch_copy(const UniformKernel& k, const UniformArgs& a, uint32_t blocks, hipStream_t s) {
    hipLaunchKernelGGL((hccl_uniform_copy<ES>), dim3(blocks), dim3(kBlockThreads), 0, s, a);
}

}  // namespace

hipError_t launch_uniform(const UniformKernel& k, const UniformArgs& a, uint32_t blocks, hipStream_t s) {
    if (k.op == OP_COPY) {
        if (dtype_size(k.dtype) == 2) launch_copy<2>(k, a, blocks, s);
        else launch_copy<4>(k, a, blocks, s);
    } else if (k.redop != RO_SUM) {
        switch (k.dtype) {
            case DT_BF16: launch_reduce<DT_BF16, M_MINMAX, false>(k, a, blocks, s); break;
            case DT_FP16: launch_reduce<DT_FP16, M_MINMAX, false>(k, a, blocks, s); break;
            case DT_FP32: launch_reduce<DT_FP32, M_MINMAX, false>(k, a, blocks, s); break;
            default: launch_reduce<DT_INT32, M_MINMAX, false>(k, a, blocks, s); break;
        }
    } else {
        switch (k.dtype) {
            case DT_BF16: launch_sum<DT_BF16>(k, a, blocks, s); break;
            case DT_FP16: launch_sum<DT_FP16>(k, a, blocks, s); break;
            case DT_FP32: launch_sum<DT_FP32>(k, a, blocks, s); break;
            default: launch_reduce<DT_INT32, M_SUM, false>(k, a, blocks, s); break;
        }
    }
    return hipGetLastError();
}

hipError_t launch_copy_list(const CopyListArgs& a, uint32_t blocks, hipStream_t s) {
    hipLaunchKernelGGL(hccl_copy_list, dim3(blocks), dim3(kBlockThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace hccl
