// compiler.cpp -- lowering, fusion and packing of descriptor programs (host only).
//
// Lowerings write out the schedules the paper describes (Section III-B-2: the ring AllReduce
// built from per-hop receive/compute/send steps with dependencies; Section V-D: topology-
// aware two-level schedules that keep most traffic inside a group of consecutive ranks).
// On one GPU a "send" from rank a to rank b is a read of a's buffer by the step that writes
// b's buffer, so a hop becomes a COPY or REDUCE descriptor with a dependency id on the step
// that produced its input.
//
// Every reduction visits contributors in ascending rank order (two-level: ascending inside
// each group, then ascending over groups), so results never depend on the schedule.
#include "compiler.h"

#include <algorithm>
#include <cstring>
#include <list>
#include <unordered_map>

namespace hccl {

namespace {

constexpr uint64_t kDefaultChunkBytes = 1ull << 20;
// Tile defaults measured on MI355X: copies move 8 KiB per ticket; reductions read 32 KiB
// per ticket but never less than 1024 elements (wide two-level steps).
constexpr uint32_t kDefaultCopyTileBytes = 8u * 1024u;
constexpr uint32_t kDefaultReduceTileBytes = 32u * 1024u;
constexpr uint64_t kMinReduceTileElems = 1024;
// Programs with dependencies pay a release fence per signalling tile: larger tiles. A small
// dependent program (a few chains of long steps) would then leave most wavefronts idle, so its
// tiles are halved, down to 32 KiB read, until it has at least kDependentMinTiles (measured on
// the ring all-reduce P=4 x 2^20 fp32, 64 KiB chunks, unfused: 384 tiles 117 us, 1536 tiles
// 93 us; 3072 tiles 133 us and smaller ones slower still, as fences multiply).
constexpr uint32_t kDefaultDependentTileBytes = 128u * 1024u;
constexpr uint32_t kMinDependentTileBytes = 32u * 1024u;
constexpr uint64_t kDependentMinTiles = 1024;
// A copy to this many destinations or more reads up to 32 KiB per tile, as long as its phase
// keeps about 256 tiles: each tile writes its bytes to every destination, so a few long tiles
// beat many short ones. Measured with one wavefront per tile on the copy phase of the two-level
// all-reduce of 64 ranks (every 1/64 sub-shard to 63 ranks): tiles of the phase's bytes / 1024
// -> / 256 took 8 MiB per rank 222 -> 183 us, 4 MiB 109 -> 102 us; at 32 MiB per rank 32 KiB
// tiles (1 024) 736-754 us against 64 KiB 745-762 us and 128 KiB 819-836 us; the all-gather of
// P = 64 x 512 KiB bf16 blocks 396-400 us with 32 KiB tiles, 418-424 with 64 KiB, 543-550 with
// 128 KiB, 515-525 with 8 KiB.
constexpr size_t kWideCopyDsts = 8;
constexpr uint64_t kWideCopyTileBytes = 32u * 1024u;
constexpr uint64_t kWideCopyTargetTiles = 256;
// Small collectives are latency bound: cut them into at least this many tiles (down to
// one vector per lane) so that many wavefronts share the work.
constexpr uint64_t kSmallTargetTiles = 2048;
constexpr uint32_t kWaveStepElems = kWaveSize * kVecElems;  // 512: one vector per lane
constexpr uint64_t kShardAlignElems = 64;                      // 128 B of bf16, 256 B of fp32
// Static tiles (slots) of the copy step of an AllToAllvDynamic: slot k moves dynamic tiles k,
// k + slots, ... Every slot plans the exchange itself, so more slots cost more for an exchange
// far below its capacities, while fewer leave each slot a longer run of tiles. The launch has
// one wavefront per slot; rows + ids of the 8-rank 2^18-row exchange, full / all counts zero:
// 4 096 + 1 088 slots 197-198 / 8 us, 16 384 + 1 088 194 / 14 us, 32 768 + 1 088 192-193 /
// 23-24 us, 65 536 + 1 088 190 / 44 us.
constexpr uint32_t kDynamicSlots = 32768;

// Type of partials that leave registers: FP32 for floating sums (one rounding at the end),
// the buffer type when every partial is re-quantised, or for MAX / MIN (exact in any type).
uint32_t acc_dtype(const CollectiveSpec& s) {
    if (s.dtype == DT_INT32) return DT_INT32;
    if (s.redop != RO_SUM || s.requant) return (uint32_t)s.dtype;
    return DT_FP32;
}

bool is_pow2(int v) { return v > 0 && (v & (v - 1)) == 0; }

// Contributors of an element of shard (or block) c in fold order.
std::vector<int> contributor_order(const CollectiveSpec& s, int c) {
    const int P = s.P;
    std::vector<int> v(P);
    for (int k = 0; k < P; ++k) {
        if (s.order == ORDER_RING) {
            v[k] = (c + 1 + k) % P;
        } else if (s.order == ORDER_HALVING) {
            int r = 0;  // bit reversal of k: adjacent list entries differ in bit P/2, pairs of
            for (int b = 1, t = P >> 1; b < P; b <<= 1, t >>= 1)  // pairs in bit P/4, ...
                if (k & b) r |= t;
            v[k] = r;
        } else {
            v[k] = k;
        }
    }
    return v;
}

uint64_t chunk_elems(const CollectiveSpec& s) {
    uint64_t bytes = s.chunk_bytes ? s.chunk_bytes : kDefaultChunkBytes;
    uint64_t c = bytes / dtype_size(s.dtype);
    c = (c / kShardAlignElems) * kShardAlignElems;
    return std::max<uint64_t>(c, kShardAlignElems);
}

Operand opnd(uint32_t buf, uint32_t dtype, uint64_t elem_offset) {
    Operand o;
    o.buf = buf;
    o.dtype = dtype;
    o.offset = elem_offset * dtype_size(dtype);
    return o;
}

struct Builder {
    HostProgram& prog;
    uint32_t add(uint8_t op, uint8_t redop, uint64_t nelem, std::vector<Operand> srcs,
                 std::vector<Operand> dsts, std::vector<Dep> deps = {}, uint16_t group = 0) {
        HostDesc d;
        d.op = op;
        d.redop = redop;
        d.nelem = nelem;
        d.group = group;
        d.srcs = std::move(srcs);
        d.dsts = std::move(dsts);
        d.deps = std::move(deps);
        prog.descs.push_back(std::move(d));
        return (uint32_t)(prog.descs.size() - 1);
    }
};

Dep tile_dep(uint32_t d) { return Dep{d, DEP_TILE, 0, 0}; }

template <typename F>
void for_chunks(uint64_t begin, uint64_t end, uint64_t C, F&& f) {
    uint32_t j = 0;
    for (uint64_t o = begin; o < end; o += C, ++j) f(j, o, std::min(C, end - o));
}

// ---------------------------------------------------------------------------- DIRECT
// One step per chunk: read every contributor, write every destination (the one-shot,
// all-to-all style schedule of the PE collective kernels for small messages, Section V-F-3).
void lower_direct(const CollectiveSpec& s, HostProgram& p) {
    Builder b{p};
    const int P = s.P;
    const uint64_t C = chunk_elems(s);
    const uint32_t dt = (uint32_t)s.dtype;
    const uint32_t fold = (s.order == ORDER_HALVING) ? FOLD_PAIRWISE : FOLD_LIST;
    auto reduce_step = [&](uint64_t n, const std::vector<int>& order, uint64_t src_elem, std::vector<Operand> dst) {
        std::vector<Operand> src;
        for (int r : order) src.push_back(opnd(send_buf(r), dt, src_elem));
        uint32_t i = b.add(OP_REDUCE, (uint8_t)s.redop, n, src, std::move(dst));
        p.descs[i].fold = fold;
    };
    if (s.coll == COLL_ALLREDUCE) {
        // the ring order rotates per shard, so chunks never straddle a shard boundary then
        const uint64_t q = (s.order == ORDER_RING) ? shard_size(s.count, P) : s.count;
        for (uint64_t lo = 0, c = 0; lo < s.count; lo += q, ++c) {
            const std::vector<int> order = contributor_order(s, (int)c);
            for_chunks(lo, std::min(s.count, lo + q), C, [&](uint32_t, uint64_t o, uint64_t n) {
                std::vector<Operand> dst;
                for (int r = 0; r < P; ++r) dst.push_back(opnd(recv_buf(P, r), dt, o));
                reduce_step(n, order, o, dst);
            });
        }
    } else if (s.coll == COLL_REDUCE_SCATTER) {
        const uint64_t M = s.count;
        for (int c = 0; c < P; ++c) {
            const std::vector<int> order = contributor_order(s, c);
            for_chunks(0, M, C, [&](uint32_t, uint64_t o, uint64_t n) {
                reduce_step(n, order, (uint64_t)c * M + o, {opnd(recv_buf(P, c), dt, o)});
            });
        }
    } else if (s.coll == COLL_ALLGATHER) {
        const uint64_t M = s.count;
        for (int q = 0; q < P; ++q) {
            for_chunks(0, M, C, [&](uint32_t, uint64_t o, uint64_t n) {
                std::vector<Operand> dst;
                for (int r = 0; r < P; ++r) dst.push_back(opnd(recv_buf(P, r), dt, (uint64_t)q * M + o));
                b.add(OP_COPY, RO_SUM, n, {opnd(send_buf(q), dt, o)}, dst);
            });
        }
    }
    p.algo = ALGO_DIRECT;
}

// ------------------------------------------------------------------------------ RING
// Reduce chain of one chunk: step t (t = 1 .. P-1) folds contributor t into the partial of
// contributors 0 .. t-1. Partials live in scratch in the accumulation type; the last step
// rounds into `final_dst`. Steps of all chunks are emitted step-major so every chunk's step
// t is available while step t+1 waits only for the same tile of its own chain.
struct Chain {
    int owner = 0;        // shard / block the chain reduces (fixes the ring order's start)
    uint64_t src_elem;    // element offset of the chunk in every send buffer
    uint64_t nelem;
    Operand final_dst;
    uint64_t scratch_elem;  // element offset of the partial in scratch (accumulation type)
    uint32_t last = 0;      // descriptor of the final step
    uint32_t prev = 0;
};

void emit_reduce_chains(const CollectiveSpec& s, HostProgram& p, std::vector<Chain>& chains) {
    Builder b{p};
    const int P = s.P;
    const uint32_t dt = (uint32_t)s.dtype;
    const uint32_t acc = acc_dtype(s);
    if (P == 1) {
        for (auto& ch : chains)
            ch.last = b.add(OP_REDUCE, (uint8_t)s.redop, ch.nelem, {opnd(send_buf(0), dt, ch.src_elem)},
                            {ch.final_dst});
        return;
    }
    std::vector<std::vector<int>> order(P);
    for (int c = 0; c < P; ++c) order[c] = contributor_order(s, c);
    for (int t = 1; t < P; ++t) {
        for (auto& ch : chains) {
            const std::vector<int>& seq = order[ch.owner];
            Operand partial = opnd(scratch_buf(P), acc, ch.scratch_elem);
            std::vector<Operand> src;
            if (t == 1) src.push_back(opnd(send_buf(seq[0]), dt, ch.src_elem));
            else src.push_back(partial);
            src.push_back(opnd(send_buf(seq[t]), dt, ch.src_elem));
            Operand dst = (t == P - 1) ? ch.final_dst : partial;
            std::vector<Dep> deps;
            if (t > 1) deps.push_back(tile_dep(ch.prev));
            ch.prev = b.add(OP_REDUCE, (uint8_t)s.redop, ch.nelem, src, {dst}, deps);
            if (t == P - 1) ch.last = ch.prev;
        }
    }
}

void lower_ring(const CollectiveSpec& s, HostProgram& p) {
    Builder b{p};
    const int P = s.P;
    const uint64_t C = chunk_elems(s);
    const uint32_t dt = (uint32_t)s.dtype;
    const uint32_t acc = acc_dtype(s);

    if (s.coll == COLL_ALLGATHER) {
        // hop 0 places block q in rank q's output; hop h forwards it from rank q+h-1 to q+h.
        const uint64_t M = s.count;
        struct Hop { int q; uint64_t o, n; uint32_t prev; };
        std::vector<Hop> hops;
        for (int q = 0; q < P; ++q)
            for_chunks(0, M, C, [&](uint32_t, uint64_t o, uint64_t n) { hops.push_back({q, o, n, 0}); });
        for (auto& h : hops)
            h.prev = b.add(OP_COPY, RO_SUM, h.n, {opnd(send_buf(h.q), dt, h.o)},
                           {opnd(recv_buf(P, h.q), dt, (uint64_t)h.q * M + h.o)});
        for (int step = 1; step < P; ++step) {
            for (auto& h : hops) {
                int from = (h.q + step - 1) % P, to = (h.q + step) % P;
                uint64_t at = (uint64_t)h.q * M + h.o;
                h.prev = b.add(OP_COPY, RO_SUM, h.n, {opnd(recv_buf(P, from), dt, at)},
                               {opnd(recv_buf(P, to), dt, at)}, {tile_dep(h.prev)});
            }
        }
        p.algo = ALGO_RING;
        return;
    }

    std::vector<Chain> chains;
    std::vector<int> owner;
    if (s.coll == COLL_REDUCE_SCATTER) {
        const uint64_t M = s.count;
        for (int c = 0; c < P; ++c)
            for_chunks(0, M, C, [&](uint32_t, uint64_t o, uint64_t n) {
                Chain ch;
                ch.owner = c;
                ch.src_elem = (uint64_t)c * M + o;
                ch.nelem = n;
                ch.final_dst = opnd(recv_buf(P, c), dt, o);
                ch.scratch_elem = (uint64_t)c * M + o;
                chains.push_back(ch);
                owner.push_back(c);
            });
        p.scratch_bytes = (P > 2) ? (uint64_t)P * M * dtype_size(acc) : 0;
    } else {  // allreduce: owner c reduces shard c, then the result travels around the ring
        const uint64_t q = shard_size(s.count, P);
        for (int c = 0; c < P; ++c) {
            uint64_t lo = std::min(s.count, (uint64_t)c * q), hi = std::min(s.count, lo + q);
            for_chunks(lo, hi, C, [&](uint32_t, uint64_t o, uint64_t n) {
                Chain ch;
                ch.owner = c;
                ch.src_elem = o;
                ch.nelem = n;
                ch.final_dst = opnd(recv_buf(P, c), dt, o);
                ch.scratch_elem = o;
                chains.push_back(ch);
                owner.push_back(c);
            });
        }
        p.scratch_bytes = (P > 2) ? s.count * dtype_size(acc) : 0;
    }
    emit_reduce_chains(s, p, chains);

    if (s.coll == COLL_ALLREDUCE) {
        for (int step = 1; step < P; ++step) {
            for (size_t i = 0; i < chains.size(); ++i) {
                Chain& ch = chains[i];
                int from = (owner[i] + step - 1) % P, to = (owner[i] + step) % P;
                ch.last = b.add(OP_COPY, RO_SUM, ch.nelem, {opnd(recv_buf(P, from), dt, ch.src_elem)},
                                {opnd(recv_buf(P, to), dt, ch.src_elem)}, {tile_dep(ch.last)});
            }
        }
    }
    p.algo = ALGO_RING;
}

// ------------------------------------------------------------------------------- RHD
// Recursive halving reduce-scatter (and recursive doubling all-gather) for P = 2^L ranks.
// The vector is cut into P blocks; block b ends at rank b. At halving step j (distance
// d = P >> (j+1)) rank r keeps the blocks that agree with r on every bit handled so far; for
// each kept block it combines its own value with the value of partner r ^ d, which kept the
// same block one step earlier. Partials live in scratch slot (r, b) in the accumulation type;
// the last step writes the owner's receive buffer. The tree this builds for every element
// pairs ranks differing in bit P/2 first, then bit P/4, ..., then bit 1. Doubling step j
// (distance d = 1 << j) copies the d blocks a rank holds to its partner r ^ d.
void lower_rhd(const CollectiveSpec& s, HostProgram& p) {
    Builder b{p};
    const int P = s.P;
    const uint64_t C = chunk_elems(s);
    const uint32_t dt = (uint32_t)s.dtype;
    const uint32_t acc = acc_dtype(s);
    const bool ag_only = s.coll == COLL_ALLGATHER;
    // block geometry: element offset of block b in a send buffer / in a receive buffer
    const uint64_t N = s.count;
    const uint64_t q = (s.coll == COLL_ALLREDUCE) ? shard_size(N, P) : N;
    auto blo = [&](int blk) { return std::min<uint64_t>((uint64_t)blk * q, s.coll == COLL_ALLREDUCE ? N : (uint64_t)P * N); };
    auto bhi = [&](int blk) { return std::min<uint64_t>(blo(blk) + q, s.coll == COLL_ALLREDUCE ? N : (uint64_t)P * N); };
    // receive-side element offset of block b: all-reduce and all-gather keep the send layout;
    // reduce-scatter writes its block at offset 0 of the owner's buffer
    auto rlo = [&](int blk) { return s.coll == COLL_REDUCE_SCATTER ? 0 : blo(blk); };

    // producer of the value rank r holds for (block, chunk offset), per step
    std::vector<std::unordered_map<uint64_t, uint32_t>> prev(P), next(P);
    auto key = [&](int blk, uint64_t o) { return ((uint64_t)blk << 40) | (o - blo(blk)); };

    if (!ag_only) {
        int steps = 0;
        while ((1 << steps) < P) ++steps;
        uint64_t mask = 0;
        for (int j = 0; j < steps; ++j) {
            const int d = P >> (j + 1);
            mask |= (uint64_t)d;
            for (int r = 0; r < P; ++r) next[r].clear();
            for (int r = 0; r < P; ++r) {
                const int partner = r ^ d;
                for (int blk = 0; blk < P; ++blk) {
                    if (((uint64_t)blk & mask) != ((uint64_t)r & mask)) continue;
                    const bool last = (j == steps - 1);
                    for_chunks(blo(blk), bhi(blk), C, [&](uint32_t, uint64_t o, uint64_t n) {
                        const uint64_t so = (uint64_t)(r * P + blk) * q + (o - blo(blk));
                        const uint64_t po = (uint64_t)(partner * P + blk) * q + (o - blo(blk));
                        std::vector<Operand> src;
                        std::vector<Dep> deps;
                        if (j == 0) {
                            src.push_back(opnd(send_buf(r), dt, o));
                            src.push_back(opnd(send_buf(partner), dt, o));
                        } else {
                            src.push_back(opnd(scratch_buf(P), acc, so));
                            src.push_back(opnd(scratch_buf(P), acc, po));
                            deps.push_back(tile_dep(prev[r].at(key(blk, o))));
                            deps.push_back(tile_dep(prev[partner].at(key(blk, o))));
                        }
                        Operand dst = last ? opnd(recv_buf(P, r), dt, rlo(blk) + (o - blo(blk)))
                                           : opnd(scratch_buf(P), acc, so);
                        next[r][key(blk, o)] = b.add(OP_REDUCE, (uint8_t)s.redop, n, src, {dst}, deps);
                    });
                }
            }
            prev.swap(next);
        }
        p.scratch_bytes = (steps > 1) ? (uint64_t)P * P * q * dtype_size(acc) : 0;
        if (P == 1) {
            for_chunks(blo(0), bhi(0), C, [&](uint32_t, uint64_t o, uint64_t n) {
                prev[0][key(0, o)] = b.add(OP_REDUCE, (uint8_t)s.redop, n, {opnd(send_buf(0), dt, o)},
                                           {opnd(recv_buf(P, 0), dt, rlo(0) + (o - blo(0)))});
            });
        }
    } else {
        // all-gather: every rank first places its own block
        for (int r = 0; r < P; ++r)
            for_chunks(0, N, C, [&](uint32_t, uint64_t o, uint64_t n) {
                prev[r][key(r, (uint64_t)r * N + o)] =
                    b.add(OP_COPY, RO_SUM, n, {opnd(send_buf(r), dt, o)}, {opnd(recv_buf(P, r), dt, (uint64_t)r * N + o)});
            });
    }

    if (s.coll != COLL_REDUCE_SCATTER) {
        // doubling: at distance d, rank r holds the d blocks of its aligned group and sends them
        for (int d = 1; d < P; d <<= 1) {
            for (int r = 0; r < P; ++r) next[r] = prev[r];
            for (int r = 0; r < P; ++r) {
                const int partner = r ^ d;
                const int base = r & ~(d - 1);
                for (int blk = base; blk < base + d; ++blk) {
                    for_chunks(blo(blk), bhi(blk), C, [&](uint32_t, uint64_t o, uint64_t n) {
                        const uint32_t src_desc = prev[r].at(key(blk, o));
                        next[partner][key(blk, o)] =
                            b.add(OP_COPY, RO_SUM, n, {opnd(recv_buf(P, r), dt, o)}, {opnd(recv_buf(P, partner), dt, o)},
                                  {tile_dep(src_desc)});
                    });
                }
            }
            prev.swap(next);
        }
    }
    p.algo = ALGO_RHD;
}

// ------------------------------------------------------------------------- TWO_LEVEL
// P = G groups x L consecutive ranks. Shard k of the vector belongs to local rank k of every
// group and is cut into G sub-shards; sub-shard (k, g) is owned by local rank k of group g.
// Phase 1 (inside each group, reduce-scatter): the L contributors of every element are folded
// into an FP32 partial per group. Phase 2 (across groups, the all-reduce of shard k among the
// local-k ranks as reduce-scatter + all-gather): the G partials of sub-shard (k, g) are folded
// in ascending group order, rounded, and written to its owner; the owner forwards it to local
// rank k of the other groups. Phase 3 (inside each group, all-gather): local rank k forwards
// shard k to the other L-1 ranks of its group.
void lower_two_level(const CollectiveSpec& s, HostProgram& p) {
    Builder b{p};
    const int P = s.P, L = s.group_size, G = P / L;
    const uint64_t N = s.count, C = chunk_elems(s);
    const uint32_t dt = (uint32_t)s.dtype;
    const uint32_t acc = acc_dtype(s);
    const uint64_t q = shard_size(N, L);
    struct Piece { int k, g; uint64_t o, n; };
    std::vector<Piece> pieces;
    for (int k = 0; k < L; ++k) {
        const uint64_t lo = std::min(N, (uint64_t)k * q), hi = std::min(N, lo + q);
        const uint64_t qs = shard_size(hi - lo, G);
        for (int g = 0; g < G; ++g) {
            const uint64_t slo = std::min(hi, lo + (uint64_t)g * qs), shi = std::min(hi, slo + qs);
            for_chunks(slo, shi, C, [&](uint32_t, uint64_t o, uint64_t n) { pieces.push_back({k, g, o, n}); });
        }
    }
    auto rank = [&](int g, int m) { return g * L + m; };
    std::vector<std::vector<uint32_t>> rs(pieces.size(), std::vector<uint32_t>(G));
    for (int h = 0; h < G; ++h) {
        for (size_t i = 0; i < pieces.size(); ++i) {
            const Piece& pc = pieces[i];
            std::vector<Operand> src;
            for (int m = 0; m < L; ++m) src.push_back(opnd(send_buf(rank(h, m)), dt, pc.o));
            rs[i][h] = b.add(OP_REDUCE, (uint8_t)s.redop, pc.n, src,
                             {opnd(scratch_buf(P), acc, (uint64_t)h * N + pc.o)});
        }
    }
    std::vector<uint32_t> inter(pieces.size()), fwd(pieces.size());
    for (size_t i = 0; i < pieces.size(); ++i) {
        const Piece& pc = pieces[i];
        std::vector<Operand> src;
        std::vector<Dep> deps;
        for (int h = 0; h < G; ++h) {
            src.push_back(opnd(scratch_buf(P), acc, (uint64_t)h * N + pc.o));
            deps.push_back(tile_dep(rs[i][h]));
        }
        inter[i] = b.add(OP_REDUCE, (uint8_t)s.redop, pc.n, src, {opnd(recv_buf(P, rank(pc.g, pc.k)), dt, pc.o)}, deps);
    }
    for (size_t i = 0; i < pieces.size(); ++i) {
        const Piece& pc = pieces[i];
        fwd[i] = inter[i];
        if (G == 1) continue;
        std::vector<Operand> dst;
        for (int h = 0; h < G; ++h)
            if (h != pc.g) dst.push_back(opnd(recv_buf(P, rank(h, pc.k)), dt, pc.o));
        fwd[i] = b.add(OP_COPY, RO_SUM, pc.n, {opnd(recv_buf(P, rank(pc.g, pc.k)), dt, pc.o)}, dst,
                       {tile_dep(inter[i])});
    }
    if (L > 1) {
        for (int h = 0; h < G; ++h) {
            for (size_t i = 0; i < pieces.size(); ++i) {
                const Piece& pc = pieces[i];
                std::vector<Operand> dst;
                for (int m = 0; m < L; ++m)
                    if (m != pc.k) dst.push_back(opnd(recv_buf(P, rank(h, m)), dt, pc.o));
                b.add(OP_COPY, RO_SUM, pc.n, {opnd(recv_buf(P, rank(h, pc.k)), dt, pc.o)}, dst,
                      {tile_dep(h == pc.g ? inter[i] : fwd[i])});
            }
        }
    }
    p.scratch_bytes = (uint64_t)G * N * dtype_size(acc);
    p.algo = ALGO_TWO_LEVEL;
}

// ------------------------------------------------------------------------- ALLTOALLV
// Every non-empty (source, destination) block becomes COPY steps of at most one chunk; the
// steps are ordered largest first so the long blocks start early (Section IV-A: AllToAllv
// spread across parallel engines), and equal ones destination by destination: launches start
// their tiles in program order, so at any moment the chip fills one receive buffer in order
// while it reads from every send buffer (grouped AllToAllv of 8 ranks x 2^18 embedding rows,
// source-major 182.8-184.2 us, destination-major 181.0-182.5 us).
void lower_alltoallv(const CollectiveSpec& s, HostProgram& p) {
    Builder b{p};
    const int P = s.P;
    const uint32_t dt = (uint32_t)s.dtype;
    const uint64_t C = chunk_elems(s);
    struct Piece { int src, dst; uint64_t so, ro, n; };
    std::vector<Piece> pieces;
    for (int dst = 0; dst < P; ++dst) {
        for (int src = 0; src < P; ++src) {
            uint64_t n = s.sendcounts[(size_t)src * P + dst];
            uint64_t so = s.sdispls[(size_t)src * P + dst];
            uint64_t ro = s.rdispls[(size_t)dst * P + src];
            for (uint64_t o = 0; o < n; o += C) pieces.push_back({src, dst, so + o, ro + o, std::min(C, n - o)});
        }
    }
    std::stable_sort(pieces.begin(), pieces.end(), [](const Piece& a, const Piece& c) { return a.n > c.n; });
    p.descs.reserve(pieces.size());
    for (const Piece& pc : pieces)
        b.add(OP_COPY, RO_SUM, pc.n, {opnd(send_buf(pc.src), dt, pc.so)}, {opnd(recv_buf(P, pc.dst), dt, pc.ro)});
    p.algo = ALGO_DIRECT;
}

// ------------------------------------------------------------------ ALLTOALLV DYNAMIC
// Device-resident AllToAllv (Section IV-B-2): the host compiles the program once for the
// capacities, and the layout is worked out on the device when it runs. The program is one
// step of `slots` tiles; each slot reads the count matrix (and the explicit offsets, if given)
// from device memory, checks the whole layout, and moves its share of the rows. Nothing on the
// host depends on the counts, and no slot waits for another.
void lower_alltoallv_dynamic(const CollectiveSpec& s, HostProgram& p) {
    const int P = s.P;
    DynA2A a;
    std::memset(&a, 0, sizeof a);
    a.P = (uint32_t)P;
    a.elem_bytes = dtype_size(s.dtype);
    a.send0 = send_buf(0);
    a.recv0 = recv_buf(P, 0);
    a.counts = meta_buf(P, META_COUNTS);
    a.sdispls = s.dyn_sdispls ? meta_buf(P, META_SDISPLS) : kNoBuffer;
    a.rdispls = s.dyn_rdispls ? meta_buf(P, META_RDISPLS) : kNoBuffer;
    a.recvcounts = s.dyn_recvcounts ? meta_buf(P, META_RECVCOUNTS) : kNoBuffer;
    a.row_elems = s.row_elems;
    a.send_cap = s.send_cap;
    a.recv_cap = s.recv_cap;
    a.tile_elems = dynamic_tile_elems(s);
    a.slots = dynamic_slots(s);
    p.aux.push_back(a);
    p.nmeta = kMetaPerDynamicCall;
    HostDesc copy;
    copy.op = OP_DYN_COPY;
    copy.aux = 0;
    p.descs.push_back(copy);
    p.algo = ALGO_DIRECT;
}

void dedupe_deps(HostDesc& d, uint32_t self) {
    std::vector<Dep> out;
    for (const Dep& e : d.deps) {
        if (e.desc == self) continue;
        bool merged = false;
        for (Dep& o : out) {
            if (o.desc == e.desc) {
                if (e.kind == DEP_ALL) o.kind = DEP_ALL;  // the stronger wait wins
                merged = true;
                break;
            }
        }
        if (!merged) out.push_back(e);
    }
    d.deps = std::move(out);
}

struct OperandKey {
    uint32_t buf;
    uint64_t offset;
    bool operator==(const OperandKey& o) const { return buf == o.buf && offset == o.offset; }
};
struct OperandKeyHash {
    size_t operator()(const OperandKey& k) const { return std::hash<uint64_t>()(k.offset * 131 + k.buf); }
};

// Scratch is needed only if some live step still touches it.
void drop_unused_scratch(HostProgram& p) {
    if (p.scratch_bytes == 0) return;
    const uint32_t scratch = scratch_buf(p.P);
    for (const HostDesc& d : p.descs) {
        if (!d.alive) continue;
        for (const auto* list : {&d.srcs, &d.dsts})
            for (const Operand& o : *list)
                if (o.buf == scratch) return;
    }
    p.scratch_bytes = 0;
}

}  // namespace

uint64_t shard_size(uint64_t n, int parts) {
    uint64_t q = (n + parts - 1) / parts;
    return ((q + kShardAlignElems - 1) / kShardAlignElems) * kShardAlignElems;
}

bool CollectiveSpec::operator==(const CollectiveSpec& o) const {
    return coll == o.coll && P == o.P && dtype == o.dtype && redop == o.redop && count == o.count &&
           sendcounts == o.sendcounts && sdispls == o.sdispls && recvcounts == o.recvcounts &&
           rdispls == o.rdispls && in_place == o.in_place && algo == o.algo && group_size == o.group_size &&
           chunk_bytes == o.chunk_bytes && fuse == o.fuse && tile_bytes == o.tile_bytes && order == o.order &&
           requant == o.requant && phases == o.phases && row_elems == o.row_elems && send_cap == o.send_cap && recv_cap == o.recv_cap &&
           dyn_sdispls == o.dyn_sdispls && dyn_rdispls == o.dyn_rdispls && dyn_recvcounts == o.dyn_recvcounts;
}

uint64_t dynamic_tile_elems(const CollectiveSpec& s) {
    const uint64_t tb = s.tile_bytes ? s.tile_bytes : kDefaultCopyTileBytes;
    const uint64_t te = (tb / dtype_size(s.dtype)) / kWaveStepElems * kWaveStepElems;
    return std::min<uint64_t>(std::max<uint64_t>(te, kWaveStepElems), 1ull << 30);
}

uint64_t dynamic_tile_bound(const CollectiveSpec& s) {
    // a source's pairs cover at most send_cap rows, and each pair adds at most one partial tile
    const uint64_t te = dynamic_tile_elems(s);
    const uint64_t per_source = (s.send_cap * s.row_elems + te - 1) / te + (uint64_t)s.P;
    return (uint64_t)s.P * per_source;
}

uint32_t dynamic_slots(const CollectiveSpec& s) {
    return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(kDynamicSlots, dynamic_tile_bound(s)));
}

int resolve_algo(const CollectiveSpec& s) {
    if (s.coll == COLL_ALLTOALLV || s.coll == COLL_ALLTOALLV_DYNAMIC) return ALGO_DIRECT;
    if (s.algo != ALGO_AUTO) return s.algo;
    if (s.order == ORDER_HALVING) return ALGO_RHD;
    if (s.coll == COLL_ALLREDUCE && s.order == ORDER_ASCENDING && s.group_size > 1 && s.group_size < s.P &&
        s.P % s.group_size == 0)
        return ALGO_TWO_LEVEL;
    return ALGO_RING;
}

BufferSizes buffer_sizes(const CollectiveSpec& s, uint64_t scratch_bytes) {
    BufferSizes b;
    const int P = s.P;
    const uint64_t es = dtype_size(s.dtype);
    b.bytes.assign((size_t)2 * P + 1, 0);
    for (int r = 0; r < P; ++r) {
        uint64_t sb = 0, rb = 0;
        switch (s.coll) {
            case COLL_ALLREDUCE: sb = rb = s.count * es; break;
            case COLL_REDUCE_SCATTER: sb = (uint64_t)P * s.count * es; rb = s.count * es; break;
            case COLL_ALLGATHER: sb = s.count * es; rb = (uint64_t)P * s.count * es; break;
            case COLL_ALLTOALLV_DYNAMIC: sb = s.send_cap * s.row_elems * es; rb = s.recv_cap * s.row_elems * es; break;
            default:
                for (int q = 0; q < P; ++q) {
                    sb = std::max(sb, (s.sdispls[(size_t)r * P + q] + s.sendcounts[(size_t)r * P + q]) * es);
                    rb = std::max(rb, (s.rdispls[(size_t)r * P + q] + s.recvcounts[(size_t)r * P + q]) * es);
                }
        }
        b.bytes[send_buf(r)] = sb;
        b.bytes[recv_buf(P, r)] = rb;
    }
    b.bytes[scratch_buf(P)] = scratch_bytes;
    return b;
}

bool lower(const CollectiveSpec& s, HostProgram& p, std::string& err) {
    p = HostProgram();
    p.P = s.P;
    p.phase_mode = s.phases;
    if (s.coll == COLL_ALLTOALLV) {
        lower_alltoallv(s, p);
        return true;
    }
    if (s.coll == COLL_ALLTOALLV_DYNAMIC) {
        if (s.P > kMaxRanks || s.row_elems == 0) {
            err = "alltoallv_dynamic needs 1..64 ranks and row_elems >= 1";
            return false;
        }
        if (dynamic_tile_bound(s) >= (1ull << 31)) {
            err = "alltoallv_dynamic capacities too large for one exchange";
            return false;
        }
        lower_alltoallv_dynamic(s, p);
        return true;
    }
    int algo = resolve_algo(s);
    if (s.order == ORDER_HALVING && !is_pow2(s.P)) {
        err = "the recursive-halving order needs a power-of-two number of ranks";
        return false;
    }
    if (s.order == ORDER_HALVING && algo != ALGO_RHD && algo != ALGO_DIRECT) {
        err = "the recursive-halving order is produced by the RHD or DIRECT schedules";
        return false;
    }
    if (algo == ALGO_RHD && s.order != ORDER_HALVING && s.coll != COLL_ALLGATHER) {
        err = "the RHD schedule folds in the recursive-halving order (set order = HALVING)";
        return false;
    }
    if (algo == ALGO_RHD && !is_pow2(s.P)) {
        err = "the RHD schedule needs a power-of-two number of ranks";
        return false;
    }
    if (algo == ALGO_TWO_LEVEL && s.order != ORDER_ASCENDING) {
        err = "the two-level schedule has its own grouped order";
        return false;
    }
    if (algo == ALGO_RHD) {
        lower_rhd(s, p);
    } else if (algo == ALGO_TWO_LEVEL) {
        if (s.coll != COLL_ALLREDUCE) {
            err = "the two-level schedule is defined for allreduce only";
            return false;
        }
        if (s.group_size < 1 || s.P % s.group_size != 0) {
            err = "group_size must divide nranks for the two-level schedule";
            return false;
        }
        lower_two_level(s, p);
    } else if (algo == ALGO_RING) {
        lower_ring(s, p);
    } else if (algo == ALGO_DIRECT) {
        lower_direct(s, p);
    } else {
        err = "unknown algorithm";
        return false;
    }
    if (s.requant && s.redop == RO_SUM && (s.dtype == DT_BF16 || s.dtype == DT_FP16))
        for (auto& d : p.descs)
            if (d.op == OP_REDUCE) d.requant = true;
    return true;
}

// ---------------------------------------------------------------------------- fusion
//
// Rule 1 (chain): B = REDUCE(partial, x...) where partial is the scratch output of REDUCE A
//   (its only destination) and B is the only step that reads that value  ->  B = REDUCE(A's
//   sources, x...). The fold is the same sequence of operations on the same values: A's
//   result was never rounded (it is in the accumulation type), B continued from it.
// Rule 2 (groups): E = REDUCE(p_0, ..., p_{G-1}) where every p_g is the scratch output of a
//   flat REDUCE D_g of L sources that only E reads  ->  E = REDUCE(all D_g sources,
//   group = L): fold each run of L into a partial, then fold the partials, as before.
// Rule 3 (forwarding): F = COPY(x -> y...) where x is the value a step E wrote (same
//   location and element count) and F waits for E  ->  E also writes y... . Except when E is a
//   wide reduction (kSplitMinSources or more sources) and the program splits them (by its phase
//   mode and size): then F stays a step of its own, a later phase that copies E's result once
//   it is complete, and a second such copy of the same value joins the first (F also writes
//   its destinations). Measured on the two-level all-reduce P = 64 x 32 MiB bf16: one step of
//   64 sources and 64 destinations 860 us; 64 sources to one destination, then one source to 63
//   destinations in a second launch, about 770 us.
// Rule 4 (trees): E = REDUCE(a, b) where a and b are the private partials of two binary-tree
//   reductions over equally many sources  ->  E = binary tree over both source lists. This
//   is what a recursive-halving level does; the tree, and so every operation, is unchanged.
// Steps merge only if they share the operator and the re-quantisation rule.
//
// Values are tracked by version: the producer of a source is the last step, in program
// order, that wrote exactly that location. Merged steps forward to the step that absorbed
// them, so later lookups and dependencies resolve to the surviving step.
void fuse(HostProgram& p) {
    const uint32_t scratch = scratch_buf(p.P);
    p.fused = true;
    // every rule merges a step with one that it waits for
    if (std::none_of(p.descs.begin(), p.descs.end(), [](const HostDesc& d) { return !d.deps.empty(); })) {
        drop_unused_scratch(p);
        return;
    }
    const uint32_t D = (uint32_t)p.descs.size();
    std::vector<uint32_t> fwd(D);
    for (uint32_t i = 0; i < D; ++i) fwd[i] = i;
    // whether the forwarding copies of wide reductions stay separate steps (by the bytes the
    // reductions read from the send buffers)
    uint64_t reduce_bytes = 0;
    for (const auto& d : p.descs)
        if (d.op == OP_REDUCE)
            for (const Operand& o : d.srcs)
                if (o.buf < (uint32_t)p.P) reduce_bytes += d.nelem * dtype_size(o.dtype);
    const bool split = p.phase_mode == PHASE_LEVELS || (p.phase_mode == PHASE_AUTO && reduce_bytes >= kSplitMinBytes);
    // split copies, by the value they read: a second copy of that value joins the first
    std::unordered_map<OperandKey, uint32_t, OperandKeyHash> split_copy;
    auto find = [&](uint32_t x) {
        while (fwd[x] != x) {
            fwd[x] = fwd[fwd[x]];
            x = fwd[x];
        }
        return x;
    };

    // producer of every source operand, and how many sources read each written value
    std::vector<std::vector<int64_t>> prod(D);
    std::vector<std::vector<uint32_t>> nread(D);
    {
        std::unordered_map<OperandKey, std::pair<uint32_t, uint32_t>, OperandKeyHash> last;
        size_t written = 0;
        for (const HostDesc& d : p.descs) written += d.dsts.size();
        last.reserve(written);
        for (uint32_t i = 0; i < D; ++i) {
            const HostDesc& d = p.descs[i];
            nread[i].assign(d.dsts.size(), 0);
            prod[i].assign(d.srcs.size(), -1);
            for (size_t k = 0; k < d.srcs.size(); ++k) {
                auto it = last.find({d.srcs[k].buf, d.srcs[k].offset});
                if (it == last.end()) continue;
                const HostDesc& w = p.descs[it->second.first];
                if (w.dsts[it->second.second].dtype != d.srcs[k].dtype || w.nelem != d.nelem) continue;
                prod[i][k] = it->second.first;
                nread[it->second.first][it->second.second] += 1;
            }
            for (size_t k = 0; k < d.dsts.size(); ++k) last[{d.dsts[k].buf, d.dsts[k].offset}] = {i, (uint32_t)k};
        }
    }
    auto depends_on = [&](const HostDesc& d, uint32_t target) {
        for (const Dep& e : d.deps)
            if (find(e.desc) == target) return true;
        return false;
    };
    // A is a partial step (scratch output, one destination) whose single value only B reads,
    // with the same operator and rounding rule as B
    auto partial_of = [&](int64_t a, const HostDesc& B) {
        if (a < 0) return false;
        const HostDesc& A = p.descs[a];
        return A.alive && A.op == OP_REDUCE && A.dsts.size() == 1 && A.dsts[0].buf == scratch &&
               A.redop == B.redop && A.requant == B.requant && A.nelem == B.nelem && nread[a][0] == 1 &&
               depends_on(B, (uint32_t)a);
    };
    // ... folded ascending over its list
    auto private_partial = [&](int64_t a, const HostDesc& B) {
        return partial_of(a, B) && p.descs[a].group == 0 && p.descs[a].fold == FOLD_LIST;
    };
    // ... folded as a complete binary tree (a two-source step is one)
    auto tree_partial = [&](int64_t a, const HostDesc& B) {
        if (!partial_of(a, B)) return false;
        const HostDesc& A = p.descs[a];
        const size_t n = A.srcs.size();
        if ((n & (n - 1)) != 0) return false;
        return A.fold == FOLD_PAIRWISE || (n == 2 && A.group == 0);
    };
    auto absorb_deps = [&](HostDesc& into, const HostDesc& from) {
        into.deps.insert(into.deps.end(), from.deps.begin(), from.deps.end());
    };

    for (uint32_t i = 0; i < D; ++i) {
        HostDesc& B = p.descs[i];
        if (!B.alive) continue;
        if (B.op == OP_REDUCE && B.group == 0 && B.fold == FOLD_LIST && !B.srcs.empty()) {
            // Rule 4 (trees): B adds the roots of two equally sized binary trees, each a private
            // partial -> one binary tree over both leaf lists (a recursive-halving level).
            if (B.srcs.size() == 2 && tree_partial(prod[i][0], B) && tree_partial(prod[i][1], B) &&
                p.descs[prod[i][0]].srcs.size() == p.descs[prod[i][1]].srcs.size() &&
                2 * p.descs[prod[i][0]].srcs.size() <= (size_t)kMaxOperands) {
                std::vector<Operand> srcs;
                std::vector<int64_t> sprod;
                for (int k = 0; k < 2; ++k) {
                    uint32_t a = (uint32_t)prod[i][k];
                    HostDesc& A = p.descs[a];
                    srcs.insert(srcs.end(), A.srcs.begin(), A.srcs.end());
                    sprod.insert(sprod.end(), prod[a].begin(), prod[a].end());
                    absorb_deps(B, A);
                    A.alive = false;
                    fwd[a] = i;
                }
                B.srcs = std::move(srcs);
                prod[i] = std::move(sprod);
                B.fold = FOLD_PAIRWISE;
                continue;
            }
            // Rule 2: every source is a private partial of an equally sized flat reduction.
            bool groups = B.srcs.size() >= 2;
            size_t L = 0, total = 0;
            for (size_t k = 0; groups && k < B.srcs.size(); ++k) {
                int64_t a = prod[i][k];
                if (!private_partial(a, B) || (L && p.descs[a].srcs.size() != L)) {
                    groups = false;
                    break;
                }
                L = p.descs[a].srcs.size();
                total += L;
            }
            if (groups && total <= (size_t)kMaxOperands) {
                std::vector<Operand> srcs;
                std::vector<int64_t> sprod;
                size_t G = B.srcs.size();
                for (size_t k = 0; k < G; ++k) {
                    uint32_t a = (uint32_t)prod[i][k];
                    HostDesc& A = p.descs[a];
                    srcs.insert(srcs.end(), A.srcs.begin(), A.srcs.end());
                    sprod.insert(sprod.end(), prod[a].begin(), prod[a].end());
                    absorb_deps(B, A);
                    A.alive = false;
                    fwd[a] = i;
                }
                B.srcs = std::move(srcs);
                prod[i] = std::move(sprod);
                B.group = (G == 1 || L == 1) ? 0 : (uint16_t)L;
                continue;
            }
            // Rule 1: the first source is a private partial.
            int64_t a = prod[i][0];
            if (private_partial(a, B) && p.descs[a].srcs.size() + B.srcs.size() - 1 <= (size_t)kMaxOperands) {
                HostDesc& A = p.descs[a];
                std::vector<Operand> srcs = std::move(A.srcs);  // A ends here
                srcs.insert(srcs.end(), B.srcs.begin() + 1, B.srcs.end());
                std::vector<int64_t> sprod = std::move(prod[a]);
                sprod.insert(sprod.end(), prod[i].begin() + 1, prod[i].end());
                B.srcs = std::move(srcs);
                prod[i] = std::move(sprod);
                absorb_deps(B, A);
                A.alive = false;
                fwd[a] = i;
            }
            continue;
        }
        if (B.op == OP_COPY && B.srcs.size() == 1 && prod[i][0] >= 0) {
            // Rule 3: a forwarding copy of a value becomes more destinations of its producer.
            uint32_t e = find((uint32_t)prod[i][0]);
            HostDesc& E0 = p.descs[e];
            if (!E0.alive || E0.nelem != B.nelem || !depends_on(B, e)) continue;
            if (split && E0.op == OP_REDUCE && E0.srcs.size() >= kSplitMinSources) {
                // the copy of a wide reduction's result stays a step; an earlier copy of the
                // same value that waits only for that reduction takes its destinations
                bool only_e = true;
                for (const Dep& d : B.deps) only_e &= find(d.desc) == e;
                const OperandKey key{B.srcs[0].buf, B.srcs[0].offset};
                auto it = split_copy.find(key);
                if (only_e && it != split_copy.end()) {
                    HostDesc& S = p.descs[it->second];
                    bool s_only_e = true;
                    for (const Dep& d : S.deps) s_only_e &= find(d.desc) == e;
                    if (S.alive && S.nelem == B.nelem && S.srcs[0].dtype == B.srcs[0].dtype && s_only_e &&
                        S.dsts.size() + B.dsts.size() <= (size_t)kMaxOperands) {
                        S.dsts.insert(S.dsts.end(), B.dsts.begin(), B.dsts.end());
                        nread[it->second].resize(S.dsts.size(), 0);
                        B.alive = false;
                        fwd[i] = it->second;
                        continue;
                    }
                }
                if (only_e) split_copy[key] = i;
                continue;
            }
            HostDesc& E = E0;
            if (E.dsts.size() + B.dsts.size() > (size_t)kMaxOperands) continue;
            bool deps_ok = true;
            for (const Dep& d : B.deps) {
                uint32_t t = find(d.desc);
                if (t != e && t > e) deps_ok = false;
            }
            if (!deps_ok) continue;
            E.dsts.insert(E.dsts.end(), B.dsts.begin(), B.dsts.end());
            nread[e].resize(E.dsts.size(), 0);
            for (const Dep& d : B.deps)
                if (find(d.desc) != e) E.deps.push_back(d);
            B.alive = false;
            fwd[i] = e;
        }
    }
    // resolve every dependency to the step that survived
    for (uint32_t i = 0; i < D; ++i) {
        HostDesc& d = p.descs[i];
        if (!d.alive) continue;
        for (Dep& e : d.deps) e.desc = find(e.desc);
        dedupe_deps(d, i);
    }
    drop_unused_scratch(p);
}

// ------------------------------------------------------------------------------ groups
bool merge(std::vector<HostProgram>& parts, const std::vector<CollectiveSpec>& specs, HostProgram& out,
           std::string& err) {
    out = HostProgram();
    const size_t n = parts.size();
    std::vector<uint32_t> buf_base(n), nbuf(n), meta_base(n), aux_base(n);
    std::vector<uint64_t> scratch_base(n), bytes(n);
    uint32_t total = 0, nmeta = 0, naux = 0;
    uint64_t scratch = 0;
    for (size_t k = 0; k < n; ++k) {
        buf_base[k] = total;
        nbuf[k] = 2u * (uint32_t)specs[k].P;
        total += nbuf[k];
        meta_base[k] = nmeta;
        nmeta += parts[k].nmeta;
        aux_base[k] = naux;
        naux += (uint32_t)parts[k].aux.size();
        scratch_base[k] = scratch;
        scratch += (parts[k].scratch_bytes + 255) & ~uint64_t(255);
        for (const auto& d : parts[k].descs)
            if (d.alive) bytes[k] += d.nelem * (d.srcs.size() + d.dsts.size());
    }
    if (total > 2u * (uint32_t)kMaxRanks) {
        err = "a group may name at most 128 rank buffers";
        return false;
    }
    if (nmeta > (uint32_t)kMaxMetaBuffers) {
        err = "a group may hold at most two dynamic calls";
        return false;
    }
    std::vector<size_t> order(n);
    for (size_t k = 0; k < n; ++k) order[k] = k;
    std::stable_sort(order.begin(), order.end(), [&](size_t a, size_t b) { return bytes[a] < bytes[b]; });
    // merged ids: every call's rank buffers, then the one scratch, then every call's metadata
    const uint32_t scratch_id = total;
    out.P = (int)(total / 2);
    auto move_id = [&](size_t k, uint32_t id) -> uint32_t {
        if (id == kNoBuffer) return kNoBuffer;
        if (id < nbuf[k]) return id + buf_base[k];
        if (id == nbuf[k]) return scratch_id;
        return meta_buf(out.P, (int)(meta_base[k] + (id - nbuf[k] - 1)));
    };
    for (size_t k = 0; k < n; ++k) {
        for (DynA2A a : parts[k].aux) {
            a.send0 = move_id(k, a.send0);
            a.recv0 = move_id(k, a.recv0);
            a.counts = move_id(k, a.counts);
            a.sdispls = move_id(k, a.sdispls);
            a.rdispls = move_id(k, a.rdispls);
            a.recvcounts = move_id(k, a.recvcounts);
            out.aux.push_back(a);
        }
    }
    bool fused = true;
    for (size_t k : order) {
        HostProgram& p = parts[k];
        fused &= p.fused;
        std::vector<int64_t> remap(p.descs.size(), -1);
        const uint32_t first = (uint32_t)out.descs.size();
        for (size_t i = 0; i < p.descs.size(); ++i) {
            if (!p.descs[i].alive) continue;
            remap[i] = (int64_t)(first + (out.descs.size() - first));
            HostDesc d = p.descs[i];
            for (auto* list : {&d.srcs, &d.dsts}) {
                for (Operand& o : *list) {
                    if (o.buf == nbuf[k]) o.offset += scratch_base[k];
                    o.buf = move_id(k, o.buf);
                }
            }
            d.aux += aux_base[k];
            out.descs.push_back(std::move(d));
        }
        for (uint32_t i = first; i < out.descs.size(); ++i) {
            for (Dep& e : out.descs[i].deps) {
                if (remap[e.desc] < 0) {
                    err = "dependency on a removed step";
                    return false;
                }
                e.desc = (uint32_t)remap[e.desc];
            }
        }
    }
    out.nmeta = nmeta;
    out.phase_mode = specs[0].phases;
    out.algo = parts[order[0]].algo;
    out.fused = fused;
    out.scratch_bytes = scratch;
    return true;
}

// ---------------------------------------------------------------------- uniform phases
namespace {

// Tiles of a uniform phase, measured on MI355X with three sets of buffers in turn (so that a call
// does not find its own inputs in the last-level cache). Bytes per tile are those of one source.
//  * Reductions: 2 KiB, two vectors per lane and source; 1 KiB for the binary tree, which takes
//    one vector per lane. 1 / 2 / 4 KiB: 8-rank reduce-scatter of 64 MiB bf16 29.2 / 27.3 / 28.6 us,
//    ragged 31.8 / 30.7 / 36.9; all-reduce of 8 x 16 MiB bf16 58.1 / 52.9 / 58.8; 16-rank halving
//    reduce-scatter of 8 MiB fp16 23.9 / 25.2 / 28.1.
//  * From 1 GiB moved on, by the number of sources (1 / 2 / 4 KiB; the executor's kernel in brackets).
//    Many of them, or some and one destination, 1 KiB: reduce-scatter of 8 ranks, 1.2 GiB moved bf16
//    205 / 216 / 221 (234), of 8 x 256 MiB 406 / 415 / 412 (428), of 12 ranks, 1 GiB 175 / 184 / 190
//    (176); all-reduce of 12 ranks, 1.2 GiB bf16 228 / 235 / 243 (232), of 15 231 / 244 / 269 (243);
//    but reduce-scatter of 4, 1 GiB bf16 185 / 176 / 179 (196), of 2 223 / 168 / 168 (207). Two sources
//    from 2 GiB on, 4 KiB: all-reduce bf16 of 2 GiB 405 / 368 / 343 (405), of 1 GiB 188 / 172 / 177
//    (215). Others 2 KiB: all-reduce of 8 ranks, 1 GiB fp32 189 / 185 / 215 (218), 2 GiB bf16
//    428 / 390 / 386 (366), 1.2 GiB bf16 220 / 226 / 233 (236). From 16 sources on 2 KiB again: of
//    16 ranks, 1.2 GiB 225 / 228 / 233 (232). On a stream of few CUs what each of them has in flight
//    counts: never 1 KiB there. 1 / 2 KiB: reduce-scatter of 8 x 256 MiB on 16 CUs 3 046 / 2 638 us
//    (2 700), 64 829 / 746 (771), 128 488 / 468 (484), 192 387 / 399 (414), all-reduce of 12,
//    1.5 GiB on 16 CUs 3 679 / 3 297 (3 581).
//  * Copies: 4 KiB. 2 / 4 / 8 KiB: all-gather of 8 x 8 MiB 95.5 / 86.4 / 97, of 2 x 64 MiB
//    67.3 / 67.7 / 75.3, of 8 x 104 KB 6.1 / 5.1 / 5.4.
//  * Small phases are cut further, down to one vector per lane, to give more wavefronts work.
constexpr uint64_t kUniformReduceBytes = 2048;
constexpr uint64_t kUniformLargeMoved = 1ull << 30;
constexpr uint32_t kUniformManySources = 9, kUniformSomeSources = 6;
constexpr uint64_t kUniformCopyBytes = 4096;
constexpr uint64_t kUniformCopyTiles = 256;
constexpr uint64_t kUniformStepBytes = kWaveSize * 16;
// Destinations that one wavefront of a copy writes: all of them, its tile loaded once; four, the
// others left to its neighbours, while that makes fewer than this many wavefronts. One / four /
// all: all-gather of 8 x 8 MiB 96.7 / 96.5 / 86.4 us; of 8 x 1.2 MB 15.9 / 15.5 / 16.8; of
// 32 x 13.8 KB 6.3 / 5.5 / 17.3; of 64 x 9 KB 8.9 / 7.9 / 24.0.
// Segments whose length is a power of two, from this many tiles on, are the exception where they are
// aligned: neighbours that write the same place of different buffers then meet in the same
// memory channels. Four / all: all-gather of 32 x 128 KiB 29.3 / 21.6 us (executor 27.0), of 16 x
// 256 KiB 14.2 / 11.3, of 8 x 1 MiB 12.2 / 11.3; but of 32 x 131 200 bytes 28.5 / 28.9, of
// 64 x 131 200 99.7 / 110.7, with fewer tiles of 16 x 128 KiB 7.5 / 9.2, to fewer of 5 x 1 MiB
// 5.8 / 6.2.
constexpr uint32_t kUniformFewDsts = 4;
constexpr uint64_t kUniformFewWaves = 16384;
constexpr uint64_t kUniformWholeTiles = 1024;
// A reduction that moves no more than this finds its inputs in the caches, where the producer left
// them: ordinary loads (all-reduce of 8 x 64 KiB 6.0 -> 4.9 us back to back; maxima, trees and
// re-quantised sums of 8 x 512 KiB alike, with either load 5.5, 4.4 and 4.7); beyond it the
// non-temporal ones are as good or better (of 8 x 2 MiB 7.6 / 6.8, a maximum 7.5 / 7.2, of 16 x
// 8 MiB 26.4 / 23.9, the 1 GiB reduce-scatter 435 / 405). Results are stored non-temporally at
// every size (all-reduce of 4 x 4 MiB: ordinary stores 7.8, non-temporal 6.9; the reduce-scatter of
// 8 x 256 MiB on buffers other than the last call's 418 / 405, called again on the same ones, whose
// results the last-level cache then holds, 393 / 402), unless a later phase of the program reads them.
constexpr uint64_t kUniformCachedBytes = 8ull << 20;

// Copies of this many bytes to this many destinations stay on the executor's kernel where every
// operand is 16-byte aligned: its 32 KiB tiles write runs of 8 KiB to each destination in turn.
// Executor / uniform: two-level all-reduce of 64 ranks, whose second phase is such a copy, 8 MiB per
// rank 182 / 175 us for the call, 16 MiB 357 / 365, 32 MiB 720 / 758, of 32 ranks x 32 MiB 362 / 372;
// all-gather of 64 blocks of 128 KiB 101 / 89, of 256 KiB 198 / 194, 512 KiB 389 / 395, 1 MiB
// 747 / 833; of 32 blocks of 512 KiB 98 / 97, 1 MiB 199 / 192, 2 MiB 389 / 391. Other alignments
// take the executor to single elements: 32 blocks of 300 001 fp32 378 / 238, 64 of them
// 1350 / 895, 64 of 262 144 fp32 one element off a boundary 1055 / 805.
constexpr uint64_t kLongRunDsts = 32;
constexpr uint64_t kLongRunBytes = 16ull << 20;
// So does one large copy by itself (one rank, 1 GiB: executor 355 us, uniform 370, as a list 360).
bool one_long_copy(uint32_t op, uint32_t nseg, uint32_t ndst, uint64_t bytes) {
    return op == OP_COPY && nseg == 1 && ndst == 1 && bytes >= kLongRunBytes;
}

void uniform_tile(UniformPhase& u, uint64_t elems) {
    const uint64_t es = dtype_size(u.kernel.dtype);
    const uint64_t moved = elems * es * (u.nsrc() + u.ndst());
    uint64_t bytes = kUniformCopyBytes, sets = 1, want = kUniformCopyTiles;
    if (u.kernel.op == OP_REDUCE) {
        bytes = kUniformReduceBytes;
        if (u.kernel.fold == FOLD_PAIRWISE) {
            bytes = kUniformStepBytes;
        } else if (moved >= kUniformLargeMoved && u.nsrc() < kSplitMinSources) {
            if (u.nsrc() >= kUniformManySources || (u.nsrc() >= kUniformSomeSources && u.ndst() == 1)) bytes = kUniformStepBytes;
            else if (u.nsrc() <= 2 && moved >= 2 * kUniformLargeMoved) bytes = 2 * kUniformReduceBytes;
        }
        want = kSmallTargetTiles;
    } else {
        const uint64_t few = (u.ndst() + kUniformFewDsts - 1) / kUniformFewDsts;
        const bool split = (elems * es + bytes - 1) / bytes * few < kUniformFewWaves;
        u.per_wave = split ? std::min(kUniformFewDsts, u.ndst()) : u.ndst();
        sets = split ? few : 1;
        const uint64_t segment = u.seg_elems * es;
        const bool resonant = (segment & (segment - 1)) == 0 && u.ndst() >= 2 * kUniformFewDsts &&
                              elems * es / bytes >= kUniformWholeTiles;
        u.aligned_per_wave = resonant ? u.ndst() : u.per_wave;
    }
    while (bytes > kUniformStepBytes && elems * es / bytes * sets < want) bytes /= 2;
    u.tile_elems = u.few_cus_tile_elems = (uint32_t)(bytes / es);
    if (u.kernel.op == OP_REDUCE && u.kernel.fold != FOLD_PAIRWISE && moved >= kUniformLargeMoved)
        u.few_cus_tile_elems = (uint32_t)(std::max(bytes, kUniformReduceBytes) / es);
}

bool same_bufs(const std::vector<Operand>& a, const std::vector<Operand>& b) {
    if (a.size() != b.size()) return false;
    for (size_t i = 0; i < a.size(); ++i)
        if (a[i].buf != b[i].buf) return false;
    return true;
}

// Operands in the order of their buffer ids (a counting sort: there are few ids).
std::vector<Operand> by_buffer(const std::vector<Operand>& v) {
    uint32_t most = 0;
    for (const Operand& o : v) most = std::max(most, o.buf);
    std::vector<uint32_t> at(most + 2, 0);
    for (const Operand& o : v) ++at[o.buf + 1];
    for (uint32_t b = 0; b < most; ++b) at[b + 1] += at[b];
    std::vector<Operand> out(v.size());
    for (const Operand& o : v) out[at[o.buf]++] = o;
    return out;
}

// The uniform form of the steps [d0, d1) of one phase, none of which waits for another. `tile`
// is the tile size of a configured tile_bytes (0: chosen here), which the caller asked for step
// by step: then only a single step has this form. `reread`: a later phase reads the results.
UniformPhase find_uniform(const std::vector<HostDesc>& all, uint32_t d0, uint32_t d1, uint32_t tile, bool reread) {
    UniformPhase u;
    if (d0 == d1 || (tile && d1 - d0 != 1)) return u;
    const HostDesc& f = all[d0];
    if (f.op != OP_COPY && f.op != OP_REDUCE) return u;
    if (f.srcs.empty() || f.dsts.empty()) return u;
    const uint32_t dt = f.srcs[0].dtype;
    const uint64_t es = dtype_size(dt);
    struct Step {
        const std::vector<Operand>* srcs;
        const std::vector<Operand>* dsts;
        uint64_t nelem;
        uint64_t bufs;  // a hash of the buffers named, so that steps of the same ones sort together
    };
    // whether b continues p in every operand
    auto continues = [&](const Step& p, const std::vector<Operand>& srcs, const std::vector<Operand>& dsts) {
        bool joins = srcs.size() == p.srcs->size() && dsts.size() == p.dsts->size();
        const uint64_t by = p.nelem * es;
        auto follow = [&](const std::vector<Operand>& a, const std::vector<Operand>& b) {
            bool same = true;
            for (size_t k = 0; k < a.size(); ++k)
                same &= a[k].buf == b[k].buf && a[k].dtype == b[k].dtype && a[k].offset + by == b[k].offset;
            return same;
        };
        return joins && follow(*p.srcs, srcs) && follow(*p.dsts, dsts);
    };
    // The chunks of a step mostly follow it in the program: joined as they come, there is less to
    // hash and sort. Steps that name more than kMaxOperands different sets of buffers (the pairs of a
    // wide exchange) stay more than that many segments: they are given up as soon as that shows.
    std::vector<Step> steps;
    constexpr size_t kSlots = 4 * kMaxOperands;
    uint64_t seen[kSlots] = {0};  // hashes of the sets, open addressing
    uint32_t sets = 0;
    for (uint32_t i = d0; i < d1; ++i) {
        const HostDesc& d = all[i];
        if (d.op != f.op || d.redop != f.redop || d.group != f.group || d.fold != f.fold || d.requant != f.requant ||
            !d.deps.empty() || d.nelem == 0 || d.srcs.size() != f.srcs.size() || d.dsts.size() != f.dsts.size())
            return u;
        if (!steps.empty() && continues(steps.back(), d.srcs, d.dsts)) {
            steps.back().nelem += d.nelem;
            continue;
        }
        // (the order of a step's destinations is free, that of its sources is not)
        uint64_t in = 0, out = 0;
        for (const Operand& o : d.srcs) {
            if (o.dtype != dt) return u;
            in = (in ^ o.buf) * 0x9E3779B97F4A7C15ull + 1;
        }
        for (const Operand& o : d.dsts) {
            if (o.dtype != dt) return u;
            const uint64_t h = (o.buf + 1) * 0x9E3779B97F4A7C15ull;
            out += h ^ (h >> 29);
        }
        const uint64_t bufs = (in ^ out) | 1;
        size_t at = (bufs >> 32) % kSlots;
        while (seen[at] != 0 && seen[at] != bufs) at = (at + 1) % kSlots;
        if (seen[at] == 0) {
            seen[at] = bufs;
            if (++sets > (uint32_t)kMaxOperands) return u;
        }
        steps.push_back({&d.srcs, &d.dsts, d.nelem, bufs});
    }
    // all segments are of one length, but for one that may be shorter
    auto lengths_fit = [](const std::vector<Step>& v) {
        uint64_t longest = 0;
        size_t others = 0;
        for (const Step& d : v) longest = std::max(longest, d.nelem);
        for (const Step& d : v) others += d.nelem != longest;
        return others <= 1;
    };
    if (sets == steps.size() && !lengths_fit(steps)) return u;  // (no two of these can join)
    std::list<std::vector<Operand>> sorted;
    auto by_buf = [](const Operand& a, const Operand& b) { return a.buf < b.buf; };
    for (Step& d : steps)
        if (!std::is_sorted(d.dsts->begin(), d.dsts->end(), by_buf)) {
            sorted.push_back(by_buffer(*d.dsts));
            d.dsts = &sorted.back();
        }
    // join the steps that continue one another elsewhere in the program
    std::stable_sort(steps.begin(), steps.end(), [](const Step& a, const Step& b) {
        return a.bufs != b.bufs ? a.bufs < b.bufs : (*a.dsts)[0].offset < (*b.dsts)[0].offset;
    });
    std::vector<Step> segs;
    for (const Step& d : steps) {
        if (!segs.empty() && continues(segs.back(), *d.srcs, *d.dsts)) segs.back().nelem += d.nelem;
        else segs.push_back(d);
        if (segs.size() > (size_t)kMaxOperands) return u;
    }
    if (!lengths_fit(segs)) return u;
    std::stable_sort(segs.begin(), segs.end(), [](const Step& a, const Step& b) {
        const Operand &ad = (*a.dsts)[0], &bd = (*b.dsts)[0], &as = (*a.srcs)[0], &bs = (*b.srcs)[0];
        if (ad.offset != bd.offset) return ad.offset < bd.offset;
        if (as.offset != bs.offset) return as.offset < bs.offset;
        return as.buf < bs.buf;
    });
    const Step& s0 = segs[0];
    const std::vector<Operand>& src0 = *s0.srcs;
    const std::vector<Operand>& dst0 = *s0.dsts;
    const uint32_t n = (uint32_t)segs.size();
    for (uint32_t g = 1; g < n; ++g)
        if (g + 1 < n ? segs[g].nelem != s0.nelem : segs[g].nelem > s0.nelem) return u;

    // one list for every segment, at a constant step?
    auto shared = [&](const std::vector<Operand>* Step::*list, uint64_t& step) {
        const std::vector<Operand>& base = *(s0.*list);
        step = n > 1 ? (*(segs[1].*list))[0].offset - base[0].offset : 0;
        for (uint32_t g = 1; g < n; ++g) {
            if (!same_bufs(*(segs[g].*list), base)) return false;
            for (size_t k = 0; k < base.size(); ++k)
                if ((*(segs[g].*list))[k].offset != base[k].offset + g * step) return false;
        }
        return true;
    };
    // the sources of segment g are those of one list from its place g + 1 on (ring order)?
    auto rotated = [&](uint64_t step, std::vector<Operand>& base) {
        const uint32_t m = (uint32_t)src0.size();
        base.resize(m);
        for (uint32_t k = 0; k < m; ++k) base[(k + 1) % m] = src0[k];
        for (uint32_t g = 0; g < n; ++g)
            for (uint32_t k = 0; k < m; ++k) {
                const Operand &o = base[(k + g + 1) % m], &x = (*segs[g].srcs)[k];
                if (x.buf != o.buf || x.offset != o.offset + g * step) return false;
            }
        return n <= m;
    };
    // ... or those of segment 0 with the bits of g, in reverse, flipped in their place (halving order)?
    auto flipped = [&](uint64_t step) {
        const uint32_t m = (uint32_t)src0.size();
        if ((m & (m - 1)) != 0 || n > m) return false;
        for (uint32_t g = 0; g < n; ++g) {
            uint32_t rev = 0;
            for (uint32_t b = 1, t = m >> 1; b < m; b <<= 1, t >>= 1)
                if (g & b) rev |= t;
            for (uint32_t k = 0; k < m; ++k) {
                const Operand &o = src0[k ^ rev], &x = (*segs[g].srcs)[k];
                if (x.buf != o.buf || x.offset != o.offset + g * step) return false;
            }
        }
        return true;
    };
    std::vector<Operand> base;
    if (shared(&Step::srcs, u.src_step)) {
        u.srcs = src0;
    } else if (src0.size() == 1) {
        u.flags |= UF_SRC_PER_SEG;
        u.src_step = 0;
        for (const Step& d : segs) u.srcs.push_back((*d.srcs)[0]);
    } else if (rotated(u.src_step = (*segs[1].srcs)[0].offset - src0[0].offset, base)) {
        u.flags |= UF_ROTATE;
        u.srcs = base;
    } else if (flipped(u.src_step)) {
        u.flags |= UF_FLIP;
        u.srcs = src0;
    } else {
        return u;
    }
    if (shared(&Step::dsts, u.dst_step)) {
        u.dsts = dst0;
    } else if (dst0.size() == 1) {
        u.flags |= UF_DST_PER_SEG;
        u.dst_step = 0;
        for (const Step& d : segs) u.dsts.push_back((*d.dsts)[0]);
    } else if (f.op == OP_COPY && dst0.size() < (size_t)kMaxOperands) {
        // copies of one location of every buffer but the source's own (the results of a two-level
        // all-reduce): the list of all of them; a wavefront leaves out the destination that is
        // its source
        const size_t m = dst0.size() + 1;
        // operand k of a segment's destinations with its source among them
        auto place = [&](const Step& d) { return std::upper_bound(d.dsts->begin(), d.dsts->end(), (*d.srcs)[0], by_buf) - d.dsts->begin(); };
        auto with_source = [](const Step& d, size_t at, size_t k) -> const Operand& {
            return k == at ? (*d.srcs)[0] : (*d.dsts)[k - (k > at)];
        };
        for (size_t k = 0; k < m; ++k) u.dsts.push_back(with_source(s0, place(s0), k));
        for (size_t k = 1; k < m; ++k)
            if (u.dsts[k].buf == u.dsts[k - 1].buf) return u;
        u.dst_step = with_source(segs[1], place(segs[1]), 0).offset - u.dsts[0].offset;
        for (uint32_t g = 1; g < n; ++g) {
            const size_t at = place(segs[g]);
            for (size_t k = 0; k < m; ++k) {
                const Operand& o = with_source(segs[g], at, k);
                if (o.buf != u.dsts[k].buf || o.offset != u.dsts[k].offset + g * u.dst_step) return u;
            }
        }
    } else {
        return u;
    }
    u.group = f.group;
    u.nseg = n;
    u.seg_elems = s0.nelem;
    u.last_elems = segs[n - 1].nelem;
    uint64_t total = 0;
    for (const Step& d : segs) total += d.nelem;
    u.kernel = {f.op, (uint8_t)dt, f.redop, (uint8_t)f.fold, f.requant, 0};
    // (a maximum, a minimum and a wrapping sum do not depend on how their list is bracketed)
    if (f.op == OP_REDUCE && (f.redop != RO_SUM || dt == DT_INT32)) u.kernel.fold = FOLD_LIST, u.group = 0;
    if (f.op == OP_REDUCE && (f.redop != RO_SUM || dt == DT_INT32 || dt == DT_FP32)) u.kernel.requant = false;
    if (f.op == OP_REDUCE && reread) u.kernel.mem = MEM_STORE;
    else if (f.op == OP_REDUCE && total * es * (u.nsrc() + u.ndst()) <= kUniformCachedBytes) u.kernel.mem = MEM_LOAD;
    u.per_wave = u.aligned_per_wave = 1;
    if (tile) u.tile_elems = u.few_cus_tile_elems = tile;
    else uniform_tile(u, total);
    u.long_run = f.op == OP_COPY && u.ndst() >= kLongRunDsts && total * es >= kLongRunBytes;
    u.ok = u.ntiles(u.tile_elems, u.per_wave) < (1ull << 31) && !one_long_copy(f.op, u.nseg, u.ndst(), total * es);
    return u;
}

// The copy list of a program of one phase (see CopyEntry), destination by destination, the calls of a
// group in the order of its steps: at any moment the chip fills one receive buffer in order. Empty
// if the program is not of that form.
std::vector<CopyEntry> copy_list(const HostProgram& p, uint32_t& ntiles) {
    std::vector<CopyEntry> list;
    // Copies by destination buffer, in the order in which the destinations first come up, then by
    // source buffer (two counting sorts): those of packed receive ranges are then in their order.
    constexpr uint32_t kBufs = 2u * kMaxRanks;
    uint32_t place[kBufs], dst_at[kBufs + 1] = {0}, src_at[kBufs + 1] = {0}, ndst = 0;
    std::fill_n(place, kBufs, ~0u);
    for (const HostDesc& d : p.descs) {
        if (d.op != OP_COPY || d.srcs.size() != 1 || d.dsts.size() != 1 || !d.deps.empty() || d.nelem == 0) return list;
        if (d.srcs[0].buf >= kBufs || d.dsts[0].buf >= kBufs) return list;
        uint32_t& k = place[d.dsts[0].buf];
        if (k == ~0u) k = ndst++;
        ++dst_at[k + 1];
        ++src_at[d.srcs[0].buf + 1];
    }
    for (uint32_t k = 0; k < kBufs; ++k) dst_at[k + 1] += dst_at[k], src_at[k + 1] += src_at[k];
    std::vector<uint32_t> by_src(p.descs.size());
    for (size_t i = 0; i < p.descs.size(); ++i) by_src[src_at[p.descs[i].srcs[0].buf]++] = (uint32_t)i;
    std::vector<CopyEntry> v(p.descs.size());
    for (uint32_t i : by_src) {
        const Operand &s = p.descs[i].srcs[0], &t = p.descs[i].dsts[0];
        v[dst_at[place[t.buf]]++] = {s.offset, t.offset, p.descs[i].nelem * dtype_size(s.dtype), s.buf | t.buf << 16, 0};
    }
    auto by_offset = [](const CopyEntry& a, const CopyEntry& b) { return a.dst_off < b.dst_off; };
    for (uint32_t k = 0; k < ndst; ++k) {  // (dst_at[k] is where destination k ends now)
        const auto from = v.begin() + (k ? dst_at[k - 1] : 0u), to = v.begin() + dst_at[k];
        if (!std::is_sorted(from, to, by_offset)) std::sort(from, to, by_offset);
    }
    list.reserve(v.size());
    for (const CopyEntry& e : v) {
        if (!list.empty() && list.back().bufs == e.bufs && list.back().src_off + list.back().bytes == e.src_off &&
            list.back().dst_off + list.back().bytes == e.dst_off)
            list.back().bytes += e.bytes;
        else
            list.push_back(e);
    }
    uint64_t t = 0;
    for (CopyEntry& e : list) {
        e.tile0 = (uint32_t)t;
        t += (e.bytes + kListTileBytes - 1) / kListTileBytes;
    }
    if (list.size() > kListMaxEntries || t >= (1ull << 31) || (list.size() == 1 && one_long_copy(OP_COPY, 1, 1, list[0].bytes)))
        list.clear();
    ntiles = (uint32_t)t;
    return list;
}

}  // namespace

// ---------------------------------------------------------------------------- packing
bool finalize(HostProgram& p, uint32_t tile_bytes, std::string& err) {
    // compact
    std::vector<int64_t> remap(p.descs.size(), -1);
    size_t live = 0;
    for (size_t i = 0; i < p.descs.size(); ++i) {
        if (!p.descs[i].alive) continue;
        remap[i] = (int64_t)live;
        if (live != i) p.descs[live] = std::move(p.descs[i]);
        ++live;
    }
    p.descs.resize(live);
    for (size_t i = 0; i < live; ++i) {
        for (Dep& d : p.descs[i].deps) {
            if (remap[d.desc] < 0) {
                err = "dependency on a removed step";
                return false;
            }
            d.desc = (uint32_t)remap[d.desc];
        }
        dedupe_deps(p.descs[i], (uint32_t)i);
    }

    // Phases. A step's level is 0 without dependencies, else one more than the highest level it
    // waits for. Run level by level, one launch each, every dependency is met by the launch
    // order: the steps are laid out level by level (program order inside a level) and carry no
    // dependencies on the device. Otherwise the whole program is one launch and its
    // dependencies are waited for tile by tile.
    {
        const uint32_t n = (uint32_t)p.descs.size();
        std::vector<uint32_t> level(n, 0);
        uint32_t nlev = 1;
        bool deps_here = false;
        for (uint32_t i = 0; i < n; ++i) {
            for (const Dep& d : p.descs[i].deps) level[i] = std::max(level[i], level[d.desc] + 1);
            deps_here |= !p.descs[i].deps.empty();
            nlev = std::max(nlev, level[i] + 1);
        }
        const bool by_level = deps_here && nlev <= kMaxPhases &&
                              (p.phase_mode == PHASE_LEVELS || (p.phase_mode == PHASE_AUTO && nlev <= kAutoMaxPhases));
        p.desc_phase.assign(n, 0);
        if (by_level) {
            std::vector<uint32_t> order(n);
            for (uint32_t i = 0; i < n; ++i) order[i] = i;
            std::stable_sort(order.begin(), order.end(), [&](uint32_t a, uint32_t b) { return level[a] < level[b]; });
            std::vector<HostDesc> sorted;
            sorted.reserve(n);
            for (uint32_t k = 0; k < n; ++k) {
                sorted.push_back(std::move(p.descs[order[k]]));
                sorted.back().deps.clear();  // met by the launch order
                p.desc_phase[k] = level[order[k]];
            }
            p.descs = std::move(sorted);
        }
    }
    const uint32_t nphase = p.descs.empty() ? 1u : p.desc_phase.back() + 1;

    // One tile size for a program with dependencies, so per-tile dependencies line up; without
    // them every step gets the tile size for its own element width (the bf16 rows of a group
    // with int32 ids keep 8 KiB tiles instead of taking the ids' element count).
    uint64_t max_bpe = 1, total_elems = 0;
    std::vector<uint64_t> phase_elems(nphase, 0), phase_wide_copy_bytes(nphase, 0);
    bool any_reduce = false, any_deps = false;
    for (size_t i = 0; i < p.descs.size(); ++i) {
        const auto& d = p.descs[i];
        uint64_t bpe = 0;
        for (const Operand& o : d.srcs) bpe += dtype_size(o.dtype);
        max_bpe = std::max(max_bpe, bpe);
        any_reduce |= d.op == OP_REDUCE;
        any_deps |= !d.deps.empty();
        total_elems += d.nelem;
        phase_elems[p.desc_phase[i]] += d.nelem;
        if (d.op == OP_COPY && d.dsts.size() >= kWideCopyDsts) phase_wide_copy_bytes[p.desc_phase[i]] += d.nelem * bpe;
    }
    uint64_t tb = tile_bytes;
    if (!tb) tb = any_deps ? kDefaultDependentTileBytes : any_reduce ? kDefaultReduceTileBytes : kDefaultCopyTileBytes;
    uint64_t te = (tb / max_bpe) / kWaveStepElems * kWaveStepElems;
    if (!tile_bytes && any_reduce) te = std::max<uint64_t>(te, kMinReduceTileElems);
    if (!tile_bytes && !any_deps)
        te = std::min<uint64_t>(te, total_elems / kSmallTargetTiles / kWaveStepElems * kWaveStepElems);
    if (!tile_bytes && any_deps) {
        auto count_tiles = [&](uint64_t e) {
            uint64_t n = 0;
            for (const auto& d : p.descs) n += std::max<uint64_t>(1, (d.nelem + e - 1) / e);
            return n;
        };
        while (count_tiles(te) < kDependentMinTiles && (te / 2) * max_bpe >= kMinDependentTileBytes &&
               (te / 2) % kWaveStepElems == 0)
            te /= 2;
    }
    te = std::max<uint64_t>(te, kWaveStepElems);
    te = std::min<uint64_t>(te, 1ull << 30);
    p.tile_elems = (uint32_t)te;
    auto step_tile = [&](const HostDesc& h, uint32_t phase) -> uint64_t {
        if (any_deps || tile_bytes) return te;
        uint64_t bpe = 0;
        for (const Operand& o : h.srcs) bpe += dtype_size(o.dtype);
        if (bpe == 0) return te;
        // a copy to many destinations writes its tile to each of them: longer runs per
        // destination, and enough work per tile without cutting it for parallelism
        const bool wide_copy = h.op == OP_COPY && h.dsts.size() >= kWideCopyDsts;
        const uint64_t wide_tb = std::max<uint64_t>(
            kDefaultCopyTileBytes, std::min<uint64_t>(kWideCopyTileBytes, phase_wide_copy_bytes[phase] / kWideCopyTargetTiles));
        uint64_t t = ((wide_copy ? wide_tb : tb) / bpe) / kWaveStepElems * kWaveStepElems;
        if (any_reduce && !wide_copy) t = std::max<uint64_t>(t, kMinReduceTileElems);
        if (!wide_copy)
            t = std::min<uint64_t>(t, phase_elems[phase] / kSmallTargetTiles / kWaveStepElems * kWaveStepElems);
        return std::min<uint64_t>(std::max<uint64_t>(t, kWaveStepElems), 1ull << 30);
    };

    const uint32_t nd = (uint32_t)p.descs.size();
    std::vector<Desc> out(nd);
    std::vector<Operand> ops;
    std::vector<Dep> deps;
    size_t nops = 0, nedges = 0;
    for (const HostDesc& h : p.descs) nops += h.srcs.size() + h.dsts.size(), nedges += h.deps.size();
    ops.reserve(nops);
    deps.reserve(nedges);
    uint64_t ntiles = 0;
    p.bytes_read = p.bytes_written = 0;
    p.max_srcs = 0;
    p.step_tile_min = p.step_tile_max = 0;
    bool has_deps = false;
    for (uint32_t i = 0; i < nd; ++i) {
        const HostDesc& h = p.descs[i];
        Desc& d = out[i];
        std::memset(&d, 0, sizeof d);
        d.op = h.op;
        d.redop = h.redop;
        d.group = h.group;
        d.nsrc = (uint16_t)h.srcs.size();
        d.ndst = (uint16_t)h.dsts.size();
        d.nelem = h.nelem;
        // A maximum, a minimum and a wrapping sum do not depend on how their list is bracketed (ties
        // and NaNs keep the first in list order), and only 16-bit sums round their partials: the
        // kernels have trees and re-quantised folds for sums alone.
        const bool sum = h.op == OP_REDUCE && h.redop == RO_SUM, wide = !h.dsts.empty() && dtype_size(h.dsts[0].dtype) == 4;
        d.fold = sum && h.dsts[0].dtype != DT_INT32 ? h.fold : (uint32_t)FOLD_LIST;
        d.requant = sum && !wide && h.requant ? 1u : 0u;
        const uint64_t dte = step_tile(h, p.desc_phase[i]);
        d.tile_elems = (uint32_t)dte;
        if (h.op == OP_COPY || h.op == OP_REDUCE) {
            p.step_tile_min = p.step_tile_min ? std::min<uint32_t>(p.step_tile_min, (uint32_t)dte) : (uint32_t)dte;
            p.step_tile_max = std::max<uint32_t>(p.step_tile_max, (uint32_t)dte);
        }
        d.aux = h.aux;
        uint64_t nt = (h.nelem + dte - 1) / dte;
        if (h.op == OP_DYN_COPY) {
            if (h.aux >= p.aux.size()) {
                err = "dynamic step without its record";
                return false;
            }
            nt = p.aux[h.aux].slots;
        }
        if (nt == 0) nt = 1;
        d.ntiles = (uint32_t)nt;
        d.tile0 = (uint32_t)ntiles;
        ntiles += nt;
        if (ntiles >= (1ull << 31)) {
            err = "program has too many tiles";
            return false;
        }
        d.sig = SIG_INVALID;
        if (h.op == OP_REDUCE && !h.srcs.empty() && !h.dsts.empty()) {
            uint32_t tr = h.srcs.size() > 1 ? h.srcs[1].dtype : h.srcs[0].dtype;
            d.sig = reduce_signature(h.srcs[0].dtype, tr, h.dsts[0].dtype);
        }
        d.src = (uint32_t)ops.size();
        ops.insert(ops.end(), h.srcs.begin(), h.srcs.end());
        d.dst = (uint32_t)ops.size();
        ops.insert(ops.end(), h.dsts.begin(), h.dsts.end());
        d.dep = (uint32_t)deps.size();
        d.ndep = (uint16_t)h.deps.size();
        deps.insert(deps.end(), h.deps.begin(), h.deps.end());
        has_deps |= !h.deps.empty();
        p.max_srcs = std::max<uint32_t>(p.max_srcs, d.nsrc);
        for (const Operand& o : h.srcs) p.bytes_read += h.nelem * dtype_size(o.dtype);
        for (const Operand& o : h.dsts) p.bytes_written += h.nelem * dtype_size(o.dtype);
    }
    p.ntiles = (uint32_t)ntiles;
    p.nstate = has_deps ? (uint32_t)(kStateDescBase + nd + ntiles) : kStateDescBase;
    p.flags = has_deps ? (uint32_t)PF_HAS_DEPS : 0u;
    // dependency targets: expected values, state words, signal flags
    for (uint32_t i = 0; i < nd; ++i) {
        for (uint32_t k = 0; k < out[i].ndep; ++k) {
            Dep& e = deps[out[i].dep + k];
            Desc& t = out[e.desc];
            if (e.kind == DEP_ALL) {
                e.expected = t.ntiles;
                e.state = kStateDescBase + e.desc;
                t.flags |= DF_SIGNAL_DESC;
            } else {
                e.expected = 1;
                e.state = kStateDescBase + nd + t.tile0;
                t.flags |= DF_SIGNAL_TILE;
            }
        }
    }
    p.ndeps = (uint32_t)deps.size();
    p.noperands = (uint32_t)ops.size();

    // the leanest executor kernel that covers every step of [d0, d1)
    auto kernel_for = [&](uint32_t d0, uint32_t d1) {
        int kind = kKindCopyOnly;
        bool dynamic = false;
        for (uint32_t i = d0; i < d1; ++i) dynamic |= out[i].op == OP_DYN_COPY;
        for (uint32_t i = d0; i < d1; ++i) {
            if (out[i].op != OP_REDUCE) continue;
            const bool plain = out[i].sig <= SIG_INT32 && out[i].redop == RO_SUM && out[i].fold == FOLD_LIST &&
                               !out[i].requant;
            if (!plain) { kind = kKindGeneric; break; }
            if (kind == kKindCopyOnly) kind = out[i].sig;
            else if (kind != out[i].sig) { kind = kKindGeneric; break; }
        }
        if (dynamic) kind = (kind == kKindCopyOnly) ? kKindDynamic : kKindGeneric;  // the two that run them
        if (kind == kKindCopyOnly) {
            bool aligned = true;
            for (uint32_t i = d0; i < d1; ++i)
                for (uint32_t k = 0; k < (uint32_t)out[i].nsrc + out[i].ndst; ++k) aligned &= (ops[out[i].src + k].offset % 16) == 0;
            if (aligned) kind = kKindCopyAligned;  // the launch falls back if a buffer is not aligned
        }
        return kind;
    };
    p.kind = kernel_for(0, nd);
    p.phase_tile.assign(1, 0);
    p.phase_kind.clear();
    p.phase_xcd.clear();
    p.uniform.clear();
    for (uint32_t q = 0, i = 0; q < nphase; ++q) {
        const uint32_t d0 = i;
        while (i < nd && p.desc_phase[i] == q) ++i;
        p.phase_kind.push_back(kernel_for(d0, i));
        // A phase of wide reductions reads many buffers per wavefront; numbered XCD by XCD, each
        // XCD works on one stretch of them at a time.
        bool wide = i > d0;
        for (uint32_t k = d0; k < i; ++k) wide &= out[k].op == OP_REDUCE && out[k].nsrc >= kSplitMinSources;
        p.phase_xcd.push_back(wide ? 1 : 0);
        p.uniform.push_back(has_deps ? UniformPhase() : find_uniform(p.descs, d0, i, tile_bytes ? p.tile_elems : 0, q + 1 < nphase));
        if (wide) p.uniform.back().flags |= UF_XCD;
        p.phase_tile.push_back(i < nd ? out[i].tile0 : p.ntiles);
    }

    auto align16 = [](uint64_t x) { return (x + 15) & ~uint64_t(15); };
    ProgramHeader hdr;
    std::memset(&hdr, 0, sizeof hdr);
    hdr.magic = kProgramMagic;
    hdr.version = kProgramVersion;
    hdr.ndesc = nd;
    hdr.ntiles = p.ntiles;
    hdr.noperand = p.noperands;
    hdr.ndep = p.ndeps;
    hdr.flags = p.flags;
    hdr.nstate = p.nstate;
    hdr.off_desc = align16(sizeof(ProgramHeader));
    hdr.off_operand = align16(hdr.off_desc + (uint64_t)nd * sizeof(Desc));
    hdr.off_dep = align16(hdr.off_operand + ops.size() * sizeof(Operand));
    hdr.off_tile_desc = align16(hdr.off_dep + deps.size() * sizeof(Dep));
    hdr.off_aux = align16(hdr.off_tile_desc + (uint64_t)p.ntiles * sizeof(uint32_t));
    hdr.naux = (uint32_t)p.aux.size();
    hdr.nphase = nphase;
    hdr.off_phase = align16(hdr.off_aux + p.aux.size() * sizeof(DynA2A));
    const uint64_t off_list = align16(hdr.off_phase + p.phase_tile.size() * sizeof(uint32_t));
    std::vector<CopyEntry> list;
    if (nphase == 1 && !tile_bytes && !p.uniform[0].ok) list = copy_list(p, p.list_tiles);
    p.list_entries = (uint32_t)list.size();
    std::vector<uint32_t> ends;
    if (!list.empty()) {
        p.list_offset = hdr.off_list = off_list;
        ends.assign(64 + (list.size() + 63) / 64 * 64, ~0u);
        for (size_t i = 0; i < list.size(); ++i)
            ends[64 + i] = ends[i / 64] = i + 1 < list.size() ? list[i + 1].tile0 : p.list_tiles;
    }
    hdr.total_bytes = off_list + ends.size() * sizeof(uint32_t) + list.size() * sizeof(CopyEntry);
    hdr.scratch_bytes = p.scratch_bytes;
    p.image.assign(hdr.total_bytes, 0);
    std::memcpy(p.image.data(), &hdr, sizeof hdr);
    if (nd) std::memcpy(p.image.data() + hdr.off_desc, out.data(), (size_t)nd * sizeof(Desc));
    if (!ops.empty()) std::memcpy(p.image.data() + hdr.off_operand, ops.data(), ops.size() * sizeof(Operand));
    if (!deps.empty()) std::memcpy(p.image.data() + hdr.off_dep, deps.data(), deps.size() * sizeof(Dep));
    uint32_t* owner = (uint32_t*)(p.image.data() + hdr.off_tile_desc);  // (the image is allocated at any type's alignment)
    for (uint32_t i = 0; i < nd; ++i) owner = std::fill_n(owner, out[i].ntiles, i);
    if (!p.aux.empty()) std::memcpy(p.image.data() + hdr.off_aux, p.aux.data(), p.aux.size() * sizeof(DynA2A));
    if (!list.empty()) {
        std::memcpy(p.image.data() + off_list, ends.data(), ends.size() * sizeof(uint32_t));
        std::memcpy(p.image.data() + off_list + ends.size() * sizeof(uint32_t), list.data(), list.size() * sizeof(CopyEntry));
    }
    std::memcpy(p.image.data() + hdr.off_phase, p.phase_tile.data(), p.phase_tile.size() * sizeof(uint32_t));
    return true;
}

}  // namespace hccl
