// The uniform form of a phase (one fold or copy over equal segments, sent in the launch packet)
// says the same as the phase's steps: every destination element has the same sources in the same
// order, the same operator and the same rounding, and no element is written that the steps do not
// write. This driver compiles collectives over orders, schedules, types, chunkings, groups and odd
// counts with the library's own lowering, fusion and finalisation, expands both forms element by
// element and compares them; it also walks the tiles of every segment as the kernels cut them. Prints
// one line per disagreement and a summary; exit status 1 on any.
#include <cstdint>
#include <cstdio>
#include <map>
#include <string>
#include <utility>
#include <vector>

#include "compiler.h"

using namespace hccl;

namespace {

typedef std::pair<uint32_t, uint64_t> Place;  // buffer, byte
typedef std::map<Place, std::vector<uint64_t>> Writes;

int turn = 0, programs = 0, uniform = 0, bad = 0;

void write(Writes& w, Place at, const std::vector<uint64_t>& value, const char* what) {
    if (!w.emplace(at, value).second) {
        std::printf("TWICE %s: buffer %u byte %llu\n", what, at.first, (unsigned long long)at.second);
        ++bad;
    }
}

// what one element becomes: the fold, then its sources in order
std::vector<uint64_t> value(uint32_t op, uint32_t redop, uint32_t group, uint32_t fold, bool requant, uint32_t dt,
                            const std::vector<Place>& srcs) {
    if (op == OP_COPY) redop = group = fold = requant = 0;
    // these do not depend on the bracketing of their list, or are never rounded in between
    if (op == OP_REDUCE && (redop != RO_SUM || dt == DT_INT32)) group = 0, fold = FOLD_LIST;
    if (redop != RO_SUM || dt == DT_INT32 || dt == DT_FP32) requant = false;
    std::vector<uint64_t> v{op, redop, group, fold, requant ? 1u : 0u, dt};
    for (const Place& s : srcs) v.push_back(s.first), v.push_back(s.second);
    return v;
}

Writes from_steps(const HostProgram& p, uint32_t phase, const char* what) {
    Writes w;
    for (size_t i = 0; i < p.descs.size(); ++i) {
        if (p.desc_phase[i] != phase) continue;
        const HostDesc& d = p.descs[i];
        const uint64_t es = dtype_size(d.srcs[0].dtype);
        for (uint64_t e = 0; e < d.nelem; ++e) {
            std::vector<Place> s;
            for (const Operand& o : d.srcs) s.push_back({o.buf, o.offset + e * es});
            for (const Operand& o : d.dsts)
                write(w, {o.buf, o.offset + e * es}, value(d.op, d.redop, d.group, d.fold, d.requant, d.srcs[0].dtype, s), what);
        }
    }
    return w;
}

Writes from_uniform(const UniformPhase& u, uint64_t pad, const char* what) {
    Writes w;
    const uint64_t es = dtype_size(u.kernel.dtype);
    for (uint32_t g = 0; g < u.nseg; ++g) {
        const uint64_t n = g + 1 < u.nseg ? u.seg_elems : u.last_elems;
        const uint64_t tiles = (n + u.tile_elems - 1) / u.tile_elems;
        uint32_t rev = 0;
        for (uint32_t b = 1, t = u.nsrc() >> 1; b < u.nsrc(); b <<= 1, t >>= 1)
            if (g & b) rev |= t;
        for (uint64_t k = 0; k < tiles; ++k) {
            // tile 0 takes `pad` elements more than the others, which all start that much later
            const uint64_t e0 = k ? k * u.tile_elems + pad : 0, most = k ? u.tile_elems : u.tile_elems + pad;
            for (uint64_t e = e0; e < n && e < e0 + most; ++e) {
                std::vector<Place> s;
                for (uint32_t i = 0; i < u.nsrc(); ++i) {
                    uint32_t k2 = i;
                    if (u.flags & UF_ROTATE) k2 = (i + g + 1) % u.nsrc();
                    if (u.flags & UF_FLIP) k2 = i ^ rev;
                    const Operand& o = u.srcs[u.flags & UF_SRC_PER_SEG ? g : k2];
                    s.push_back({o.buf, o.offset + g * u.src_step + e * es});
                }
                for (uint32_t j = 0; j < u.ndst(); ++j) {
                    const Operand& o = u.dsts[u.flags & UF_DST_PER_SEG ? g : j];
                    const Place d{o.buf, o.offset + g * u.dst_step + e * es};
                    if (u.kernel.op == OP_COPY && d == s[0]) continue;
                    write(w, d, value(u.kernel.op, u.kernel.redop, u.group, u.kernel.fold, u.kernel.requant, u.kernel.dtype, s), what);
                }
            }
        }
    }
    return w;
}

// The copies of a program's list, found tile by tile as the kernel finds them, in 2-byte units.
Writes from_list(const HostProgram& p, const char* what) {
    Writes w;
    const uint8_t* base = p.image.data() + p.list_offset;
    const uint32_t* ends = (const uint32_t*)base;
    const uint32_t n = p.list_entries;
    const CopyEntry* entries = (const CopyEntry*)(base + 256 + 256 * ((n + 63) / 64));
    for (uint32_t t = 0; t < p.list_tiles; ++t) {
        uint32_t b = 0, i = 0;
        if (n > 64)
            for (uint32_t l = 0; l < 64; ++l) b += ends[l] <= t;
        for (uint32_t l = 0; l < 64; ++l) i += ends[64 + 64 * b + l] <= t;
        const CopyEntry& e = entries[64 * b + i];
        const uint64_t pad = (t - e.tile0) ? 10 : 0;  // tile 0 takes 10 units more, the others start later
        const uint64_t first = (uint64_t)(t - e.tile0) * (kListTileBytes / 2) + pad;
        const uint64_t most = kListTileBytes / 2 + (t == e.tile0 ? 10 : 0);
        for (uint64_t k = first; k < first + most && k < e.bytes / 2; ++k)
            write(w, {e.bufs >> 16, e.dst_off + 2 * k}, {e.bufs & 0xFFFFu, e.src_off + 2 * k}, what);
    }
    return w;
}

Writes halves_of_steps(const HostProgram& p, const char* what) {
    Writes w;
    for (const HostDesc& d : p.descs)
        for (uint64_t k = 0; k < d.nelem * dtype_size(d.srcs[0].dtype) / 2; ++k)
            write(w, {d.dsts[0].buf, d.dsts[0].offset + 2 * k}, {d.srcs[0].buf, d.srcs[0].offset + 2 * k}, what);
    return w;
}

CollectiveSpec exchange(int P, int dtype, uint64_t rows, uint64_t width, uint64_t chunk, uint32_t seed) {
    CollectiveSpec s;
    s.coll = COLL_ALLTOALLV;
    s.P = P;
    s.dtype = dtype;
    s.chunk_bytes = chunk;
    s.sendcounts.resize(P * P), s.sdispls.resize(P * P), s.recvcounts.resize(P * P), s.rdispls.resize(P * P);
    auto next = [&] { return (seed = seed * 1664525u + 1013904223u) >> 8; };
    for (int i = 0; i < P * P; ++i) s.sendcounts[i] = next() % 3 ? next() % (rows + 1) * width : 0;
    for (int a = 0; a < P; ++a) {
        uint64_t so = next() % 3, ro = next() % 3;
        for (int b = 0; b < P; ++b) {
            s.sdispls[a * P + b] = so, so += s.sendcounts[a * P + b] + (b % 2);
            s.recvcounts[a * P + b] = s.sendcounts[b * P + a];
            s.rdispls[a * P + b] = ro, ro += s.recvcounts[a * P + b] + (a % 2);
        }
    }
    return s;
}

void lists() {
    for (int P : {1, 2, 8, 9, 24})
        for (uint64_t chunk : {uint64_t(0), uint64_t(512)})
            for (int grouped = 0; grouped < 2; ++grouped) {
                const std::string what = "exchange P " + std::to_string(P) + " chunk " + std::to_string(chunk) + " grouped " + std::to_string(grouped);
                std::vector<CollectiveSpec> specs{exchange(P, DT_BF16, 9, P < 9 ? 701 : 5, chunk, P)};
                if (grouped) specs.push_back(exchange(P, DT_INT32, 9, 1, chunk, P + 1));
                std::vector<HostProgram> parts(specs.size());
                std::string err;
                for (size_t k = 0; k < specs.size(); ++k) lower(specs[k], parts[k], err), fuse(parts[k]);
                HostProgram p;
                if (grouped) merge(parts, specs, p, err);
                else p = parts[0];
                finalize(p, 0, err);
                ++programs;
                if (p.descs.empty() || p.uniform[0].ok) continue;
                if (!p.list_entries || from_list(p, what.c_str()) != halves_of_steps(p, what.c_str())) {
                    std::printf("LIST DIFFERS %s\n", what.c_str());
                    ++bad;
                }
            }
}

}  // namespace

int main() {
    lists();
    const int algos[] = {ALGO_AUTO, ALGO_DIRECT, ALGO_RING, ALGO_RHD, ALGO_TWO_LEVEL};
    struct Shape { int P; uint64_t count; };
    const Shape shapes[] = {{1, 5}, {2, 1}, {2, 777}, {3, 700}, {4, 129}, {8, 300}, {8, 8 * 64}, {16, 70}, {64, 3}};
    for (int coll : {COLL_ALLREDUCE, COLL_REDUCE_SCATTER, COLL_ALLGATHER})
        for (int algo : algos)
            for (int order : {ORDER_ASCENDING, ORDER_RING, ORDER_HALVING})
                for (const Shape& sh : shapes)
                    for (uint64_t chunk : {uint64_t(0), uint64_t(256)})
                        for (int n = 0; n < 3; ++n) {
                            const int variant = turn++ % 6;
                            CollectiveSpec s;
                            s.coll = coll;
                            s.P = sh.P;
                            s.count = sh.count;
                            s.algo = algo;
                            s.order = order;
                            s.chunk_bytes = chunk;
                            s.dtype = (const int[]){DT_BF16, DT_FP32, DT_INT32, DT_FP16, DT_BF16, DT_FP32}[variant];
                            s.redop = (const int[]){RO_SUM, RO_SUM, RO_SUM, RO_MAX, RO_SUM, RO_MIN}[variant];
                            s.requant = variant == 4;
                            s.phases = variant == 1 ? PHASE_LEVELS : PHASE_AUTO;
                            s.fuse = !(variant == 5 && sh.P == 8);
                            s.tile_bytes = variant == 2 && sh.P == 4 ? 4096 : 0;
                            s.group_size = sh.P % 8 == 0 ? 8 : sh.P % 2 == 0 ? 2 : 0;
                            HostProgram p;
                            std::string err;
                            if (!lower(s, p, err)) continue;
                            if (s.fuse) fuse(p);
                            if (!finalize(p, s.tile_bytes, err)) continue;
                            ++programs;
                            const std::string what = "coll " + std::to_string(coll) + " algo " + std::to_string(algo) + " order " +
                                std::to_string(order) + " P " + std::to_string(sh.P) + " count " + std::to_string(sh.count) +
                                " chunk " + std::to_string(chunk) + " variant " + std::to_string(variant);
                            for (uint32_t q = 0; q < p.nphase(); ++q) {
                                const UniformPhase& u = p.uniform[q];
                                if (!u.ok) {
                                    // the fused default schedules all have the form
                                    if (s.fuse && !s.tile_bytes && p.nphase() == 1 && !p.descs.empty() && sh.P <= 16) {
                                        std::printf("NOT UNIFORM %s\n", what.c_str());
                                        ++bad;
                                    }
                                    continue;
                                }
                                ++uniform;
                                const Writes a = from_steps(p, q, what.c_str());
                                for (uint64_t pad : {0, 31})
                                    if (a != from_uniform(u, pad, what.c_str())) {
                                        std::printf("DIFFERS %s phase %u pad %d\n", what.c_str(), q, (int)pad);
                                        ++bad;
                                    }
                            }
                        }
    std::printf("programs %d, uniform phases %d, bad %d\n", programs, uniform, bad);
    return bad || !uniform ? 1 : 0;
}
