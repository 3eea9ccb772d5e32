// What the forms that a launch may take (a uniform phase, a copy list) cost when a wide exchange is
// packed. Every pair of ranks is a step, and the forms are looked for among all of them: that search
// has to stay a pass or two over the steps, since an exchange whose counts change is compiled anew
// for each call. Packs the same steps with and without the search (a configured tile size has
// neither form), prints the least time of each over many rounds and their ratio; exit status 1 where
// the ratio is above the limit given as an argument.
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <string>

#include "compiler.h"

using namespace hccl;

namespace {

CollectiveSpec exchange(int P, uint64_t rows, uint64_t width) {
    CollectiveSpec s;
    s.coll = COLL_ALLTOALLV;
    s.P = P;
    s.dtype = DT_BF16;
    s.sendcounts.resize(P * P), s.sdispls.resize(P * P), s.recvcounts.resize(P * P), s.rdispls.resize(P * P);
    uint32_t seed = 7;
    for (uint64_t& c : s.sendcounts) c = (1 + ((seed = seed * 1664525u + 1013904223u) >> 8) % (2 * rows / P)) * width;
    for (int a = 0; a < P; ++a) {
        uint64_t so = 0, ro = 0;
        for (int b = 0; b < P; ++b) {
            s.sdispls[a * P + b] = so, so += s.sendcounts[a * P + b];
            s.recvcounts[a * P + b] = s.sendcounts[b * P + a];
            s.rdispls[a * P + b] = ro, ro += s.recvcounts[a * P + b];
        }
    }
    return s;
}

double us(std::chrono::steady_clock::time_point a, std::chrono::steady_clock::time_point b) {
    return std::chrono::duration<double, std::micro>(b - a).count();
}

}  // namespace

int main(int argc, char** argv) {
    const double limit = argc > 1 ? std::atof(argv[1]) : 1e9;
    const CollectiveSpec s = exchange(64, 256, 2048);
    HostProgram lowered;
    std::string err;
    if (!lower(s, lowered, err)) return 2;
    double with = 1e9, without = 1e9;
    for (int i = 0; i < 200; ++i) {
        HostProgram a = lowered, b = lowered;
        const auto t0 = std::chrono::steady_clock::now();
        if (!finalize(a, 0, err) || a.list_entries == 0) return 2;
        const auto t1 = std::chrono::steady_clock::now();
        if (!finalize(b, 8192, err) || b.list_entries != 0 || b.ntiles != a.ntiles) return 2;
        const auto t2 = std::chrono::steady_clock::now();
        with = std::min(with, us(t0, t1));
        without = std::min(without, us(t1, t2));
    }
    std::printf("64-rank exchange: packed in %.0f us, without the forms %.0f us, ratio %.2f\n", with, without, with / without);
    return with > limit * without ? 1 : 0;
}
