// How runs and batch classes are shared out (pimc_split.hpp): one line per problem for the checks in Python.
#include <cstdio>

#include "pimc_split.hpp"

using namespace pimc;

int main() {
    for (uint64_t wgs : {256, 512})
        for (int s = 1; s <= 12; ++s)
            for (int slots : {0, 1, s + 1})
                for (uint64_t n : {2ull, 64ull, 65ull, 4096ull, 100001ull, 900000ull, 2000000ull, 2097152ull, 2097153ull, 3000001ull,
                                   4000000ull, 5000000ull, 7000000ull, 20000000ull, 100000000ull, 1000000007ull, 1ull << 40}) {
                    const PathWork w = split_paths(n, s, slots, kFineBytes, wgs, 4);
                    std::printf("run %llu %d %d %llu %llu %llu %llu %llu %llu %u\n", (unsigned long long)wgs, s, slots,
                                (unsigned long long)n, (unsigned long long)w.n_groups, (unsigned long long)w.n_chunks,
                                (unsigned long long)w.n_coarse, (unsigned long long)w.fine(), (unsigned long long)w.n_static, w.grab);
                }
    return 0;
}
