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
    // classes of k equal tasks of 2^s slices beside k / 8 of 512 slices, long paths first
    for (uint64_t wgs : {256, 512})
        for (int s : {4, 5, 6, 8, 10})
            for (int k : {1, 8, 40, 400, 5000, 50000})
                for (uint64_t n : {2ull, 100ull, 4096ull, 20000ull, 100001ull, 2000000ull}) {
                    std::vector<uint64_t> cost;
                    uint64_t share = 0, items = 0, all = 0;
                    for (int t = 0; t < k / 8 + k; ++t) {
                        const int st = t < k / 8 ? 9 : s;
                        const uint64_t groups = (n + 63) / 64;
                        share += groups << st;
                        all += groups;
                        for (uint64_t c = 0; c * 64 < groups && cost.size() < 65536; ++c)
                            cost.push_back(std::min<uint64_t>(groups - c * 64, 64) << st);
                    }
                    std::sort(cost.rbegin(), cost.rend());
                    const uint64_t waves = 4 * wgs;
                    uint64_t left = share / 4 * 3, by_ticket = 0;
                    share /= waves;
                    for (int t = k / 8 + k; t-- > 0;) {
                        const int st = t < k / 8 ? 9 : s;
                        const uint64_t b = batch_block(st, share), of_task = ((n + 63) / 64 + b - 1) / b;
                        const uint64_t taken = std::min(of_task, (left + (b << st) - 1) / (b << st));
                        items += of_task;
                        by_ticket += taken;
                        left -= std::min(left, taken * (b << st));
                    }
                    std::printf("class %llu %d %d %llu %llu %d %llu %u %llu %llu\n", (unsigned long long)wgs, s, k, (unsigned long long)n,
                                (unsigned long long)cost.size(), batch_by_group(cost, all, wgs) ? 1 : 0, (unsigned long long)share,
                                batch_block(s, share), (unsigned long long)items, (unsigned long long)batch_dealt(items, share, waves, by_ticket));
                }
    // k tasks of 64 groups, N = 32 << i % kinds first, long paths first, on 512 workgroups
    for (int k : {512, 700, 1024, 1400, 2000, 3000})
        for (int kinds : {1, 2, 3, 5})
            for (int s : {5, 6, 8}) {
                std::vector<uint64_t> cost;
                for (int t = 0; t < k; ++t) cost.push_back(64ull << (s + t % kinds));
                std::sort(cost.rbegin(), cost.rend());
                uint64_t total = 0;
                for (uint64_t c : cost) total += c;
                std::printf("mix %d %d %d %llu %d\n", k, kinds, s, (unsigned long long)(total / (64ull * uint64_t(k))),
                            batch_by_group(cost, 64ull * uint64_t(k), 512) ? 1 : 0);
            }
    return 0;
}
