// How the paths of a run are shared out: the numbers that the kernels of pimc_chunks.hpp work by (host code).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <functional>
#include <queue>
#include <vector>

#include "pimc.h"

namespace pimc {

// Canonical chunk of the estimators: kChunkPaths consecutive path indices, in kChunkGroups groups of
// 64 consecutive paths (the lanes of one wave). A group's per-level sums are a wave butterfly;
// group g is added to accumulator slot g mod kChunkSlots, each slot in increasing g, and the chunk
// sum is slot 0 + slot 1 + slot 2 + slot 3. The order is fixed by the path indices alone, so the
// chunk sums -- and the amplitudes -- do not depend on the workgroup size (64, 128 or 256 lanes:
// wave w of a workgroup of W waves takes groups w, w + W, ..., and no two waves share a slot), on
// the subtree depth or slice batch of the walker, on N (level n of an s-run is bitwise the n-run),
// or on which workgroup ran the chunk.
constexpr uint32_t kChunkPaths = PIMC_CHUNK_PATHS;
constexpr int kChunkGroups = int(kChunkPaths / 64);
constexpr int kChunkSlots = 4;

// The paths of one launch (pimc_chunks.hpp): chunks 0 .. n_coarse-1 whole, the groups of the others
// (fine groups) one by one.
struct PathWork {
    uint64_t n_groups;                 // ceil(n_paths / 64)
    uint64_t n_chunks;                 // ceil(n_paths / kChunkPaths)
    uint64_t n_coarse;
    uint64_t n_static;                 // fine groups dealt to the waves in turn (none when n_coarse > 0)
    double* gsum;                      // device [slot][fine group][3], or null (per-path actions only)
    unsigned long long* queue;         // device: the coarse and the fine counter, 0 at launch
    uint32_t grab;                     // fine groups per ticket
    uint64_t fine() const { return n_groups > n_coarse * kChunkGroups ? n_groups - n_coarse * kChunkGroups : 0; }
};

// Group sums a run may keep: 24 bytes per group and level, 992 chunks (63,488 groups) with the eleven
// levels of N = 1024.
constexpr size_t kFineBytes = size_t(16) << 20;

// A ticket costs 12.4 ns of the whole GPU (one address, measured as the time of runs that it bounds), 25 us
// for one round of 2048 waves. The cheapest slice of a group takes a wave 0.22 us (quartic, p = 1, level s
// alone), so a ticket should be worth kTicketSlices of them.
constexpr uint32_t kTicketSlices = 128;
inline uint32_t ticket_groups(int s) { return s >= 7 ? 1u : (s >= 3 ? kTicketSlices >> s : 16u); }

// Whole chunks of a run of n_chunks chunks on wgs workgroups, R = n_chunks / wgs rounds.
//   R <= 1: none, with chunks workgroups would have no work (1e6 paths, N = 256, p = 18: 1.19 ms, 0.99 by group);
//   N <= 32: from R = 4 on all, the tail of a chunk is short there and tickets for short groups are dear (2e7 paths,
//     N = 8, p = 1: 1.1 times as long by group). Below that all where the last round is about half full, because one of the two
//     workgroups of a CU gets ahead of the other and then has one chunk more; else none, all groups are dealt in
//     turn. Time by chunk over dealt at R = 1.03, 1.25, 1.5, 1.75, 1.95, 2.05, 2.25, 2.5, 2.75, 3.1, 3.5, 4.1: quartic p = 18,
//     N = 8, every level 1.37 1.22 1.07 1.08 1.00 1.13 1.06 0.99 1.05 1.03 0.94 0.99; N = 32, level s alone 1.20 1.07
//     0.93 1.01 0.93 1.09 1.14 1.07 0.99 0.98 0.92 0.99; four coordinates, N = 8 1.19 1.04 0.94 1.25 1.17 1.12 1.06
//     0.99 1.01 1.08 1.06 1.01;
//   else full rounds, and what remains, 0.4 to 1.4 rounds, by group (one to two from R = 3 on, where workgroups
//     have drifted apart by a chunk): 5e6 paths, N = 256, p = 18, every level: 8.3 ms by chunk, 6.4; 1e7: 13.5 and
//     12.4. A remainder of whole chunks beside groups is worse than either (3e6 paths, 1.43 rounds, 0.43 of
//     them by chunk: 6.2 ms, 4.2 by chunk and 4.1 this way), the chunks then last longer than all the rest.
inline uint64_t whole_chunks(uint64_t n_chunks, int s, uint64_t wgs) {
    if (n_chunks <= wgs) return 0;
    if (s <= 5) {
        const uint64_t eighths = n_chunks * 8 / wgs;
        return eighths >= 32 || eighths % 8 == 3 || eighths % 8 == 4 ? n_chunks : 0;
    }
    const uint64_t r10 = n_chunks * 10 / wgs;
    return wgs * (r10 < 30 ? (r10 - 4) / 10 : r10 / 10 - 1);
}

// Split of a run of n_paths paths of N = 2^s slices over `slots` evaluated levels, on `resident` workgroups of
// `wg_waves` waves; fine_bytes: room for group sums (slots = 0: nothing is summed, every group is fine). Behind
// whole chunks the groups go by ticket. A run without them deals its groups to the waves in turn, the last
// quarter of the rounds (two at least) by ticket because waves drift apart; short groups (N < 64) are all dealt,
// as those rounds would take less than their tickets.
inline PathWork split_paths(uint64_t n_paths, int s, int slots, size_t fine_bytes, uint64_t resident, int wg_waves) {
    PathWork w{};
    w.n_groups = (n_paths + 63) / 64;
    w.n_chunks = (n_paths + kChunkPaths - 1) / kChunkPaths;
    const uint64_t wgs = std::max<uint64_t>(resident, 1), waves = wgs * uint64_t(wg_waves);
    if (slots) {
        const uint64_t fit = fine_bytes / (size_t(slots) * kChunkGroups * 24);
        w.n_coarse = whole_chunks(w.n_chunks, s, wgs);
        if (w.n_chunks - w.n_coarse > fit) w.n_coarse = s <= 5 && w.n_chunks > wgs ? w.n_chunks : w.n_chunks - fit;
    }
    w.grab = ticket_groups(s);
    if (!w.n_coarse) {
        const uint64_t rounds = w.n_groups / waves, tail = std::max<uint64_t>(rounds / 4, 2);
        if (rounds < 8 * w.grab) w.grab = 1;
        w.n_static = s < 6 || rounds < 1 ? w.n_groups : (rounds > tail ? (rounds - tail) * waves : 0);
    }
    return w;
}
// Bytes of its group sums.
inline size_t group_sum_bytes(const PathWork& w, int slots) { return size_t(slots) * size_t(w.fine()) * 24; }
// Workgroups of `waves_per_wg` waves that this work can occupy, at most `resident`.
inline int work_grid(const PathWork& w, int waves_per_wg, int resident) {
    const uint64_t wgs = w.n_coarse + ((w.fine() + w.grab - 1) / w.grab + uint64_t(waves_per_wg) - 1) / uint64_t(waves_per_wg);
    const uint64_t most = uint64_t(resident < 1 ? 1 : resident);
    return int(wgs < 1 ? 1 : (wgs < most ? wgs : most));
}

// Batches. The chunks of a class (the tasks of one level p that share a launch) go to workgroups in the order of
// the tasks, long paths first; cost: slices of groups of each chunk; groups: groups of them all. A class goes by
// group where that order would leave workgroups idle, for more than a seventh of the time below 64 slices a group
// (on average) and a twentieth below 128, because a group on its own costs up to 9 % more than within a chunk there
// (1500 tasks of 4096 paths, N = 32, p = 18 0.84 and 0.88 ms; 1024 of them, N = 64, two full rounds, 1.00 and 1.07); with longer
// ones always, for the waves of a SIMD don't keep step and the last of few long chunks are walked alone (1400 tasks of 4096
// paths, N = 32..512, p = 12 3.85 ms by chunk, 3.0 by group, where the order alone leaves 6 %).
constexpr uint64_t kBatchChunks = 4;          // chunks per workgroup from which the idle end no longer matters
inline bool batch_by_group(const std::vector<uint64_t>& cost, uint64_t groups, uint64_t wgs) {
    if (cost.empty() || cost.size() >= kBatchChunks * wgs) return false;
    std::priority_queue<uint64_t, std::vector<uint64_t>, std::greater<uint64_t>> busy;     // when each workgroup is free
    uint64_t total = 0, end = 0;
    for (uint64_t c : cost) {
        uint64_t t = c;
        if (busy.size() >= wgs) {
            t += busy.top();
            busy.pop();
        }
        busy.push(t);
        total += c;
        end = std::max(end, t);
    }
    if (total >= 128 * groups) return true;
    return total >= 64 * groups ? 20 * end * wgs > 21 * total : 7 * end * wgs > 8 * total;
}

// By group the items of a class, blocks of groups for single waves, are taken in the same order. share: slices
// of groups per wave. An item is a sixteenth of that, but at least an eighth or what a ticket should be worth and
// at most twice that. Where an eighth is less the items are all dealt, so that every wave gets the same mix; else
// the items of the first quarter of the work are, and those of the rest go by ticket (two rounds at least). A
// quarter of the items by ticket, the short ones: 85 tasks of 20,000 paths, N = 32..512, p = 18 1.21 ms, this way 1.14.
inline uint32_t batch_block(int s, uint64_t share) {
    const uint64_t most = std::min<uint64_t>(std::max<uint64_t>(share / 16, kTicketSlices), 2 * kTicketSlices);
    const uint64_t q = std::min(share / 8, most) >> s;
    return q < 1 ? 1u : uint32_t(q);
}
inline uint64_t batch_dealt(uint64_t n_items, uint64_t share, uint64_t waves, uint64_t ticket_items) {
    const uint64_t tail = std::max(2 * waves, ticket_items);
    return share < 8 * kTicketSlices ? n_items : (n_items > tail ? n_items - tail : 0);
}

}  // namespace pimc
