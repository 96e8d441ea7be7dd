// How the estimation kernels share out the paths of a run, and the sums of a group of paths.
//
// A group is 64 consecutive paths, the lanes of one wave; a canonical chunk is 64 groups
// (pimc_internal.hpp). Two kinds of work share one persistent kernel:
//   * coarse chunks 0 .. n_coarse-1: a workgroup takes a whole chunk from a counter, its waves walk the
//     chunk's groups and add their sums in LDS, and the chunk's record is written once;
//   * fine groups, those of the chunks from n_coarse on: every wave walks groups by itself and stores
//     each group's sums; k_group_chunks adds them into the chunk records afterwards. The first
//     n_static fine groups are dealt to the waves in turn, the others go by ticket from a second counter.
// Both add in the order fixed by the path indices, so a chunk's bits do not depend on its kind.
//
// Why two kinds. A group costs from microseconds (N = 16) to milliseconds, and a GPU of 256 CUs holds
// 2048 waves at two per SIMD. With whole chunks alone a run below 512 x 4096 = 2.1e6 paths left
// workgroups without work, and above it the last round was part empty. Group sums are 24 bytes per
// group and level, so a whole run of 1e9 paths cannot keep them; the last kFineBytes worth are enough
// to fill every wave many times over.
// Why two ways of sharing out. Tickets are 8 ns each for the whole GPU (2048 waves on one counter),
// 16 us for a round of all waves: nothing beside groups of N >= 64 slices, much of the time of smaller
// ones (a call with 1e5 paths at N = 16, every level: whole chunks 156 us, tickets 109 us, dealt 75
// us). But waves drift apart, so the last rounds of long groups go by ticket.
// Measured, calls with every level, whole chunks against this: 1e6 paths at N = 1024, p = 10
// (Poeschl-Teller) 16.3 -> 13.3 ms; 3e5 at N = 64, p = 6 (sextic) 1.02 -> 0.28 ms; 5e4 at N = 64,
// p = 18 (general mode) 234 -> 42 ms; 2e7 at N = 1024, p = 18 (quartic) 102 -> 96 ms.
#pragma once

#include "pimc_device.hpp"
#include "pimc_internal.hpp"

namespace pimc {

__device__ __forceinline__ uint64_t uniform_u64(uint64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(v));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(uint32_t(v >> 32));
    return (uint64_t(hi) << 32) | lo;
}

// Where lane 0 puts a group's level sums (sum d, sum d^2, non-finite count): added to an accumulator
// slot in LDS, or stored to the group's place in device memory (stride: doubles between slots).
struct GroupSink {
    double* acc;                       // LDS, 3 doubles per level, or null
    double* out;                       // device, else
    uint64_t stride;
};

// The sums of one level over a group: d and d^2 by a wave butterfly, the non-finite count by a ballot.
__device__ __forceinline__ void reduce_level(const GroupSink& k, int lane, int slot, double S, double shift, bool valid) {
    const double d = valid ? expm1(-(S - shift)) : 0.0;
    const bool bad = valid && !isfinite(d);
    const double sd = wave_sum(d);
    const double sd2 = wave_sum(d * d);
    const double nb = double(__popcll(__ballot(bad)));
    if (lane == 0) {
        if (k.acc) {
            double* a = k.acc + slot * 3;
            a[0] += sd;
            a[1] += sd2;
            a[2] += nb;
        } else {
            double* a = k.out + uint64_t(slot) * k.stride;
            a[0] = sd;
            a[1] = sd2;
            a[2] = nb;
        }
    }
}

// A whole chunk's record from its accumulator slots, by one thread per evaluated level (tid < slots).
__device__ __forceinline__ void write_chunk(const double* acc, int nlev, int hier, double* partials, uint64_t n_chunks,
                                            uint64_t c, uint64_t n_paths, int tid) {
    if (tid >= (hier ? nlev : 1)) return;
    const uint64_t rem = n_paths - c * kChunkPaths;
    double s1 = 0.0, s2 = 0.0, nb = 0.0;
    for (int q = 0; q < kChunkSlots; ++q) {
        const double* a = acc + (q * nlev + tid) * 3;
        s1 += a[0];
        s2 += a[1];
        nb += a[2];
    }
    double* o = partials + (uint64_t(tid) * n_chunks + c) * 4;
    o[0] = double(rem < kChunkPaths ? rem : kChunkPaths);
    o[1] = s1;
    o[2] = s2;
    o[3] = nb;
}

// The persistent loop of one workgroup of BS threads. run(group, sink) walks the 64 paths of a group
// and reduces them into the sink (one call site: its code is the whole kernel); acc: the accumulator
// slots in LDS, kChunkSlots * nlev * 3 doubles. Every wave of a workgroup leaves the coarse phase at
// the same ticket, so its barriers are met by all; a fine ticket is asked for before the groups of the
// one in hand are walked (the answer is back long before it is needed).
template <int BS, class RunGroup>
__device__ __forceinline__ void run_groups(const PathWork& w, int nlev, int hier, uint64_t n_paths, double* partials,
                                           double* acc, RunGroup run) {
    constexpr int WAVES = BS / 64;
    __shared__ unsigned long long s_chunk;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint64_t fine0 = w.n_coarse * kChunkGroups;
    const uint64_t n_fine = w.n_groups > fine0 ? w.n_groups - fine0 : 0;
    auto take = [&]() -> unsigned long long {
        unsigned long long t = 0;
        if ((tid & 63) == 0) t = atomicAdd(w.queue + 1, (unsigned long long)w.grab);
        return w.n_static + t;
    };
    bool coarse = w.n_coarse > 0;
    uint64_t deal = coarse ? w.n_static : uint64_t(blockIdx.x) * WAVES + uint64_t(wave);   // next group dealt to this wave
    unsigned long long ticket = n_fine;
    if (!coarse && w.n_static < n_fine) ticket = take();
    while (true) {
        uint64_t g, last, step, c = 0;
        if (coarse) {
            __syncthreads();
            if (tid == 0) s_chunk = atomicAdd(w.queue, 1ull);
            __syncthreads();
            c = uniform_u64(s_chunk);
            if (c >= w.n_coarse) {
                coarse = false;
                if (w.n_static < n_fine) ticket = take();
                continue;
            }
            for (int i = tid; i < kChunkSlots * nlev * 3; i += BS) acc[i] = 0.0;
            __syncthreads();
            g = c * kChunkGroups + uint64_t(wave);
            last = (c + 1) * kChunkGroups;
            step = WAVES;
        } else if (deal < w.n_static) {
            g = fine0 + deal;
            last = fine0 + w.n_static;
            step = uint64_t(gridDim.x) * WAVES;
            deal = w.n_static;
        } else {
            const uint64_t f = uniform_u64(ticket);
            if (f >= n_fine) break;
            ticket = take();
            g = fine0 + f;
            last = g + w.grab;
            step = 1;
        }
        if (last > w.n_groups) last = w.n_groups;
        for (; g < last; g += step) {
            GroupSink k;
            k.acc = coarse ? acc + int(g % kChunkSlots) * nlev * 3 : nullptr;
            k.out = w.gsum + (g - fine0) * 3;
            k.stride = n_fine * 3;
            run(g, k);
        }
        if (coarse) {
            __syncthreads();
            write_chunk(acc, nlev, hier, partials, w.n_chunks, c, n_paths, tid);
        }
    }
}

// Reference actions on the device, for the evaluators whose slice costs too much on the host (24,196
// monomials at p = 18 of the general mode: 14 ms of host time at N = 64, 230 ms at N = 1024). Level n
// (blockIdx.x + 1) of the straight line from a to b: block y takes the y-th part of its 2^n slices, and
// the parts are added by k_line_sum. slice(level, k, N) is one slice's action. Parts and orders depend
// on n alone, so level n of an s-run has the reference of the n-run.
__host__ __device__ inline int line_parts(int n) { return n <= 8 ? 1 : (n >= 14 ? kLineParts : 1 << (n - 8)); }

template <class Slice>
__device__ __forceinline__ void line_part(double* __restrict__ parts, Slice slice) {
    const int n = int(blockIdx.x) + 1;
    const int np = line_parts(n);
    if (int(blockIdx.y) >= np) return;
    const int N = 1 << n, per = N / np;
    double S = 0.0;
    for (int i = threadIdx.x; i < per; i += kBlock) S += slice(n, int(blockIdx.y) * per + i, N);
    __shared__ double red[kBlock];
    red[threadIdx.x] = S;
    __syncthreads();
    for (int w = kBlock / 2; w >= 1; w >>= 1) {
        if (int(threadIdx.x) < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) parts[n * kLineParts + int(blockIdx.y)] = red[0];
}

}  // namespace pimc
