// How the estimation kernels share out the paths of a run, and the sums of a group of paths.
//
// A group is 64 consecutive paths, the lanes of one wave; a canonical chunk is 64 groups
// (pimc_split.hpp). Two kinds of work share one persistent kernel:
//   * coarse chunks 0 .. n_coarse-1: a workgroup takes a whole chunk from a counter, its waves walk the
//     chunk's groups and add their sums in LDS, and the chunk's record is written once;
//   * fine groups, those of the chunks from n_coarse on: every wave walks groups by itself and stores
//     each group's sums; k_group_chunks adds them into the chunk records afterwards. The first
//     n_static fine groups are dealt to the waves in turn, the others go by ticket from a second counter.
// Both add in the order fixed by the path indices, so a chunk's bits do not depend on its kind.
// pimc_split.hpp decides how many of each there are.
//
// Why two kinds. A group costs from microseconds (N = 16) to milliseconds, and a GPU of 256 CUs holds
// 2048 waves at two per SIMD. With whole chunks alone a run below 512 x 4096 = 2.1e6 paths leaves
// workgroups without work, and above it the last round is part empty.
// Measured, calls with every level, whole chunks against this: 1e5 paths at N = 16, p = 4 156 -> 67 us; 1e6
// at N = 1024, p = 10 (Poeschl-Teller) 16.3 -> 13.3 ms; 3e5 at N = 64, p = 6 (sextic) 1.02 -> 0.28 ms; 5e4 at
// N = 64, p = 18 (general mode) 234 -> 42 ms; 2e7 at N = 1024, p = 18 (quartic) 102 -> 96 ms.
#pragma once

#include "pimc_device.hpp"
#include "pimc_internal.hpp"

namespace pimc {

__device__ __forceinline__ uint64_t uniform_u64(uint64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(v));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(uint32_t(v >> 32));
    return (uint64_t(hi) << 32) | lo;
}
__device__ __forceinline__ uint32_t uniform_u32(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// Where lane 0 puts a group's level sums (sum d, sum d^2, non-finite count): added to an accumulator
// slot in LDS (whole chunks), or stored to the group's place in device memory (stride: doubles between levels).
typedef __attribute__((address_space(1))) double gdouble;
struct GroupSink {
    bool whole;
    double* acc;                       // LDS, 3 doubles per level
    gdouble* out;
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
        if (k.whole) {
            double* a = k.acc + slot * 3;
            a[0] += sd;
            a[1] += sd2;
            a[2] += nb;
        } else {
            gdouble* a = k.out + uint64_t(slot) * k.stride;
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

// The loop of one workgroup of BS threads over whole chunks.
template <int BS, class RunGroup>
__device__ __forceinline__ void run_chunks(const PathWork& w, int nlev, int hier, uint64_t n_paths, double* partials,
                                           double* acc, RunGroup run) {
    __shared__ unsigned long long s_chunk;
    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    while (true) {
        __syncthreads();
        if (tid == 0) s_chunk = atomicAdd(w.queue, 1ull);
        __syncthreads();
        const uint64_t c = uniform_u64(s_chunk);
        if (c >= w.n_chunks) break;
        for (int i = tid; i < kChunkSlots * nlev * 3; i += BS) acc[i] = 0.0;
        __syncthreads();
        for (int g = wave; g < kChunkGroups; g += BS / 64) {
            if ((c * kChunkGroups + uint64_t(g)) * 64 >= n_paths) break;   // wave-uniform: the rest of the chunk is empty
            run(c * kChunkGroups + uint64_t(g), [&]() __attribute__((always_inline)) {
                return GroupSink{true, acc + (g % kChunkSlots) * nlev * 3, nullptr, 0};
            });
        }
        __syncthreads();
        write_chunk(acc, nlev, hier, partials, w.n_chunks, c, n_paths, tid);
    }
}

// What the loop of a workgroup works by, in LDS. In registers (the launch's arguments are scalar) it would be
// live over the walk, whose constants take all scalar registers: 70 more lane reads a group to bring it back,
// 5 % of a call with 1e8 paths at N = 16, p = 1.
struct SharedWork {
    PathWork w;
    uint64_t fine0, n_fine;            // first fine group, fine groups
    unsigned long long chunk;          // the whole chunk in hand
};

// The persistent loop of one workgroup of BS threads. run(group, sink) walks the 64 paths of a group
// and reduces them into sink() (one call site: its code is the whole kernel); acc: the accumulator
// slots in LDS, kChunkSlots * nlev * 3 doubles. Every wave of a workgroup leaves the coarse phase at the same ticket, so its barriers are met by all. A ticket for fine groups is asked for before the groups of
// the one in hand are walked (the answer is back long before it is needed); one for a chunk only when the
// workgroup is free, or the last chunks would go to workgroups that are still at their last but one.
template <int BS, class RunGroup>
__device__ __forceinline__ void run_groups(const PathWork& w, int nlev, int hier, uint64_t n_paths, double* partials,
                                           double* acc, RunGroup run) {
    constexpr int WAVES = BS / 64;
    __shared__ SharedWork sw;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid == 0) {
        const uint64_t f0 = w.n_coarse * kChunkGroups;
        sw.w = w;
        sw.fine0 = f0;
        sw.n_fine = w.n_groups > f0 ? w.n_groups - f0 : 0;
    }
    auto take = [&](uint32_t grab) -> unsigned long long {         // the next ticket for fine groups (in lane 0)
        unsigned long long t = 0;
        if ((tid & 63) == 0) t = atomicAdd(w.queue + 1, (unsigned long long)grab);
        return t;
    };
    // Without a coarse phase the groups dealt to this wave come first: a wave of a short run has one, and every look
    // into LDS and barrier before it costs that run 0.1 us. (With their bounds from the arguments too, for them alone, the
    // component evaluator is 3 % slower in two coordinates.)
    bool coarse = w.n_coarse > 0, dealt = !coarse;
    unsigned long long ticket = 0;
    if (dealt && w.n_static < w.n_groups) ticket = take(w.grab);
    __syncthreads();
    while (true) {
        uint64_t g, last;
        uint32_t step;
        if (dealt) {
            dealt = false;
            g = uint64_t(blockIdx.x) * WAVES + uint64_t(wave);
            last = uniform_u64(sw.w.n_static);
            step = gridDim.x * WAVES;
        } else if (coarse) {
            __syncthreads();                                       // the chunk before is written
            if (tid == 0) sw.chunk = atomicAdd(w.queue, 1ull);
            __syncthreads();
            const uint64_t c = uniform_u64(sw.chunk);
            if (c >= uniform_u64(sw.w.n_coarse)) {
                coarse = false;
                if (uniform_u64(sw.n_fine) == 0) break;
                ticket = take(uniform_u32(sw.w.grab));
                continue;
            }
            for (int i = tid; i < kChunkSlots * nlev * 3; i += BS) acc[i] = 0.0;
            __syncthreads();
            g = c * kChunkGroups + uint64_t(wave);
            last = (c + 1) * kChunkGroups;
            step = WAVES;
            const uint64_t end = uniform_u64(sw.w.n_groups);
            if (last > end) last = end;
        } else {
            const uint64_t f = uniform_u64(sw.w.n_static) + uniform_u64(ticket), n = uniform_u64(sw.n_fine);
            if (f >= n) break;
            const uint32_t grab = uniform_u32(sw.w.grab);
            ticket = take(grab);
            g = uniform_u64(sw.fine0) + f;
            last = g + (n - f < grab ? n - f : grab);
            step = 1;
        }
        for (; g < last; g += step) {
            run(g, [&]() __attribute__((always_inline)) {
                if (coarse) return GroupSink{true, acc + int(g % kChunkSlots) * nlev * 3, nullptr, 0};
                return GroupSink{false, nullptr, (gdouble*)sw.w.gsum + (g - sw.fine0) * 3, sw.n_fine * 3};
            });
        }
        if (coarse) {
            __syncthreads();
            write_chunk(acc, nlev, hier, partials, sw.w.n_chunks, uniform_u64(sw.chunk), n_paths, tid);
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
