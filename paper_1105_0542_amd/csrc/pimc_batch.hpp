// Persistent batched estimation kernel (the walker of pimc_walker.hpp over an atomic queue of
// (task, chunk) items) for the quartic evaluators, and the launch-shape lists the autotuner picks
// from. Included by pimc_kernels_batch.hip (default shapes, every p) and one translation unit per
// tuned level p (pimc_batch_p*.hip), so the variants compile in parallel.
#pragma once

#include <hip/hip_runtime.h>

#include "pimc_walker.hpp"

namespace pimc {

template <class... Ss>
struct ShapeList {
    static constexpr int size = sizeof...(Ss);
};

// Candidate shapes of the tuned classes. Tasks with N >= 32 may use 4- or 5-level subtrees; tasks
// with N = 16 (s = 4) have at most 4. Shape 0 of each list is the default (the single-call shape).
using BatchShapesN32 = ShapeList<Shape<4, 256, 2, 16>, Shape<4, 256, 2, 8>, Shape<5, 256, 2, 16>, Shape<5, 256, 2, 8>,
                                 Shape<4, 128, 2, 16>, Shape<4, 256, 1, 16>, Shape<4, 256, 3, 8>, Shape<4, 64, 2, 16>>;
using BatchShapesN16 = ShapeList<Shape<4, 256, 2, 16>, Shape<4, 256, 2, 8>, Shape<4, 128, 2, 16>, Shape<4, 256, 3, 8>,
                                 Shape<4, 256, 1, 16>>;
using BatchDefaultN32 = ShapeList<DefaultShape<4>>;
using BatchDefaultN16 = ShapeList<DefaultShape<4>>;

// Persistent kernel over the items of one class (level p, launch shape), numbered task by task (task t
// owns items item0[t] .. item0[t+1] - 1), so an item maps to its task by binary search over the
// wave-uniform task records. An item is
//   * by group (classes of few chunks, by batch_by_group): `block` consecutive groups, taken by one wave, whose sums are stored
//     and added into the chunk records afterwards (pimc_chunks.hpp: the same sums as any other split). A
//     task of 20,000 paths has 5 chunks, a class of 85 such tasks 425 of them for 512 resident
//     workgroups, those with N = 512 16 times as long as those with N = 32. The first n_static items are
//     dealt to the waves in turn;
//   * a whole chunk (every other class), taken by a workgroup.
// The other items are taken `grab` at a time from an atomic counter until it passes n_items; every wave (by
// group) or workgroup (by chunk) reaches the exit test with one value.
// Two kernels: in one the branches cost the chunks 3 % (4 tasks of 2e7 paths, N = 16, p = 4: 2.77 and 2.86 ms).
template <class S, class Eval, bool BY_GROUP>
__global__ void __launch_bounds__(S::BS) __attribute__((amdgpu_waves_per_eu(S::WPE)))
k_batch(BatchArgs B, Eval ev0) {
    extern __shared__ double smem[];
    __shared__ unsigned long long s_item;
    constexpr int WAVES = S::BS / 64;
    const const_ptr<BatchTask> T = as_const(B.tasks);
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    load_bm_table(smem, S::BS);
    __syncthreads();
    auto take = [&]() -> unsigned long long {
        unsigned long long t = 0;
        if ((tid & 63) == 0) t = atomicAdd(B.queue, (unsigned long long)B.grab);
        return t;
    };
    uint64_t deal = uint64_t(blockIdx.x) * WAVES + uint64_t(wave);
    unsigned long long ticket = 0;
    if (BY_GROUP && B.n_static < B.n_items) ticket = take();
    while (true) {
        uint64_t first, end;
        if (BY_GROUP && deal < B.n_static) {
            first = deal;
            end = deal + 1;
            deal += uint64_t(gridDim.x) * WAVES;
        } else {
            if (BY_GROUP) {
                first = B.n_static + uniform_u64(ticket);
                if (first >= B.n_items) break;
                ticket = take();
            } else {
                __syncthreads();
                if (tid == 0) s_item = atomicAdd(B.queue, (unsigned long long)B.grab);
                __syncthreads();
                first = uniform_u64(s_item);
                if (first >= B.n_items) break;
            }
            end = first + B.grab < B.n_items ? first + B.grab : B.n_items;
        }
        for (uint64_t item = first; item < end; ++item) {
            int lo = 0, hi = B.n_tasks - 1;                  // last task with item0 <= item
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (T[mid].item0 <= item) lo = mid; else hi = mid - 1;
            }
            AmpArgs A;
            A.tab64 = T[lo].tab;
            A.tab32 = nullptr;
            A.gdeg = nullptr;
            A.gK = 0;
            A.gstride = 0;
            A.a = T[lo].a;
            A.b = T[lo].b;
            A.sig = T[lo].sig;
            A.shift = T[lo].shift;
            A.key = B.key;
            A.key.stream = T[lo].stream;
            A.first_path = 0;
            A.n_paths = T[lo].n_paths;
            A.work = PathWork{};
            A.s = T[lo].s;
            A.D = T[lo].s - S::U;
            A.hier = B.hier;
            A.partials = T[lo].partials;
            A.dump = nullptr;
            Eval ev = ev0;
            ev.tab = T[lo].tab;
            const int nlev = A.s + 1;
            const uint64_t n_groups = (A.n_paths + 63) / 64;
            double* acc = smem + kBoxMullerTable + size_t(3 * A.D + 2) * S::BS;
            uint64_t g = item - T[lo].item0, last, step = 1;
            if (BY_GROUP) {
                g *= T[lo].block;
                last = g + T[lo].block;
            } else {
                for (int i = tid; i < kChunkSlots * nlev * 3; i += S::BS) acc[i] = 0.0;
                __syncthreads();
                g = g * kChunkGroups + uint64_t(wave);
                last = g - uint64_t(wave) + kChunkGroups;
                step = WAVES;
            }
            if (last > n_groups) last = n_groups;
            for (; g < last; g += step) {
                process_group<S, Eval>(ev, A, g, [&]() __attribute__((always_inline)) {
                    if constexpr (BY_GROUP) return GroupSink{false, nullptr, (gdouble*)T[lo].gsum + g * 3, n_groups * 3};
                    return GroupSink{true, acc + int(g % kChunkSlots) * nlev * 3, nullptr, 0};
                }, smem, smem + kBoxMullerTable + tid);
            }
            if (!BY_GROUP) {
                __syncthreads();
                write_chunk(acc, nlev, B.hier, A.partials, T[lo].n_chunks, item - T[lo].item0, A.n_paths, tid);
                __syncthreads();
            }
        }
    }
}

// Shape idx of a list: launch, occupancy and description.
template <int P, class List>
struct BatchLauncher;

template <int P>
struct BatchLauncher<P, ShapeList<>> {
    static hipError_t launch(int, const BatchArgs&, int, size_t, hipStream_t) { return hipErrorInvalidValue; }
    static int resident(int, size_t, int) { return 0; }
    static bool desc(int, ShapeDesc&) { return false; }
};

template <int P, class S0, class... Ss>
struct BatchLauncher<P, ShapeList<S0, Ss...>> {
    using Rest = BatchLauncher<P, ShapeList<Ss...>>;
    static hipError_t launch(int idx, const BatchArgs& B, int grid, size_t lds, hipStream_t st) {
        if (idx != 0) return Rest::launch(idx - 1, B, grid, lds, st);
        QuarticEval64<P> ev{nullptr};
        if (B.by_group)
            hipLaunchKernelGGL((k_batch<S0, QuarticEval64<P>, true>), dim3(grid), dim3(S0::BS), lds, st, B, ev);
        else
            hipLaunchKernelGGL((k_batch<S0, QuarticEval64<P>, false>), dim3(grid), dim3(S0::BS), lds, st, B, ev);
        return hipGetLastError();
    }
    static int resident(int idx, size_t lds, int device) {
        if (idx != 0) return Rest::resident(idx - 1, lds, device);
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_batch<S0, QuarticEval64<P>, false>, S0::BS, lds) !=
            hipSuccess)
            per_cu = 1;
        int ncu = 0;
        if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) ncu = 256;
        return (per_cu < 1 ? 1 : per_cu) * ncu;
    }
    static bool desc(int idx, ShapeDesc& d) {
        if (idx != 0) return Rest::desc(idx - 1, d);
        d = ShapeDesc{S0::U, S0::BS, S0::WPE, S0::BATCH};
        return true;
    }
};

// The tuned classes of level P (defined in pimc_batch_p<P>.hip).
#define PIMC_BATCH_TUNED_DECL(P)                                                                                      \
    hipError_t launch_batch_tuned_##P(bool n16, int idx, const BatchArgs& B, int grid, size_t lds, hipStream_t st);   \
    int resident_batch_tuned_##P(bool n16, int idx, size_t lds, int device);

#define PIMC_BATCH_TUNED_DEF(P)                                                                                       \
    hipError_t launch_batch_tuned_##P(bool n16, int idx, const BatchArgs& B, int grid, size_t lds, hipStream_t st) {  \
        return n16 ? BatchLauncher<P, BatchShapesN16>::launch(idx, B, grid, lds, st)                                  \
                   : BatchLauncher<P, BatchShapesN32>::launch(idx, B, grid, lds, st);                                 \
    }                                                                                                                 \
    int resident_batch_tuned_##P(bool n16, int idx, size_t lds, int device) {                                         \
        return n16 ? BatchLauncher<P, BatchShapesN16>::resident(idx, lds, device)                                     \
                   : BatchLauncher<P, BatchShapesN32>::resident(idx, lds, device);                                    \
    }

PIMC_BATCH_TUNED_DECL(8)
PIMC_BATCH_TUNED_DECL(12)
PIMC_BATCH_TUNED_DECL(18)

}  // namespace pimc
