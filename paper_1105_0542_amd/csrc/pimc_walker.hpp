// The bisection walker and estimation kernel template of the PIMC amplitude (Sec. 4 of Balaz et al.)
// for gfx950, shared by the translation units that instantiate it with their slice evaluators.
//
// One lane owns one path at a time. The path is built depth first, left to right, and never
// leaves the lane: the bottom U bisection levels of each subtree live in registers (2^U + 1
// points), the levels above them keep one pending right endpoint and one cached sibling normal per
// level in LDS. Every level-n slice is evaluated as soon as both of its endpoints exist, which for
// n < s is the moment its midpoint (a level-(n+1) node) is generated; the level-s slices are the
// leaves. Levels D..s of a subtree are evaluated coefficient-major over the slices of the level
// (up to BATCH at once) so that each wave-uniform table coefficient feeds independent FMA chains.
//
// Per level, each path's weight enters as d = exp(-(S_n - S_ref,n)) - 1 (a shift by the
// straight-line action only changes rounding); a wave butterfly sums d and d^2 over a group of 64
// consecutive paths, and lane 0 adds the group sum to the group's accumulator slot (canonical
// chunk, pimc_internal.hpp); at the end of a chunk the slots are added in slot order and written to
// the chunk's record. The chunk records are summed in chunk order by k_seg_reduce, so the result is
// bitwise independent of the launch shape, of the grid size, of which workgroup ran which chunk,
// and of whether the run was launched alone or as one task of a batch.
#pragma once

#include <hip/hip_runtime.h>

#include "pimc_chunks.hpp"
#include "pimc_internal.hpp"

namespace pimc {

// ---------------------------------------------------------------------------- subtree (registers)
template <int U, int L, class Src>
__device__ __forceinline__ void gen_level(const AmpArgs& A, const Src& src, uint32_t root, int D,
                                          double (&q)[(1 << U) + 1]) {
    if constexpr (L <= U) {
        constexpr int step = 1 << (U - L);
        const double sg = as_const(A.sig)[D + L];
#pragma unroll
        for (int i2 = 0; i2 < (1 << (L - 2)); ++i2) {
            const uint32_t parent = (root << (L - 2)) + uint32_t(i2);   // node of sub-level L-1
            double ze, zo;
            src.pair(parent, ze, zo);                                    // children 2*parent, 2*parent+1
            const int jl = (4 * i2 + 1) * step;
            const int jr = (4 * i2 + 3) * step;
            q[jl] = sg * ze + 0.5 * (q[jl - step] + q[jl + step]);
            q[jr] = sg * zo + 0.5 * (q[jr - step] + q[jr + step]);
        }
        gen_level<U, L + 1, Src>(A, src, root, D, q);
    }
}

// Add the 2^L slices of sub-level L (point stride 2^(U-L)) at tree level `level` to S, left to right.
template <int U, int BATCH, int L, class Eval>
__device__ __forceinline__ void level_sum(const Eval& ev, int level, const double (&q)[(1 << U) + 1], double& S) {
    constexpr int W = 1 << L;
    constexpr int ST = 1 << (U - L);
    constexpr int B = W < BATCH ? W : BATCH;
#pragma unroll
    for (int b0 = 0; b0 < W; b0 += B) {
        double qa[B], qb[B];
#pragma unroll
        for (int i = 0; i < B; ++i) {
            qa[i] = q[(b0 + i) * ST];
            qb[i] = q[(b0 + i + 1) * ST];
        }
        ev.template eval<B>(level, qa, qb, S);
    }
}

template <int U, int BATCH, int L, class Eval>
__device__ __forceinline__ void hier_levels(const Eval& ev, int D, const double (&q)[(1 << U) + 1],
                                            double (&Ssub)[U + 1]) {
    if constexpr (L < U) {
        level_sum<U, BATCH, L, Eval>(ev, D + L, q, Ssub[L]);
        hier_levels<U, BATCH, L + 1, Eval>(ev, D, q, Ssub);
    }
}

// Subtree rooted at heap node `root` (level D+1) over the level-D slice (qL, qR) with root normal z.
template <int U, int BATCH, class Eval, class Src>
__device__ __forceinline__ void run_subtree(const Eval& ev_in, const AmpArgs& A, const Src& src,
                                            uint32_t root, int D, double qL, double qR, double zroot,
                                            double (&Ssub)[U + 1]) {
    Eval ev = ev_in;
    ev.launder();
    double q[(1 << U) + 1];
    q[0] = qL;
    q[1 << U] = qR;
    q[1 << (U - 1)] = as_const(A.sig)[D + 1] * zroot + 0.5 * (qL + qR);
    gen_level<U, 2, Src>(A, src, root, D, q);
    if (A.hier) hier_levels<U, BATCH, 0, Eval>(ev, D, q, Ssub);
    level_sum<U, BATCH, U, Eval>(ev, D + U, q, Ssub[U]);
}

// ---------------------------------------------------------------------------- one path
// top: this lane's LDS slots (stride BS): S_top[n] at slot n (n < D), pending right endpoint
// of level L at slot D+L, pending normal at slot 2D+1+L (L = 2..D).
template <int U, int BS, int BATCH, class Eval, class Src>
__device__ __forceinline__ void walk_path(const Eval& ev, const AmpArgs& A, const Src& src, double* top,
                                          double (&Ssub)[U + 1]) {
    const int D = A.D;
#pragma unroll
    for (int j = 0; j <= U; ++j) Ssub[j] = 0.0;
    double z0_unused, z1;
    src.pair(0u, z0_unused, z1);                      // node 1 = sine output of call 0
    if (D == 0) {
        run_subtree<U, BATCH, Eval, Src>(ev, A, src, 1u, 0, A.a, A.b, z1, Ssub);
        return;
    }
    for (int n = 0; n < D; ++n) top[n * BS] = 0.0;
    double* R = top + D * BS;
    double* Z = top + (2 * D + 1) * BS;
    const uint32_t nTop = 1u << (D - 1);             // level-D nodes nTop .. 2 nTop - 1
    double qlast = A.a;
    for (uint32_t J = 0; J < nTop; ++J) {
        int L;
        uint32_t node;
        double qL = qlast, qR, z;
        if (J == 0) {
            L = 1;
            node = 1u;
            qR = A.b;
            z = z1;
        } else {
            const int t = __builtin_ctz(J);
            L = D - t;
            node = (nTop + J) >> t;
            qR = R[L * BS];
            z = Z[L * BS];
        }
        double qm, zl, zr;
        while (true) {
            if (A.hier) {
                const double qa1[1] = {qL};
                const double qb1[1] = {qR};
                double St = top[(L - 1) * BS];
                ev.template eval<1>(L - 1, qa1, qb1, St);
                top[(L - 1) * BS] = St;
            }
            qm = as_const(A.sig)[L] * z + 0.5 * (qL + qR);
            src.pair(node, zl, zr);
            if (L == D) break;
            R[(L + 1) * BS] = qR;                     // right child of `node`: (qm, qR), normal zr
            Z[(L + 1) * BS] = zr;
            qR = qm;
            z = zl;
            node = 2u * node;
            ++L;
        }
        run_subtree<U, BATCH, Eval, Src>(ev, A, src, 2u * node, D, qL, qm, zl, Ssub);
        run_subtree<U, BATCH, Eval, Src>(ev, A, src, 2u * node + 1u, D, qm, qR, zr, Ssub);
        qlast = qR;
    }
}

// ---------------------------------------------------------------------------- estimation kernel
// One group: paths 64 g + lane of the run described by A. Its level sums go to sink() (slot = level
// with every level evaluated, else 0 for level s) when A.partials is set, the per-path level actions to
// A.dump when that is. bm: the Box-Muller table, top: this lane's stack (both LDS).
template <class S, class Eval, class Sink>
__device__ __forceinline__ void process_group(const Eval& ev, const AmpArgs& A, uint64_t g, Sink sink,
                                              const double* bm, double* top) {
    constexpr int U = S::U;
    constexpr int BS = S::BS;
    const int lane = threadIdx.x & 63;
    const int D = A.D;
    const uint64_t local = g * 64 + uint64_t(lane);
    const bool valid = local < A.n_paths;
    double Ssub[U + 1];
    const PhiloxSource src{A.key, path_rng(A.key, A.first_path + local), bm};
    walk_path<U, BS, S::BATCH, Eval, PhiloxSource>(ev, A, src, top, Ssub);
    if (A.dump && valid) {
        double* o = A.dump + local * uint64_t(A.s + 1);
        for (int n = 0; n < D; ++n) o[n] = A.hier ? top[n * BS] : 0.0;
#pragma unroll
        for (int j = 0; j <= U; ++j) o[D + j] = (A.hier || j == U) ? Ssub[j] : 0.0;
    }
    if (A.partials) {
        const GroupSink k = sink();
        const const_ptr<double> shift = as_const(A.shift);
        if (A.hier) {
            for (int n = 0; n < D; ++n) reduce_level(k, lane, n, top[n * BS], shift[n], valid);
#pragma unroll
            for (int j = 0; j < U; ++j) reduce_level(k, lane, D + j, Ssub[j], shift[D + j], valid);
        }
        reduce_level(k, lane, A.hier ? D + U : 0, Ssub[U], shift[D + U], valid);
    }
}

// LDS of a workgroup: the Box-Muller table, the per-lane stacks, the accumulator slots.
// WHOLE: a run of whole chunks alone.
template <class S, class Eval, bool WHOLE>
__global__ void __launch_bounds__(S::BS) __attribute__((amdgpu_waves_per_eu(S::WPE)))
k_amplitude(AmpArgs A, Eval ev) {
    extern __shared__ double smem[];
    load_bm_table(smem, S::BS);     // the loops below begin with a barrier
    double* top = smem + kBoxMullerTable + threadIdx.x;
    double* acc = smem + kBoxMullerTable + size_t(3 * A.D + 2) * S::BS;
    auto run = [&](uint64_t g, auto sink) __attribute__((always_inline)) {
        process_group<S, Eval>(ev, A, g, sink, smem, top);
    };
    if constexpr (WHOLE)
        run_chunks<S::BS>(A.work, A.s + 1, A.hier, A.n_paths, A.partials, acc, run);
    else
        run_groups<S::BS>(A.work, A.s + 1, A.hier, A.n_paths, A.partials, acc, run);
}

// Whether an evaluator has the kernel for whole chunks alone: the quick ones, whose groups cost so little that
// the other form's additional state shows (1e8 paths, p = 1: N = 16, every level 5.38 ms in the other form, 5.16
// in this one; N = 2 0.97 and 0.91).
template <class Eval> constexpr bool kWholeKernel = true;

template <class S, class Eval>
inline hipError_t launch_one(const AmpArgs& A, const Eval& ev, int grid, LaunchOn st) {
    const size_t lds = amp_lds_bytes(A.D, A.s, S::BS);
    if constexpr (kWholeKernel<Eval>) {
        if (A.partials && A.work.n_coarse == A.work.n_chunks) {
            hipExtLaunchKernelGGL((k_amplitude<S, Eval, true>), dim3(grid), dim3(S::BS), lds, st.st, st.start, st.stop, 0, A, ev);
            return hipGetLastError();
        }
    }
    hipExtLaunchKernelGGL((k_amplitude<S, Eval, false>), dim3(grid), dim3(S::BS), lds, st.st, st.start, st.stop, 0, A, ev);
    return hipGetLastError();
}

// Reference actions of the straight line from A.a to A.b (pimc_chunks.hpp).
template <class Eval>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2))) k_line(AmpArgs A, Eval ev, double* parts) {
    line_part(parts, [&](int level, int k, int N) __attribute__((always_inline)) {
        const double qa[1] = {A.a + (A.b - A.a) * double(k) / double(N)};
        const double qb[1] = {A.a + (A.b - A.a) * double(k + 1) / double(N)};
        double S = 0.0;
        ev.template eval<1>(level, qa, qb, S);
        return S;
    });
}

template <class Eval>
inline hipError_t launch_line(const AmpArgs& A, const Eval& ev, double* parts, hipStream_t st) {
    if (A.s < 1) return hipSuccess;
    hipLaunchKernelGGL((k_line<Eval>), dim3(A.s, line_parts(A.s)), dim3(kBlock), 0, st, A, ev, parts);
    return hipGetLastError();
}

template <class S, class Eval>
inline int resident_one(size_t lds, int device) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_amplitude<S, Eval, false>, S::BS, lds) != hipSuccess)
        per_cu = 1;
    int ncu = 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) ncu = 256;
    return (per_cu < 1 ? 1 : per_cu) * ncu;
}

}  // namespace pimc
