// Estimation kernels of the bisection PIMC amplitude (Sec. 4 of Balaz et al.) for gfx950: the walker
// (pimc_walker.hpp) with the runtime-shaped evaluators (any polynomial, Poeschl-Teller), raw normals,
// the canonical chunk reduction and the launch dispatch. The compile-time table shapes are
// instantiated in pimc_kernels_q64.hip, pimc_kernels_q32.hip, pimc_kernels_tanh.hip and
// pimc_general_kernels.hip (one translation unit per evaluator family, built in parallel) and the
// batched kernel in pimc_kernels_batch.hip and pimc_batch_p*.hip.
#include <hip/hip_runtime.h>

#include "pimc_walker.hpp"

namespace pimc {

__global__ void k_fill_u64(unsigned long long* p, int n, unsigned long long v) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// ---------------------------------------------------------------------------- raw normals
// One thread per (path, node pair): nodes 2j and 2j+1 of path first_path + i, written where
// 1 <= node <= n_nodes.
__global__ void __launch_bounds__(kBlock) k_normals(RngKey key, uint64_t first_path, uint64_t k_paths,
                                                    uint32_t n_nodes, double* __restrict__ out) {
    __shared__ double bm[kBoxMullerTable];
    load_bm_table(bm, kBlock);
    __syncthreads();
    const uint32_t pairs = n_nodes / 2 + 1;
    const uint64_t gid = uint64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (gid >= k_paths * pairs) return;
    const uint64_t i = gid / pairs;
    const uint32_t j = uint32_t(gid % pairs);
    const PathRng pr = path_rng(key, first_path + i);
    double ze, zo;
    normal_pair(key, pr, j, bm, ze, zo);
    double* o = out + i * n_nodes;
    const uint32_t he = 2 * j, ho = 2 * j + 1;
    if (he >= 1 && he <= n_nodes) o[he - 1] = ze;
    if (ho <= n_nodes) o[ho - 1] = zo;
}

hipError_t launch_normals(const RngKey& key, uint64_t first_path, uint64_t k_paths, uint32_t n_nodes, double* out,
                          hipStream_t st) {
    const uint64_t work = k_paths * (uint64_t(n_nodes) / 2 + 1);
    const uint64_t blocks = (work + kBlock - 1) / kBlock;
    if (blocks == 0) return hipSuccess;
    if (blocks > 0x7fffffffull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_normals, dim3(uint32_t(blocks)), dim3(kBlock), 0, st, key, first_path, k_paths, n_nodes, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------- chunk reduction
// Group sums into chunk records (pimc_chunks.hpp): component q of the record of the chunk whose first
// group is g0 (of n_groups), by a quad of lanes: lane q adds groups q, q + 4, ... of the chunk -- an
// accumulator slot -- and then the four slots are added in order. Bound by latency: a chunk's 64 x 24
// bytes are read with the 16 groups' loads of a lane in flight.
__device__ __forceinline__ double chunk_component(const double* __restrict__ gsum, uint64_t g0, uint64_t n_groups,
                                                  double cnt, bool live) {
    const int q = int(threadIdx.x & 3u);
    double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < kChunkGroups / kChunkSlots; ++k) {
        const uint64_t g = g0 + uint64_t(k * kChunkSlots + q);
        if (live && g < n_groups) {
#pragma unroll
            for (int j = 0; j < 3; ++j) s[j] += gsum[g * 3 + j];
        }
    }
    double t[3];
    const int lane0 = int(threadIdx.x & 63u) & ~3;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        t[j] = 0.0;
#pragma unroll
        for (int k = 0; k < kChunkSlots; ++k) t[j] += __shfl(s[j], lane0 + k, 64);
    }
    return q == 0 ? cnt : (q == 1 ? t[0] : (q == 2 ? t[1] : t[2]));
}

__device__ __forceinline__ double chunk_count(uint64_t n_paths, uint64_t c) {
    const uint64_t rem = n_paths - c * kChunkPaths;
    return double(rem < kChunkPaths ? rem : kChunkPaths);
}

__global__ void __launch_bounds__(kBlock) k_group_chunks(const double* __restrict__ gsum, uint64_t first_chunk,
                                                         uint64_t n_fine, uint64_t n_chunks, uint64_t n_paths,
                                                         double* __restrict__ partials) {
    const uint64_t i = uint64_t(blockIdx.x) * kBlock + threadIdx.x;
    const uint64_t c = first_chunk + (i >> 2);
    const uint64_t slot = blockIdx.y;
    const bool live = c < n_chunks;
    const double v = chunk_component(gsum + slot * n_fine * 3, (i >> 2) * kChunkGroups, n_fine, chunk_count(n_paths, c), live);
    if (live) partials[(slot * n_chunks + c) * 4 + (i & 3u)] = v;
}

hipError_t launch_group_chunks(const PathWork& w, int slots, uint64_t n_paths, double* partials, hipStream_t st) {
    if (w.n_coarse >= w.n_chunks || slots < 1) return hipSuccess;
    const uint64_t blocks = ((w.n_chunks - w.n_coarse) * 4 + kBlock - 1) / kBlock;
    if (blocks > 0x7fffffffull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_group_chunks, dim3(uint32_t(blocks), uint32_t(slots)), dim3(kBlock), 0, st, w.gsum, w.n_coarse,
                       w.fine(), w.n_chunks, n_paths, partials);
    return hipGetLastError();
}

// Canonical reduction: segment i (one level of one run) is the sequence of chunk sums
// partials[base[i] + c*4 .. +3], c = 0..len[i]-1. One workgroup of kBlock threads per segment:
// thread t adds chunks t, t + kBlock, ... in order, then a fixed halving tree over the threads.
// The order depends only on the chunk count, so any run -- single or one task of a batch, any
// grid -- gives the same bits for the same chunks.
__device__ __forceinline__ void seg_reduce(const double* p, uint64_t n, double* __restrict__ out) {
    __shared__ double red[4][kBlock];
    const int tid = threadIdx.x;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (uint64_t c = tid; c < n; c += kBlock) {
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j] += p[c * 4 + j];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) red[j][tid] = s[j];
    __syncthreads();
    for (int w = kBlock / 2; w >= 1; w >>= 1) {
        if (tid < w) {
#pragma unroll
            for (int j = 0; j < 4; ++j) red[j][tid] += red[j][tid + w];
        }
        __syncthreads();
    }
    if (tid < 4) out[tid] = red[tid][0];
}

__global__ void __launch_bounds__(kBlock) k_seg_reduce(const double* __restrict__ partials,
                                                       const uint64_t* __restrict__ base,
                                                       const uint64_t* __restrict__ len,
                                                       double* __restrict__ out) {
    const uint64_t seg = blockIdx.x;
    seg_reduce(partials + base[seg], len[seg], out + seg * 4);
}

// The same from group sums: the workgroup first forms its segment's chunk records (64 quads), then
// reduces them. One launch instead of two, for segments of few chunks.
__device__ __forceinline__ uint64_t group_records(const GroupSegment* __restrict__ segs) {
    const const_ptr<GroupSegment> S = as_const(segs) + blockIdx.x;
    const double* gsum = S->gsum;
    double* rec = S->records;
    const uint64_t n_paths = S->n_paths;
    const uint64_t n_groups = (n_paths + 63) / 64;
    const uint64_t n_chunks = (n_paths + kChunkPaths - 1) / kChunkPaths;
    for (uint64_t c0 = 0; c0 < n_chunks; c0 += kPieceChunks) {
        const uint64_t c = c0 + (threadIdx.x >> 2);
        const bool live = c < n_chunks;
        const double v = chunk_component(gsum, c * kChunkGroups, n_groups, chunk_count(n_paths, c), live);
        if (live) rec[c * 4 + (threadIdx.x & 3u)] = v;
    }
    return n_chunks;
}

__global__ void __launch_bounds__(kBlock) k_seg_groups(const GroupSegment* __restrict__ segs, double* __restrict__ out) {
    const uint64_t n_chunks = group_records(segs);
    __syncthreads();
    seg_reduce((as_const(segs) + blockIdx.x)->records, n_chunks, out + uint64_t(blockIdx.x) * 4);
}

__global__ void __launch_bounds__(kBlock) k_group_records(const GroupSegment* __restrict__ pieces) { (void)group_records(pieces); }

hipError_t launch_group_records(const GroupSegment* pieces, uint64_t n_pieces, hipStream_t st) {
    if (n_pieces == 0) return hipSuccess;
    if (n_pieces > 0x7fffffffull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_group_records, dim3(uint32_t(n_pieces)), dim3(kBlock), 0, st, pieces);
    return hipGetLastError();
}

hipError_t launch_seg_groups(const GroupSegment* segs, uint64_t n_seg, double* out, hipStream_t st) {
    if (n_seg == 0) return hipSuccess;
    if (n_seg > 0x7fffffffull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_seg_groups, dim3(uint32_t(n_seg)), dim3(kBlock), 0, st, segs, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------- dispatch

template <bool EVEN>
static hipError_t launch_generic(const AmpArgs& A, int U, int grid, LaunchOn st) {
    GenericEval64<EVEN> ev{A.tab64, A.gdeg, A.gK, A.gstride};
    switch (U) {
        case 1: return launch_one<DefaultShape<1>>(A, ev, grid, st);
        case 2: return launch_one<DefaultShape<2>>(A, ev, grid, st);
        case 3: return launch_one<DefaultShape<3>>(A, ev, grid, st);
        case 4: return launch_one<DefaultShape<4>>(A, ev, grid, st);
        default: return hipErrorInvalidValue;
    }
}

static hipError_t launch_tanh(const AmpArgs& A, int U, int grid, LaunchOn st) {
    TanhEval64 ev{A.tab64, A.gdeg, A.gK, A.gstride, A.alpha};
    switch (U) {
        case 1: return launch_one<DefaultShape<1>>(A, ev, grid, st);
        case 2: return launch_one<DefaultShape<2>>(A, ev, grid, st);
        case 3: return launch_one<DefaultShape<3>>(A, ev, grid, st);
        case 4: return launch_one<DefaultShape<4>>(A, ev, grid, st);
        default: return hipErrorInvalidValue;
    }
}


hipError_t launch_amplitude(const AmpArgs& A, EvalKind kind, int p, int U, int grid, LaunchOn st) {
    switch (kind) {
        case EvalKind::Quartic64: return launch_quartic64(A, p, U, grid, st);
        case EvalKind::Quartic32: return launch_quartic32(A, p, U, grid, st);
        case EvalKind::GenericEven64: return launch_generic<true>(A, U, grid, st);
        case EvalKind::GenericOdd64: return launch_generic<false>(A, U, grid, st);
        case EvalKind::Tanh64: return launch_tanh(A, U, grid, st);
        case EvalKind::Tanh64P:
            if (U != 4) return hipErrorInvalidValue;
            return launch_tanh_fixed(A, p, grid, st);
        case EvalKind::General64: return launch_general_compiled(A, p, U, grid, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_seg_reduce(const double* partials, const uint64_t* base, const uint64_t* len, uint64_t n_seg,
                             double* out, hipStream_t st) {
    if (n_seg == 0) return hipSuccess;
    if (n_seg > 0x7fffffffull) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_seg_reduce, dim3(uint32_t(n_seg)), dim3(kBlock), 0, st, partials, base, len, out);
    return hipGetLastError();
}

// Level n = blockIdx.x + 1: its parts added by a wave butterfly.
__global__ void __launch_bounds__(64) k_line_sum(const double* __restrict__ parts, double* shift, double* shift_host) {
    const int n = int(blockIdx.x) + 1;
    const double S = wave_sum(int(threadIdx.x) < line_parts(n) ? parts[n * kLineParts + int(threadIdx.x)] : 0.0);
    if (threadIdx.x == 0) {
        shift[n] = S;
        shift_host[n] = S;
    }
}

hipError_t launch_line_sum(const double* parts, int s, double* shift, double* shift_host, hipStream_t st) {
    static_assert(kLineParts == 64, "one lane per part");
    if (s < 1) return hipSuccess;
    hipLaunchKernelGGL(k_line_sum, dim3(s), dim3(64), 0, st, parts, shift, shift_host);
    return hipGetLastError();
}

hipError_t launch_fill_u64(unsigned long long* p, int n, unsigned long long v, hipStream_t st) {
    hipLaunchKernelGGL(k_fill_u64, dim3((n + 63) / 64), dim3(64), 0, st, p, n, v);
    return hipGetLastError();
}



int amplitude_resident_blocks(EvalKind kind, int p, int U, size_t lds_bytes, int device) {
    switch (kind) {
        case EvalKind::Quartic64: return resident_quartic64(p, U, lds_bytes, device);
        case EvalKind::Quartic32: return resident_quartic32(p, U, lds_bytes, device);
        case EvalKind::GenericEven64:
        case EvalKind::GenericOdd64:
            switch (U) {
                case 1: return resident_one<DefaultShape<1>, GenericEval64<true>>(lds_bytes, device);
                case 2: return resident_one<DefaultShape<2>, GenericEval64<true>>(lds_bytes, device);
                case 3: return resident_one<DefaultShape<3>, GenericEval64<true>>(lds_bytes, device);
                default: return resident_one<DefaultShape<4>, GenericEval64<true>>(lds_bytes, device);
            }
        case EvalKind::Tanh64:
            switch (U) {
                case 1: return resident_one<DefaultShape<1>, TanhEval64>(lds_bytes, device);
                case 2: return resident_one<DefaultShape<2>, TanhEval64>(lds_bytes, device);
                case 3: return resident_one<DefaultShape<3>, TanhEval64>(lds_bytes, device);
                default: return resident_one<DefaultShape<4>, TanhEval64>(lds_bytes, device);
            }
        case EvalKind::Tanh64P:
            return resident_tanh_fixed(p, lds_bytes, device);
        case EvalKind::General64:
            return general_compiled_resident(p, U, lds_bytes, device);
    }
    return 256;
}

}  // namespace pimc
