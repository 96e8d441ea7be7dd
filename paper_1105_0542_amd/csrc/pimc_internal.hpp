// Internal interface between the host library (pimc_host.cpp) and the kernels (pimc_kernels.hip).
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pimc.h"
#include "pimc_device.hpp"
#include "pimc_split.hpp"

namespace pimc {

constexpr int kBlock = 256;            // threads per workgroup of the auxiliary kernels (4 waves)

// Launch shape of the estimation walker: U bisection levels of each subtree in registers
// (2^U + 1 points), BS threads per workgroup, occupancy target WPE waves per SIMD (register budget
// 512/WPE), slices evaluated together coefficient-major (BATCH). Every shape gives the same bits.
template <int U_, int BS_, int WPE_, int BATCH_>
struct Shape {
    static constexpr int U = U_;
    static constexpr int BS = BS_;
    static constexpr int WPE = WPE_;
    static constexpr int BATCH = BATCH_;
    static_assert(BS_ == 64 || BS_ == 128 || BS_ == 256, "workgroup of 1, 2 or 4 waves");
};
// The default shapes: 256 threads, 2 waves per SIMD, 16 slices at once, U-level subtrees (the
// quartic kernels use U = 4: measured fastest on MI355X at p = 8, 12 and 18 for N from 64 to 1024;
// U = 5 needs more registers than 2 waves per SIMD leave and spills to scratch).
template <int U>
using DefaultShape = Shape<U, 256, 2, 16>;

// Arguments of one estimation launch (passed by value in the kernel argument segment, so every
// field is wave-uniform and scalar-loaded).
struct AmpArgs {
    const double* tab64;               // device: level tables, level-major
    const float* tab32;                // device: FP32 copy (PIMC_FP32_POLY)
    const int* gdeg;                   // device: generic shape, degree of each P_k
    int gK;                            // generic shape: number of P_k
    int gstride;                       // generic shape: doubles per level table
    double a, b;                       // endpoints (after the mass rescaling)
    double alpha;                      // Poeschl-Teller: tanh argument scale (after the mass rescaling)
    GenTables gen;                     // general-potential mode: derivative tables (coefficients in tab64)
    const double* sig;                 // device: sigma_n = sqrt(T / 2^(n+1)), n = 0..s (0 unused)
    const double* shift;               // device: straight-line level action S_ref,n, n = 0..s
    RngKey key;
    uint64_t first_path;               // path index of local path 0
    uint64_t n_paths;                  // local paths 0..n_paths-1
    PathWork work;                     // how the paths are shared out (not used by the batched kernel)
    int s;                             // N = 2^s
    int D;                             // s - U: levels walked with the explicit stack
    int hier;                          // evaluate every level (else level s only)
    double* partials;                  // device [level][chunk][4] or null
    double* dump;                      // device [path][s+1] or null
};

// Tanh64P: the Poeschl-Teller tables with the compile-time shape of level p (K = p groups of degree
// p), U = 4.
enum class EvalKind { Quartic64, Quartic32, GenericEven64, GenericOdd64, Tanh64, Tanh64P, General64 };

// Dynamic LDS bytes of the estimation kernel: the Box-Muller table; per lane, 3D+2 slots of the
// explicit stack; per accumulator slot and level, three sums.
inline size_t amp_lds_bytes(int D, int s, int BS) {
    return (size_t(kBoxMullerTable) + size_t(3 * D + 2) * size_t(BS) + size_t(kChunkSlots * (s + 1) * 3)) *
           sizeof(double);
}

// Where an estimation kernel is launched, and the events (or null) that its own dispatch records: a
// recorded event of its own is another packet and a gap of some us before and after the kernel.
struct LaunchOn {
    hipStream_t st;
    hipEvent_t start, stop;
    LaunchOn(hipStream_t stream, hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr) : st(stream), start(e0), stop(e1) {}
};

// Launch the estimation kernel; p selects the quartic specialization, U = s - D the unrolled
// subtree depth. Returns hipErrorInvalidValue for an unsupported combination.
hipError_t launch_amplitude(const AmpArgs& A, EvalKind kind, int p, int U, int grid, LaunchOn st);

// The compile-time shapes of level p with U = 4 (pimc_kernels_q64.hip, pimc_kernels_q32.hip,
// pimc_kernels_tanh.hip): hipErrorInvalidValue / 256 for p outside 1..kMaxP.
hipError_t launch_quartic64(const AmpArgs& A, int p, int U, int grid, LaunchOn st);
hipError_t launch_quartic32(const AmpArgs& A, int p, int U, int grid, LaunchOn st);
hipError_t launch_tanh_fixed(const AmpArgs& A, int p, int grid, LaunchOn st);
int resident_quartic64(int p, int U, size_t lds_bytes, int device);
int resident_quartic32(int p, int U, size_t lds_bytes, int device);
int resident_tanh_fixed(int p, size_t lds_bytes, int device);

// General-potential mode (pimc_general_kernels.hip): the evaluators generated for level p; the
// number of monomials of the level-p table (-1 outside 1..kGenMaxP).
hipError_t launch_general_compiled(const AmpArgs& A, int p, int U, int grid, LaunchOn st);
int general_compiled_resident(int p, int U, size_t lds_bytes, int device);
int general_compiled_nrec(int p);
// The levels up to kGenInlineMaxP in two translation units (pimc_general_inline.hip), LO = 1 and 5 their
// first levels.
template <int LO>
hipError_t gen_inline_launch(const AmpArgs& A, int p, int U, int grid, LaunchOn st);
template <int LO>
int gen_inline_resident(int p, int U, size_t lds_bytes, int device);
template <int LO>
int gen_inline_nrec(int p);
template <int LO>
hipError_t gen_inline_line(const AmpArgs& A, int p, double* parts, hipStream_t st);
#define PIMC_GEN_INLINE_DECLARE(LO)                                                          \
    template <>                                                                               \
    hipError_t gen_inline_launch<LO>(const AmpArgs& A, int p, int U, int grid, LaunchOn st); \
    template <>                                                                               \
    int gen_inline_resident<LO>(int p, int U, size_t lds_bytes, int device);                 \
    template <>                                                                               \
    int gen_inline_nrec<LO>(int p);                                                          \
    template <>                                                                               \
    hipError_t gen_inline_line<LO>(const AmpArgs& A, int p, double* parts, hipStream_t st);
PIMC_GEN_INLINE_DECLARE(1)
PIMC_GEN_INLINE_DECLARE(5)
#undef PIMC_GEN_INLINE_DECLARE
// The levels above kGenInlineMaxP, one translation unit each (pimc_general_hi.hip built with
// PIMC_GEN_P = p): launch, resident workgroups per CU and monomial count of that level's evaluator.
template <int P>
hipError_t gen_hi_launch(const AmpArgs& A, int U, int grid, LaunchOn st);
template <int P>
int gen_hi_resident(int U, size_t lds_bytes, int device);
template <int P>
int gen_hi_nrec();
template <int P>
hipError_t gen_hi_line(const AmpArgs& A, double* parts, hipStream_t st);
#define PIMC_GEN_HI_DECLARE(P)                                                         \
    template <>                                                                         \
    hipError_t gen_hi_launch<P>(const AmpArgs& A, int U, int grid, LaunchOn st);    \
    template <>                                                                         \
    int gen_hi_resident<P>(int U, size_t lds_bytes, int device);                        \
    template <>                                                                         \
    int gen_hi_nrec<P>();                                                               \
    template <>                                                                         \
    hipError_t gen_hi_line<P>(const AmpArgs& A, double* parts, hipStream_t st);
PIMC_GEN_HI_DECLARE(11)
PIMC_GEN_HI_DECLARE(12)
PIMC_GEN_HI_DECLARE(13)
PIMC_GEN_HI_DECLARE(14)
PIMC_GEN_HI_DECLARE(15)
PIMC_GEN_HI_DECLARE(16)
PIMC_GEN_HI_DECLARE(17)
PIMC_GEN_HI_DECLARE(18)
#undef PIMC_GEN_HI_DECLARE

// Raw standard normals of heap nodes 1..n_nodes for k_paths paths: out[path][node-1] (device).
hipError_t launch_normals(const RngKey& key, uint64_t first_path, uint64_t k_paths, uint32_t n_nodes, double* out,
                          hipStream_t st);

// Straight-line reference actions formed on the device (pimc_chunks.hpp): at most kLineParts partial sums
// per level, `parts` [s+1][kLineParts]; then level n's action, n = 1..s, into shift[n] and shift_host[n].
constexpr int kLineParts = 64;
hipError_t launch_line_sum(const double* parts, int s, double* shift, double* shift_host, hipStream_t st);
hipError_t launch_line_general(const AmpArgs& A, int p, double* parts, hipStream_t st);

// Adds the group sums of a run's fine chunks into their chunk records, each chunk in the canonical
// order (group g to slot g mod kChunkSlots in increasing g, then the slots in order).
hipError_t launch_group_chunks(const PathWork& w, int slots, uint64_t n_paths, double* partials, hipStream_t st);

// Canonical reduction: segment i = len[i] chunk sums of 4 doubles at partials + base[i], added in a
// fixed order that depends only on len[i]; out[i][4] (all device).
hipError_t launch_seg_reduce(const double* partials, const uint64_t* base, const uint64_t* len, uint64_t n_seg,
                             double* out, hipStream_t st);

// A segment whose groups are all fine: its group sums, where its chunk records go, its paths.
struct GroupSegment {
    const double* gsum;                // [group][3]
    double* records;                   // [chunk][4]
    uint64_t n_paths;
};
// Chunk records and canonical reduction of such segments: out[i][4] (all device).
hipError_t launch_seg_groups(const GroupSegment* segs, uint64_t n_seg, double* out, hipStream_t st);
// The chunk records alone, of pieces of at most kPieceChunks chunks (a long segment is several).
constexpr uint64_t kPieceChunks = kBlock / 4;
hipError_t launch_group_records(const GroupSegment* pieces, uint64_t n_pieces, hipStream_t st);
// Above this many chunks a segment's records are formed by many workgroups instead of its own one.
constexpr uint64_t kShortSegment = 128;

// One task of a batch, as the persistent kernel reads it (device array, wave-uniform loads).
struct BatchTask {
    const double* tab;                 // level tables of the task's (system, T, p), quartic layout
    const double* sig;                 // sigma_n, n = 0..s
    const double* shift;               // S_ref,n, n = 0..s
    double* partials;                  // [slot][chunk][4]
    double a, b;                       // endpoints after the mass rescaling
    uint64_t n_paths;
    uint64_t n_chunks;
    uint64_t item0;                    // queue index of the task's first item
    double* gsum;                      // [slot][group][3], by group; null: by whole chunk
    uint32_t block;                    // groups per item (by group)
    uint32_t stream;
    int s;
};

// Arguments of a class's launch (by value, wave-uniform).
struct BatchArgs {
    const BatchTask* tasks;            // device
    uint64_t n_items;
    uint64_t n_static;                 // items dealt to the waves in turn (by group)
    unsigned long long* queue;         // device: the item counter, 0 at launch
    RngKey key;                        // stream: the task's
    uint32_t grab;                     // items per ticket
    int n_tasks;
    int by_group;
    int hier;
};

// A launch shape as the host sees it.
struct ShapeDesc {
    int U, BS, WPE, BATCH;
};

// Batched estimation (pimc_kernels_batch.hip). A class is the tasks of one level p with N = 16
// (n16: subtrees of at most 4 levels) or with N >= 32; shape selects one of its compiled launch
// shapes (0 = the default; levels 8, 12 and 18 have several for the autotuner, every other level
// only the default).
int batch_shape_count(int p, bool n16);
bool batch_shape(int p, bool n16, int idx, ShapeDesc& d);
hipError_t launch_batch(const BatchArgs& B, int p, bool n16, int shape, int grid, size_t lds, hipStream_t st);
int batch_resident_blocks(int p, bool n16, int shape, size_t lds_bytes, int device);
hipError_t launch_fill_u64(unsigned long long* p, int n, unsigned long long v, hipStream_t st);

// Occupancy-derived number of resident workgroups of the estimation kernel on this device.
int amplitude_resident_blocks(EvalKind kind, int p, int U, size_t lds_bytes, int device);

}  // namespace pimc
