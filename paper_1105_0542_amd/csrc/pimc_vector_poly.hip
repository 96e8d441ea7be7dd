// Vector estimation kernels of the component evaluator (any polynomial V) for one dimension,
// chosen at build time by PIMC_POLY_DIM (this file is compiled once per dimension, in parallel:
// subtrees of up to kPolyU1 (kPolyU, kPolyU3) levels make these the largest kernels of the vector mode). With
// PIMC_POLY_DEEP it holds only the deepest subtree of that dimension, when that is kPolySplitU
// levels or more, so that the deepest and the shallower kernels compile in parallel.
// Built without loop-invariant code motion on machine code (as pimc_general_inline.hip), with and without it:
// 6e5 paths, N = 256, d = 1, p = 8 1.02 and 0.98 ms; 5e5 paths, N = 256, d = 2, p = 10 12.0 both; 5e4 paths, N = 128,
// d = 3, p = 5 1.13 and 1.03; 2.1e6 paths, N = 16, d = 4, p = 4, level s alone 1.88 and 1.31.
#include "pimc_vector_impl.hpp"

#ifndef PIMC_POLY_DIM
#error "PIMC_POLY_DIM (the number of coordinates of this translation unit) is not defined"
#endif
#ifndef PIMC_POLY_DEEP
#define PIMC_POLY_DEEP 0
#endif

namespace pimc {

constexpr int kUDeep = poly_subtree_levels(PIMC_POLY_DIM);
constexpr bool kSplit = kUDeep >= kPolySplitU;

#if PIMC_POLY_DEEP

template <>
hipError_t launch_vector_poly_deep<PIMC_POLY_DIM>(const VecArgs& A, int grid, LaunchOn st) {
    if constexpr (kSplit) {
        const vec::PolyEvalRT<PIMC_POLY_DIM> ev{A.tab, A.shape, A.stride};
        return vec::launch_one<PIMC_POLY_DIM, kUDeep>(A, ev, grid, st);
    } else {
        return hipErrorInvalidValue;
    }
}

template <>
int vector_poly_resident_deep<PIMC_POLY_DIM>(size_t lds, int device) {
    if constexpr (kSplit) return vec::resident_one<PIMC_POLY_DIM, kUDeep, vec::PolyEvalRT<PIMC_POLY_DIM>>(lds, device);
    else return 0;
}

#else

constexpr int kUShallow = kSplit ? kPolySplitU - 1 : kUDeep;

template <>
hipError_t launch_vector_poly_dim<PIMC_POLY_DIM>(const VecArgs& A, int U, int grid, LaunchOn st) {
    if constexpr (kSplit)
        if (U == kUDeep) return launch_vector_poly_deep<PIMC_POLY_DIM>(A, grid, st);
    return vec::launch_poly<PIMC_POLY_DIM, kUShallow>(A, U, grid, st);
}

template <>
hipError_t launch_line_poly_dim<PIMC_POLY_DIM>(const VecArgs& A, double* parts, hipStream_t st) {
    if (A.s < 1) return hipSuccess;
    const vec::PolyEvalRT<PIMC_POLY_DIM> ev{A.tab, A.shape, A.stride};
    hipLaunchKernelGGL((vec::k_line_vec<PIMC_POLY_DIM, vec::PolyEvalRT<PIMC_POLY_DIM>>), dim3(A.s, line_parts(A.s)),
                       dim3(kBlock), 0, st, A, ev, parts);
    return hipGetLastError();
}

template <>
int vector_poly_resident_dim<PIMC_POLY_DIM>(int U, size_t lds, int device) {
    if constexpr (kSplit)
        if (U == kUDeep) return vector_poly_resident_deep<PIMC_POLY_DIM>(lds, device);
    return vec::resident_poly<PIMC_POLY_DIM, kUShallow>(U, lds, device);
}

#endif

}  // namespace pimc
