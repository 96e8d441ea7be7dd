// Estimation kernels of the general-potential mode with inlined evaluators: the walker (pimc_walker.hpp)
// instantiated with the code generated for p = PIMC_GEN_LO..PIMC_GEN_HI (pimc_general_device.hpp),
// subtrees of U = 1..gen_subtree_levels(p) levels. Built twice: levels 5..kGenInlineMaxP without loop-
// invariant code motion on machine code, which hoisted the moves of the literal coefficients (p = 8: 193)
// out of the walker's loops into registers that then spilled; levels 1..4 fit and are 5 % faster with it.
// 1e6 paths, N = 256, every level, with and without: p = 4 3.49 and 3.68 ms, p = 6 10.25 and 8.76, p = 8
// 11.17 and 8.88, p = 10 39.7 and 21.3. (Out-of-line functions for four slices instead: 10.4, 10.3, 20.0 at
// p = 6, 8, 10: the calls' scratch traffic.)
#include <hip/hip_runtime.h>

#include "pimc_general_device.hpp"
#include "pimc_walker.hpp"

#if !defined(PIMC_GEN_LO) || !defined(PIMC_GEN_HI)
#error "PIMC_GEN_LO and PIMC_GEN_HI (the levels of this translation unit) are not defined"
#endif

namespace pimc {

template <int P> constexpr bool kWholeKernel<GenCompiledEval<P>> = false;

static_assert(PIMC_GEN_HI <= kGenInlineMaxP, "inlined levels");

namespace {

template <int P>
hipError_t launch_p(const AmpArgs& A, int p, int U, int grid, LaunchOn st) {
    if constexpr (P <= PIMC_GEN_HI) {
        if (p != P) return launch_p<P + 1>(A, p, U, grid, st);
        const GenCompiledEval<P> ev{A.tab64, A.gen};
        switch (U) {
            case 1: return launch_one<DefaultShape<1>>(A, ev, grid, st);
            case 2: if constexpr (gen_subtree_levels(P) >= 2) return launch_one<DefaultShape<2>>(A, ev, grid, st); else break;
            case 3: if constexpr (gen_subtree_levels(P) >= 3) return launch_one<DefaultShape<3>>(A, ev, grid, st); else break;
            case 4: if constexpr (gen_subtree_levels(P) >= 4) return launch_one<DefaultShape<4>>(A, ev, grid, st); else break;
            default: break;
        }
        return hipErrorInvalidValue;
    } else {
        return hipErrorInvalidValue;
    }
}

template <int P>
int resident_p(int p, int U, size_t lds, int device) {
    if constexpr (P <= PIMC_GEN_HI) {
        if (p != P) return resident_p<P + 1>(p, U, lds, device);
        switch (U) {
            case 2: if constexpr (gen_subtree_levels(P) >= 2) return resident_one<DefaultShape<2>, GenCompiledEval<P>>(lds, device); else break;
            case 3: if constexpr (gen_subtree_levels(P) >= 3) return resident_one<DefaultShape<3>, GenCompiledEval<P>>(lds, device); else break;
            case 4: if constexpr (gen_subtree_levels(P) >= 4) return resident_one<DefaultShape<4>, GenCompiledEval<P>>(lds, device); else break;
            default: break;
        }
        return resident_one<DefaultShape<1>, GenCompiledEval<P>>(lds, device);
    } else {
        return 256;
    }
}

template <int P>
int nrec_p(int p) {
    if constexpr (P <= PIMC_GEN_HI) {
        return p == P ? GenCompiled<P>::NREC : nrec_p<P + 1>(p);
    } else {
        return -1;
    }
}

template <int P>
hipError_t line_p(const AmpArgs& A, int p, double* parts, hipStream_t st) {
    if constexpr (P <= PIMC_GEN_HI) {
        if (p != P) return line_p<P + 1>(A, p, parts, st);
        return launch_line(A, GenCompiledEval<P>{A.tab64, A.gen}, parts, st);
    } else {
        return hipErrorInvalidValue;
    }
}

}  // namespace

template <>
hipError_t gen_inline_launch<PIMC_GEN_LO>(const AmpArgs& A, int p, int U, int grid, LaunchOn st) {
    return launch_p<PIMC_GEN_LO>(A, p, U, grid, st);
}

template <>
int gen_inline_resident<PIMC_GEN_LO>(int p, int U, size_t lds_bytes, int device) {
    return resident_p<PIMC_GEN_LO>(p, U, lds_bytes, device);
}

template <>
int gen_inline_nrec<PIMC_GEN_LO>(int p) {
    return nrec_p<PIMC_GEN_LO>(p);
}

template <>
hipError_t gen_inline_line<PIMC_GEN_LO>(const AmpArgs& A, int p, double* parts, hipStream_t st) {
    return line_p<PIMC_GEN_LO>(A, p, parts, st);
}

}  // namespace pimc
