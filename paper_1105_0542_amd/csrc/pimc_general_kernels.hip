// Estimation kernels of the general-potential mode: dispatch by level to the translation units of the
// inlined evaluators (pimc_general_inline.hip, p = 1..4 and 5..kGenInlineMaxP) and of the out-of-line
// ones (pimc_general_hi.hip, one per level).
#include <hip/hip_runtime.h>

#include "pimc_internal.hpp"

namespace pimc {

hipError_t launch_line_general(const AmpArgs& A, int p, double* parts, hipStream_t st) {
    switch (p) {
        case 11: return gen_hi_line<11>(A, parts, st);
        case 12: return gen_hi_line<12>(A, parts, st);
        case 13: return gen_hi_line<13>(A, parts, st);
        case 14: return gen_hi_line<14>(A, parts, st);
        case 15: return gen_hi_line<15>(A, parts, st);
        case 16: return gen_hi_line<16>(A, parts, st);
        case 17: return gen_hi_line<17>(A, parts, st);
        case 18: return gen_hi_line<18>(A, parts, st);
        default: return p <= 4 ? gen_inline_line<1>(A, p, parts, st) : gen_inline_line<5>(A, p, parts, st);
    }
}


static_assert(kGenInlineMaxP == 10 && kGenMaxP == 18, "the out-of-line levels 11..18 are declared in pimc_internal.hpp");

hipError_t launch_general_compiled(const AmpArgs& A, int p, int U, int grid, LaunchOn st) {
    switch (p) {
        case 11: return gen_hi_launch<11>(A, U, grid, st);
        case 12: return gen_hi_launch<12>(A, U, grid, st);
        case 13: return gen_hi_launch<13>(A, U, grid, st);
        case 14: return gen_hi_launch<14>(A, U, grid, st);
        case 15: return gen_hi_launch<15>(A, U, grid, st);
        case 16: return gen_hi_launch<16>(A, U, grid, st);
        case 17: return gen_hi_launch<17>(A, U, grid, st);
        case 18: return gen_hi_launch<18>(A, U, grid, st);
        default: return p <= 4 ? gen_inline_launch<1>(A, p, U, grid, st) : gen_inline_launch<5>(A, p, U, grid, st);
    }
}

int general_compiled_resident(int p, int U, size_t lds_bytes, int device) {
    switch (p) {
        case 11: return gen_hi_resident<11>(U, lds_bytes, device);
        case 12: return gen_hi_resident<12>(U, lds_bytes, device);
        case 13: return gen_hi_resident<13>(U, lds_bytes, device);
        case 14: return gen_hi_resident<14>(U, lds_bytes, device);
        case 15: return gen_hi_resident<15>(U, lds_bytes, device);
        case 16: return gen_hi_resident<16>(U, lds_bytes, device);
        case 17: return gen_hi_resident<17>(U, lds_bytes, device);
        case 18: return gen_hi_resident<18>(U, lds_bytes, device);
        default: return p <= 4 ? gen_inline_resident<1>(p, U, lds_bytes, device) : gen_inline_resident<5>(p, U, lds_bytes, device);
    }
}

int general_compiled_nrec(int p) {
    switch (p) {
        case 11: return gen_hi_nrec<11>();
        case 12: return gen_hi_nrec<12>();
        case 13: return gen_hi_nrec<13>();
        case 14: return gen_hi_nrec<14>();
        case 15: return gen_hi_nrec<15>();
        case 16: return gen_hi_nrec<16>();
        case 17: return gen_hi_nrec<17>();
        case 18: return gen_hi_nrec<18>();
        default: return p <= 4 ? gen_inline_nrec<1>(p) : gen_inline_nrec<5>(p);
    }
}

}  // namespace pimc
