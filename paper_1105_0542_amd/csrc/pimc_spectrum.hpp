// Spectrum from the space-discretized evolution operator: launchers shared by the kernels
// (pimc_spectrum.hip) and the host driver (pimc_spectrum_host.cpp).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pimc_device.hpp"

namespace pimc {

// The level-0 table of a problem with T = t (the short-time amplitude), device pointers.
struct SpecTable {
    const double* tab;      // folded P_k, highest power first, consecutive in k
    const int* deg;         // K degrees
    int K;
    int stride;             // doubles in the table
    int even;               // P_k in mid^2 (even potential) or mid
};

// M[i*ld + j] = pref * exp(-(y_j - y_i)^2/(2t) - t W_p) for the grid x_i = -L + (i + 1/2) D,
// y = sm x, i, j < n (device M, ld >= n).
hipError_t launch_evolution_matrix(const SpecTable& tb, double L, double D, double sm, double t, double pref,
                                   uint32_t n, double* M, uint64_t ld, hipStream_t st);
// Packed symmetric band: tiles (I, J), I <= J <= I + bw, of kTile x kTile doubles, row-major within a
// tile, tile t at M + t * kTile^2 with map[t] = I << 16 | J, in the order of I, then J (row I starts at
// tile first(I)); nb = ceil(n / kTile) row blocks, elements beyond n are zero. bw < nb leaves out tiles
// whose elements are all exactly zero (the cut of k_evolution_matrix); bw = nb - 1 is the upper triangle.
constexpr int kTile = 64;
struct TileBand {
    uint32_t nb, bw;
    __host__ __device__ uint64_t first(uint32_t I) const {
        const uint64_t e = I > nb - bw ? I - (nb - bw) : 0;        // row r has bw + 1 tiles, less from r = nb - bw on
        return uint64_t(I) * (bw + 1) - e * (e + 1) / 2;
    }
    uint64_t tiles() const { return first(nb); }
};
// The band that holds every element with |y_j - y_i| of step `dy` per index and exponent
// (y_j - y_i)^2 / (2t) within the cut, with a margin beyond the rounding of the kernel's test.
TileBand tile_band(uint32_t n, double dy, double t);
hipError_t launch_evolution_tiles(const SpecTable& tb, double L, double D, double sm, double t, double pref,
                                  uint32_t n, const uint32_t* map, uint32_t ntiles, double* M, hipStream_t st);
// Step j of the Lanczos iteration: w = (1 - Q Q^T) M q_j with q_j = column j of Q (leading dimension ldq),
// by classical Gram-Schmidt against columns 0..j, twice: in exact arithmetic the first pass removes
// alpha_j q_j + beta_{j-1} q_{j-1} (the three-term recurrence) and nothing else, so alpha[j] = <q_j, M q_j>
// is its coefficient of q_j; beta[j] = |w|, column j + 1 = w / beta[j]. The product goes by partial
// products per tile (prow, pcol: tiles * kTile doubles each) added per row block; every sum has a fixed
// order. w: n, h: j + 1, scratch: lanczos_scratch(nb) doubles.
size_t lanczos_scratch(uint32_t nb);
hipError_t launch_lanczos_step(const double* M, const uint32_t* map, const TileBand& band, uint32_t n, double* Q, uint64_t ldq,
                               uint32_t j, double* prow, double* pcol, double* w, double* h, double* scratch, double* alpha,
                               double* beta, hipStream_t st);
// y = M x (ld even; M and x 16-byte aligned).
hipError_t launch_gemv(const double* M, uint64_t ld, uint32_t n, const double* x, double* y, hipStream_t st);
// y = sum_c h[c] Q_c (subtract = 0) or y -= sum_c h[c] Q_c (subtract = 1).
hipError_t launch_combine_cols(const double* Q, uint64_t ldq, uint32_t n, uint32_t ncols, const double* h, double* y,
                               int subtract, hipStream_t st);
}  // namespace pimc
