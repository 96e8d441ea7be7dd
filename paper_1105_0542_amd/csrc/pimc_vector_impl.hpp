// Vector estimation kernels (several coordinates, Sec. 2.2 with the bisection estimator of Sec. 4),
// included once per dimension by pimc_vector_d{1,2,3,4}.hip and pimc_vector_poly.hip.
//
// The walk is the one of the one-dimensional kernels, with a point of DIM coordinates per node: one
// lane owns one path; the bottom U bisection levels of each subtree live in registers, the levels
// above keep one pending right endpoint per level in LDS; every level-n slice is evaluated as soon as
// both its endpoints exist. Coordinate c of heap node h takes the normal of generator call
// (h >> 1) + c * 2^20 (so coordinate 0 is the one-dimensional path). The normal of a pending right
// child is drawn again when the walk returns to it instead of being kept (one more generator call per
// coordinate for every 2^U leaves; it halves the LDS per lane).
//
// Per level, each path's weight enters as d = exp(-(S_n - S_ref,n)) - 1, summed per canonical chunk
// (kChunkPaths paths, the order of the one-dimensional kernels, pimc_internal.hpp), then over chunks
// by k_seg_reduce: the result does not depend on the grid.
#pragma once

#include "pimc_chunks.hpp"
#include "pimc_vector.hpp"

namespace pimc {
namespace vec {

template <int DIM>
struct VecSource {
    RngKey key;
    PathRng pr;
    const double* bm;                  // Box-Muller table (LDS)
    // Normals of heap nodes 2j and 2j+1 in every coordinate.
    __device__ __forceinline__ void pair(uint32_t j, double (&ze)[DIM], double (&zo)[DIM]) const {
#pragma unroll
        for (int c = 0; c < DIM; ++c) normal_pair(key, pr, j + uint32_t(c) * kCoordPairStride, bm, ze[c], zo[c]);
    }
    // Normal of heap node h in every coordinate.
    __device__ __forceinline__ void node(uint32_t h, double (&z)[DIM]) const {
#pragma unroll
        for (int c = 0; c < DIM; ++c) {
            double e, o;
            normal_pair(key, pr, (h >> 1) + uint32_t(c) * kCoordPairStride, bm, e, o);
            z[c] = (h & 1u) ? o : e;
        }
    }
};

// Invariants of B slices from their endpoints (x4: the tables are pre-scaled).
template <int DIM, int B>
__device__ __forceinline__ void invariants(const double (&qa)[B][DIM], const double (&qb)[B][DIM], double (&u)[B],
                                           double (&w2)[B], double (&z)[B]) {
#pragma unroll
    for (int i = 0; i < B; ++i) {
        double su = 0.0, sw = 0.0, sz = 0.0;
#pragma unroll
        for (int c = 0; c < DIM; ++c) {
            const double s = qa[i][c] + qb[i][c];
            const double d = qb[i][c] - qa[i][c];
            su = fma(s, s, su);
            sw = fma(s, d, sw);
            sz = fma(d, d, sz);
        }
        u[i] = su;
        w2[i] = sw * sw;
        z[i] = sz;
    }
}

// Level tables with the compile-time shape of level P. The group loops are template recursions so
// that every length and offset is a constant of the front end.
template <int P, int B, int J, int L>
__device__ __forceinline__ void radial_groups_l(const_ptr<double> t, const double (&u)[B], const double (&z)[B],
                                                double (&zs)[B]) {
    if constexpr (L >= 0) {
        constexpr int len = radial_len(P, J + L, J);
        constexpr int off = radial_off(P, J, L);
        constexpr bool top = (L == radial_nl(P, J) - 1);
        double v[B];
        if constexpr (len == 0) {
#pragma unroll
            for (int i = 0; i < B; ++i) v[i] = 0.0;
        } else {
            const double c0 = t[off];
#pragma unroll
            for (int i = 0; i < B; ++i) v[i] = c0;
#pragma unroll
            for (int e = 1; e < len; ++e) {
                const double c = t[off + e];
#pragma unroll
                for (int i = 0; i < B; ++i) v[i] = fma(v[i], u[i], c);
            }
        }
#pragma unroll
        for (int i = 0; i < B; ++i) zs[i] = top ? v[i] : fma(zs[i], z[i], v[i]);
        radial_groups_l<P, B, J, L - 1>(t, u, z, zs);
    }
}

template <int P, int B, int J>
__device__ __forceinline__ void radial_groups_j(const_ptr<double> t, const double (&u)[B], const double (&w2)[B],
                                                const double (&z)[B], double (&acc)[B]) {
    if constexpr (J >= 0) {
        asm volatile("" : "+s"(t));
        double zs[B];
        radial_groups_l<P, B, J, radial_nl(P, J) - 1>(t, u, z, zs);
        constexpr bool top = (J == radial_nj(P) - 1);
#pragma unroll
        for (int i = 0; i < B; ++i) acc[i] = top ? zs[i] : fma(acc[i], w2[i], zs[i]);
        radial_groups_j<P, B, J - 1>(t, u, w2, z, acc);
    }
}

template <int P, int DIM>
struct RadialEval {
    const double* __restrict__ tab;
    __device__ __forceinline__ void launder() { asm volatile("" : "+s"(tab)); }
    template <int B>
    __device__ __forceinline__ void eval(int level, const double (&qa)[B][DIM], const double (&qb)[B][DIM],
                                         double& S) const {
        constexpr int E = radial_size(P);
        constexpr int NJ = radial_nj(P);
        const const_ptr<double> t = as_const(tab) + level * E;
        double u[B], w2[B], z[B], acc[B];
        invariants<DIM, B>(qa, qb, u, w2, z);
        radial_groups_j<P, B, NJ - 1>(t, u, w2, z, acc);
        if constexpr (NJ > 0) {
#pragma unroll
            for (int i = 0; i < B; ++i) S += acc[i];
        }
    }
};

// The same layout with the shape read from the shape array (any p, any s).
template <int DIM>
struct RadialEvalRT {
    const double* __restrict__ tab;
    const int* __restrict__ shape;
    int stride;
    __device__ __forceinline__ void launder() { asm volatile("" : "+s"(tab)); }
    template <int B>
    __device__ __forceinline__ void eval(int level, const double (&qa)[B][DIM], const double (&qb)[B][DIM],
                                         double& S) const {
        const const_ptr<double> t = as_const(tab) + level * stride;
        const const_ptr<int> sh = as_const(shape);
        double u[B], w2[B], z[B], acc[B];
        invariants<DIM, B>(qa, qb, u, w2, z);
        const int nj = sh[0];
        int g = 1 + nj;                     // index of the next group length
        int off = 0;
        for (int j = nj - 1; j >= 0; --j) {
            const int nl = sh[1 + j];
            double zs[B];
            for (int l = nl - 1; l >= 0; --l) {
                const int len = sh[g++];
                double v[B];
#pragma unroll
                for (int i = 0; i < B; ++i) v[i] = 0.0;
                if (len > 0) {
                    const double c0 = t[off];
#pragma unroll
                    for (int i = 0; i < B; ++i) v[i] = c0;
                    for (int e = 1; e < len; ++e) {
                        const double c = t[off + e];
#pragma unroll
                        for (int i = 0; i < B; ++i) v[i] = fma(v[i], u[i], c);
                    }
                }
                off += len;
#pragma unroll
                for (int i = 0; i < B; ++i) zs[i] = (l == nl - 1) ? v[i] : fma(zs[i], z[i], v[i]);
            }
#pragma unroll
            for (int i = 0; i < B; ++i) acc[i] = (j == nj - 1) ? zs[i] : fma(acc[i], w2[i], zs[i]);
        }
        if (nj > 0) {
#pragma unroll
            for (int i = 0; i < B; ++i) S += acc[i];
        }
    }
};

// Any polynomial V (component route): eps W_p of a slice is a polynomial in the 2 DIM variables
// y_c = qb_c - qa_c (c < DIM) and y_{DIM+c} = qa_c + qb_c, evaluated by a multivariate Horner scheme
// over the prefix tree of its monomials (exponents of y_0, y_1, ... from high to low). The tree is a
// level-independent structure stream of ints (pre-order); only the coefficients depend on the level.
//   node at depth v < 2 DIM - 1:  [n >= 1 children] then per child [gap | tail << 8] and the child's
//       node; a_v = first child's value y_{v+1}^tail, then per child a_v = a_v y_v^gap + (child value)
//       y_{v+1}^tail;
//   node at depth 2 DIM - 1:      [L >= 1]: the dense Horner chain in y_{2 DIM - 1} over the next L
//       coefficients of the level's array (zeros fill the exponents that are absent);
//   stream head: [tail of the root]; the slice value is a_0 y_0^tail.
// Every count and exponent is wave-uniform (scalar loads through the constant address space), so the
// depth-nested loops are scalar branches around B-wide vector FMAs; a_v and the running pointers have
// one register home per depth (no interpreter dispatch, no copies between depths).
//
// What bounds it is the latency of those scalar loads, not the FMAs (a chain has a few coefficients and
// B = 8 slices). So the walk reads ahead: the next int of the stream is in a register when its node begins,
// and the first kPolyAhead coefficients of the next chain are loaded while a chain is computed, a longer
// chain's next group while its last one is. That reads up to kPolyAhead coefficients and one int past the
// end of the arrays, within the buffer that holds both (kPolyPadBytes).
// d = 2, p = 10, N = 256, 5e5 paths: 14.7 -> 13.6 ms (with two entries a word or indexes for pointers the
// additional scalar work cost more than it hid: 16.1 and 18.5). One coordinate has few nodes and long chains
// and reads as it goes (p = 9, N = 256: 566 us, 588 reading ahead).
constexpr int kPolyAhead = 4;                   // coefficients per scalar load group of a chain
static_assert(kPolyAhead * sizeof(double) <= kPolyPadBytes, "reads past the arrays stay in their buffer");

template <int DIM>
struct PolyEvalRT {
    static constexpr int NV = 2 * DIM;
    static constexpr bool kAhead = DIM > 1;
    const double* __restrict__ tab;      // coefficients, level-major, stride doubles per level
    const int* __restrict__ code;        // structure stream
    int stride;
    __device__ __forceinline__ void launder() { asm volatile("" : "+s"(tab), "+s"(code)); }

    // a = a * y + t in a's registers. Written as fma(), the compiler picks the two-operand form that
    // accumulates into t's registers and then copies the result back to a at every iteration of a
    // node's child loop (B 64-bit moves per child); the three-operand instruction with a tied to its
    // destination needs no copy. Same operation, same rounding.
    __device__ __forceinline__ static void fma_into(double& a, double y, double t) {
        asm("v_fma_f64 %0, %0, %1, %2" : "+v"(a) : "v"(y), "v"(t));
    }

    // x[i] *= y[i]^e for a wave-uniform e >= 0 (a scalar loop around B multiplies).
    template <int B>
    __device__ __forceinline__ static void times_pow(double (&x)[B], const double (&y)[B], int e) {
        for (int k = 0; k < e; ++k) {
#pragma unroll
            for (int i = 0; i < B; ++i) x[i] *= y[i];
        }
    }

    struct Walk {
        const_ptr<int> s;          // next int to load
        const_ptr<double> c;       // next chain's coefficients
        int nx;                    // the int before s
        double cq[kPolyAhead];     // the next chain's first coefficients
        __device__ __forceinline__ int take() {
            if constexpr (!kAhead) {
                s += 1;
                return s[-1];
            }
            const int v = nx;
            nx = s[0];
            s += 1;
            return v;
        }
        __device__ __forceinline__ void ahead() {
            if constexpr (kAhead) {
#pragma unroll
                for (int q = 0; q < kPolyAhead; ++q) cq[q] = c[q];
            }
        }
    };

    // out = out y + k[q], q = FIRST .. n - 1 (n <= kPolyAhead, wave-uniform).
    template <int FIRST, int B>
    __device__ __forceinline__ static void chain_group(const double (&k)[kPolyAhead], int n, const double (&y)[B],
                                                       double (&out)[B]) {
        if constexpr (FIRST < kPolyAhead) {
            if (n <= FIRST) return;
#pragma unroll
            for (int i = 0; i < B; ++i) out[i] = fma(out[i], y[i], k[FIRST]);
            chain_group<FIRST + 1, B>(k, n, y, out);
        }
    }

    // The node's value into out. A chain starts from its first coefficient and a node of the two
    // deepest internal levels from its first child's value (the same bits as starting from 0:
    // fma(0, y, t) = t); every node has at least one child and every chain at least one coefficient.
    template <int V, int B>
    __device__ __forceinline__ static void node(Walk& w, const double (&y)[NV][B], double (&out)[B]) {
        if constexpr (V == NV - 1) {
            const int L = w.take();
            if constexpr (!kAhead) {
                const const_ptr<double> c = w.c;
                w.c += L;
                const double c0 = c[0];
#pragma unroll
                for (int i = 0; i < B; ++i) out[i] = c0;
                int j = 1;
                for (; j + kPolyAhead <= L; j += kPolyAhead) {
                    double k[kPolyAhead];
#pragma unroll
                    for (int q = 0; q < kPolyAhead; ++q) k[q] = c[j + q];
#pragma unroll
                    for (int q = 0; q < kPolyAhead; ++q)
#pragma unroll
                        for (int i = 0; i < B; ++i) out[i] = fma(out[i], y[V][i], k[q]);
                }
                for (; j < L; ++j) {
                    const double c1 = c[j];
#pragma unroll
                    for (int i = 0; i < B; ++i) out[i] = fma(out[i], y[V][i], c1);
                }
                return;
            }
            double k[kPolyAhead];
#pragma unroll
            for (int q = 0; q < kPolyAhead; ++q) k[q] = w.cq[q];
            const const_ptr<double> c = w.c;
            w.c += L;
            w.ahead();
#pragma unroll
            for (int i = 0; i < B; ++i) out[i] = k[0];
            chain_group<1, B>(k, L, y[V], out);
            for (int j = kPolyAhead; j < L; j += kPolyAhead) {
#pragma unroll
                for (int q = 0; q < kPolyAhead; ++q) k[q] = c[j + q];
                chain_group<0, B>(k, L - j, y[V], out);
            }
        } else {
            const int n = w.take();
            int k = 0;
            if constexpr (V >= NV - 3) {
                // the two deepest internal levels (most of the nodes) let the first child write the
                // accumulator; above them it is zeroed, which keeps one copy of a child's code per
                // level instead of two (2^(2 DIM - 1) copies of the chain loop when peeled throughout)
                const int h0 = w.take();
                node<V + 1, B>(w, y, out);
                times_pow<B>(out, y[V + 1], h0 >> 8);
                k = 1;
            } else {
#pragma unroll
                for (int i = 0; i < B; ++i) out[i] = 0.0;
            }
            for (; k < n; ++k) {
                const int h = w.take();
                times_pow<B>(out, y[V], (h & 255) - 1);
                double t[B];
                node<V + 1, B>(w, y, t);
                times_pow<B>(t, y[V + 1], h >> 8);
#pragma unroll
                for (int i = 0; i < B; ++i) fma_into(out[i], y[V][i], t[i]);
            }
        }
    }

    template <int B>
    __device__ __forceinline__ void eval(int level, const double (&qa)[B][DIM], const double (&qb)[B][DIM],
                                         double& S) const {
        const int lv = __builtin_amdgcn_readfirstlane(level);
        Walk w;
        w.c = as_const(tab) + lv * stride;
        w.s = as_const(code) + (kAhead ? 1 : 0);
        w.nx = kAhead ? as_const(code)[0] : 0;
        w.ahead();
        double y[NV][B];
#pragma unroll
        for (int i = 0; i < B; ++i) {
#pragma unroll
            for (int k = 0; k < DIM; ++k) {
                y[k][i] = qb[i][k] - qa[i][k];
                y[DIM + k][i] = qa[i][k] + qb[i][k];
            }
        }
        const int tail = w.take();
        double v[B];
        node<0, B>(w, y, v);
        times_pow<B>(v, y[0], tail);
#pragma unroll
        for (int i = 0; i < B; ++i) S += v[i];
    }
};

// ---------------------------------------------------------------------------- subtree (registers)
template <int DIM, int U, int L>
__device__ __forceinline__ void gen_level(const VecArgs& A, const VecSource<DIM>& src, uint32_t root, int D,
                                          double (&q)[(1 << U) + 1][DIM]) {
    if constexpr (L <= U) {
        constexpr int step = 1 << (U - L);
        const double sg = as_const(A.sig)[D + L];
#pragma unroll
        for (int i2 = 0; i2 < (1 << (L - 2)); ++i2) {
            const uint32_t parent = (root << (L - 2)) + uint32_t(i2);   // node of sub-level L-1
            double ze[DIM], zo[DIM];
            src.pair(parent, ze, zo);                                    // children 2*parent, 2*parent+1
            const int jl = (4 * i2 + 1) * step;
            const int jr = (4 * i2 + 3) * step;
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                q[jl][c] = sg * ze[c] + 0.5 * (q[jl - step][c] + q[jl + step][c]);
                q[jr][c] = sg * zo[c] + 0.5 * (q[jr - step][c] + q[jr + step][c]);
            }
        }
        gen_level<DIM, U, L + 1>(A, src, root, D, q);
    }
}

// Add the 2^L slices of sub-level L (point stride 2^(U-L)) at tree level `level` to S, left to right.
template <int DIM, int U, int L, class Eval>
__device__ __forceinline__ void level_sum(const Eval& ev, int level, const double (&q)[(1 << U) + 1][DIM],
                                          double& S) {
    constexpr int W = 1 << L;
    constexpr int ST = 1 << (U - L);
    constexpr int B = W < kVecBatch ? W : kVecBatch;
#pragma unroll
    for (int b0 = 0; b0 < W; b0 += B) {
        double qa[B][DIM], qb[B][DIM];
#pragma unroll
        for (int i = 0; i < B; ++i)
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                qa[i][c] = q[(b0 + i) * ST][c];
                qb[i][c] = q[(b0 + i + 1) * ST][c];
            }
        ev.template eval<B>(level, qa, qb, S);
    }
}

template <int DIM, int U, int L, class Eval>
__device__ __forceinline__ void hier_levels(const Eval& ev, int D, const double (&q)[(1 << U) + 1][DIM],
                                            double (&Ssub)[U + 1]) {
    if constexpr (L < U) {
        level_sum<DIM, U, L, Eval>(ev, D + L, q, Ssub[L]);
        hier_levels<DIM, U, L + 1, Eval>(ev, D, q, Ssub);
    }
}

// The component evaluator is a long instruction sequence, and a copy of it (and of the normals) per batch of
// a subtree is far more than the instruction cache holds: its deep subtrees are loops over the levels, with one
// copy per batch width and the points in scratch memory. d = 2, p = 10, N = 256, 5e5 paths: 13.6 -> 12.1 ms (with
// subtrees of six levels; of five 13.7, and of five without the loops 13.6), p = 8 2.11 -> 1.83; d = 3, p = 5,
// N = 128, 5e4 paths 1.23 -> 1.12 ms. Subtrees of two to four levels, those of N = 4..16, fit the registers and
// are faster unrolled (2.1e6 paths, level s alone: d = 3, p = 2, N = 8 0.56 ms in loops, 0.26 unrolled; d = 2,
// p = 2, N = 16 0.40 and 0.31), of five not (d = 2, p = 2, N = 32 0.70 and 0.81), and of one the same code is in
// one place instead of three (d = 3, p = 5 0.33 and 0.42). One coordinate is faster unrolled (N = 128, p = 9,
// level s alone 362 us, 465 in loops), and four (N = 128, p = 4: 0.76 ms, 1.14).
template <class Eval, int U> constexpr bool kRolled = false;
template <int DIM, int U> constexpr bool kRolled<PolyEvalRT<DIM>, U> = (DIM == 2 || DIM == 3) && (U == 1 || U >= 5);

template <int DIM, int U, int B, class Eval>
__device__ __forceinline__ void rolled_batch(const Eval& ev, int level, int sh, int b0,
                                             const double (&q)[(1 << U) + 1][DIM], double& S) {
    double qa[B][DIM], qb[B][DIM];
#pragma unroll
    for (int i = 0; i < B; ++i)
#pragma unroll
        for (int c = 0; c < DIM; ++c) {
            qa[i][c] = i == 0 ? q[b0 << sh][c] : qb[i - 1][c];
            qb[i][c] = q[(b0 + i + 1) << sh][c];
        }
    ev.template eval<B>(level, qa, qb, S);
}

template <int DIM, int U, class Eval>
__device__ __forceinline__ void rolled_levels(const Eval& ev, const VecArgs& A, const VecSource<DIM>& src, uint32_t root,
                                              int D, double (&q)[(1 << U) + 1][DIM], double (&Ssub)[U + 1]) {
#pragma unroll 1
    for (int L = 2; L <= U; ++L) {
        const int step = 1 << (U - L);
        const double sg = as_const(A.sig)[D + L];
#pragma unroll 1
        for (int i2 = 0; i2 < (1 << (L - 2)); ++i2) {
            double ze[DIM], zo[DIM];
            src.pair((root << (L - 2)) + uint32_t(i2), ze, zo);
            const int jl = (4 * i2 + 1) * step;
            const int jr = (4 * i2 + 3) * step;
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                q[jl][c] = sg * ze[c] + 0.5 * (q[jl - step][c] + q[jl + step][c]);
                q[jr][c] = sg * zo[c] + 0.5 * (q[jr - step][c] + q[jr + step][c]);
            }
        }
    }
    static_assert(kVecBatch == 8, "widths below");
#pragma unroll 1
    for (int L = A.hier ? 0 : U; L <= U; ++L) {
        double S = Ssub[L];
        if (L == 0) {
            rolled_batch<DIM, U, 1>(ev, D, U, 0, q, S);
        } else if (L == 1) {
            rolled_batch<DIM, U, 2>(ev, D + 1, U - 1, 0, q, S);
        } else if (L == 2) {
            if constexpr (U >= 2) rolled_batch<DIM, U, 4>(ev, D + 2, U - 2, 0, q, S);
        } else {
            if constexpr (U >= 3) {
#pragma unroll 1
                for (int b0 = 0; b0 < (1 << L); b0 += kVecBatch)
                    rolled_batch<DIM, U, kVecBatch>(ev, D + L, U - L, b0, q, S);
            }
        }
        Ssub[L] = S;
    }
}

// Subtree rooted at heap node `root` (level D+1) over the level-D slice (qL, qR) with root normal z.
template <int DIM, int U, class Eval>
__device__ __forceinline__ void run_subtree(const Eval& ev_in, const VecArgs& A, const VecSource<DIM>& src,
                                            uint32_t root, int D, const double (&qL)[DIM], const double (&qR)[DIM],
                                            const double (&zroot)[DIM], double (&Ssub)[U + 1]) {
    Eval ev = ev_in;
    ev.launder();
    double q[(1 << U) + 1][DIM];
    const double sg = as_const(A.sig)[D + 1];
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
        q[0][c] = qL[c];
        q[1 << U][c] = qR[c];
        q[1 << (U - 1)][c] = sg * zroot[c] + 0.5 * (qL[c] + qR[c]);
    }
    if constexpr (kRolled<Eval, U>) {
        rolled_levels<DIM, U, Eval>(ev, A, src, root, D, q, Ssub);
        return;
    }
    gen_level<DIM, U, 2>(A, src, root, D, q);
    if (A.hier) hier_levels<DIM, U, 0, Eval>(ev, D, q, Ssub);
    level_sum<DIM, U, U, Eval>(ev, D + U, q, Ssub[U]);
}

// ---------------------------------------------------------------------------- one path
// top: this lane's LDS slots (stride kVecBlock): S_top[n] at slot n (n < D); the pending right
// endpoint of level L (L = 2..D), coordinate c, at slot D + (L-2)*DIM + c.
template <int DIM, int U, class Eval>
__device__ __forceinline__ void walk_path(const Eval& ev, const VecArgs& A, const VecSource<DIM>& src, double* top,
                                          double (&Ssub)[U + 1]) {
    const int D = A.D;
#pragma unroll
    for (int j = 0; j <= U; ++j) Ssub[j] = 0.0;
    double a[DIM], b[DIM], z1[DIM];
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
        a[c] = A.a[c];
        b[c] = A.b[c];
    }
    {
        double unused[DIM];
        src.pair(0u, unused, z1);                    // node 1 = sine output of call 0
    }
    if constexpr (!kRolled<Eval, U>) {
        if (D == 0) {
            run_subtree<DIM, U, Eval>(ev, A, src, 1u, 0, a, b, z1, Ssub);
            return;
        }
    }
    for (int n = 0; n < D; ++n) top[n * kVecBlock] = 0.0;
    double* R = top + D * kVecBlock;
    const uint32_t nTop = D > 0 ? 1u << (D - 1) : 1u;    // level-D nodes nTop .. 2 nTop - 1
    double qlast[DIM];
#pragma unroll
    for (int c = 0; c < DIM; ++c) qlast[c] = a[c];
    for (uint32_t J = 0; J < nTop; ++J) {
        int L;
        uint32_t node;
        double qL[DIM], qR[DIM], z[DIM];
#pragma unroll
        for (int c = 0; c < DIM; ++c) qL[c] = qlast[c];
        if (J == 0) {
            L = 1;
            node = 1u;
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                qR[c] = b[c];
                z[c] = z1[c];
            }
        } else {
            const int t = __builtin_ctz(J);
            L = D - t;
            node = (nTop + J) >> t;
#pragma unroll
            for (int c = 0; c < DIM; ++c) qR[c] = R[((L - 2) * DIM + c) * kVecBlock];
            src.node(node, z);
        }
        double qm[DIM], zl[DIM], zr[DIM];
        while (!kRolled<Eval, U> || D > 0) {
            if (A.hier) {
                double qa1[1][DIM], qb1[1][DIM];
#pragma unroll
                for (int c = 0; c < DIM; ++c) {
                    qa1[0][c] = qL[c];
                    qb1[0][c] = qR[c];
                }
                double St = top[(L - 1) * kVecBlock];
                ev.template eval<1>(L - 1, qa1, qb1, St);
                top[(L - 1) * kVecBlock] = St;
            }
            const double sg = as_const(A.sig)[L];
#pragma unroll
            for (int c = 0; c < DIM; ++c) qm[c] = sg * z[c] + 0.5 * (qL[c] + qR[c]);
            src.pair(node, zl, zr);
            if (L == D) break;
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                R[((L - 1) * DIM + c) * kVecBlock] = qR[c];   // right child of `node`: (qm, qR), level L+1
                qR[c] = qm[c];
                z[c] = zl[c];
            }
            node = 2u * node;
            ++L;
        }
        if constexpr (kRolled<Eval, U>) {               // one copy: both sides, or the whole tree (D = 0)
            const int sides = D > 0 ? 2 : 1;
#pragma unroll 1
            for (int side = 0; side < sides; ++side) {
                double l[DIM], r[DIM], zs[DIM];
#pragma unroll
                for (int c = 0; c < DIM; ++c) {
                    l[c] = side == 0 ? qL[c] : qm[c];
                    r[c] = side == 0 && D > 0 ? qm[c] : qR[c];
                    zs[c] = D == 0 ? z[c] : (side == 0 ? zl[c] : zr[c]);
                }
                run_subtree<DIM, U, Eval>(ev, A, src, D > 0 ? 2u * node + uint32_t(side) : 1u, D, l, r, zs, Ssub);
            }
        } else {
            run_subtree<DIM, U, Eval>(ev, A, src, 2u * node, D, qL, qm, zl, Ssub);
            run_subtree<DIM, U, Eval>(ev, A, src, 2u * node + 1u, D, qm, qR, zr, Ssub);
        }
#pragma unroll
        for (int c = 0; c < DIM; ++c) qlast[c] = qR[c];
    }
}

// ---------------------------------------------------------------------------- estimation kernel
// One group: paths 64 g + lane (the group of the one-dimensional kernels); level sums to sink(),
// per-path level actions to A.dump. bm: the Box-Muller table, top: this lane's stack (both LDS).
template <int DIM, int U, class Eval, class Sink>
__device__ __forceinline__ void process_group(const Eval& ev, const VecArgs& A, uint64_t g, Sink sink,
                                              const double* bm, double* top) {
    const int lane = threadIdx.x & 63;
    const int D = A.D;
    const uint64_t local = g * 64 + uint64_t(lane);
    const bool valid = local < A.n_paths;
    double Ssub[U + 1];
    const VecSource<DIM> src{A.key, path_rng(A.key, A.first_path + local), bm};
    walk_path<DIM, U, Eval>(ev, A, src, top, Ssub);
    if (A.dump && valid) {
        double* o = A.dump + local * uint64_t(A.s + 1);
        for (int n = 0; n < D; ++n) o[n] = A.hier ? top[n * kVecBlock] : 0.0;
#pragma unroll
        for (int j = 0; j <= U; ++j) o[D + j] = (A.hier || j == U) ? Ssub[j] : 0.0;
    }
    if (A.partials) {
        const GroupSink k = sink();
        const const_ptr<double> shift = as_const(A.shift);
        if (A.hier) {
            for (int n = 0; n < D; ++n) reduce_level(k, lane, n, top[n * kVecBlock], shift[n], valid);
#pragma unroll
            for (int j = 0; j < U; ++j) reduce_level(k, lane, D + j, Ssub[j], shift[D + j], valid);
        }
        reduce_level(k, lane, A.hier ? D + U : 0, Ssub[U], shift[D + U], valid);
    }
}

// LDS of a workgroup: the Box-Muller table, the per-lane stacks, the accumulator slots.
template <int DIM, int U, class Eval>
__global__ void __launch_bounds__(kVecBlock) __attribute__((amdgpu_waves_per_eu(2)))
k_amplitude_vec(VecArgs A, Eval ev) {
    extern __shared__ double smem[];
    load_bm_table(smem, kVecBlock);     // the loops below begin with a barrier
    double* top = smem + kBoxMullerTable + threadIdx.x;
    double* acc = smem + kBoxMullerTable + size_t(vec_top_slots(DIM, A.D)) * kVecBlock;
    run_groups<kVecBlock>(A.work, A.s + 1, A.hier, A.n_paths, A.partials, acc, [&](uint64_t g, auto sink) __attribute__((always_inline)) {
        process_group<DIM, U, Eval>(ev, A, g, sink, smem, top);
    });
}

// ---------------------------------------------------------------------------- dispatch
template <int DIM, int U, class Eval>
inline hipError_t launch_one(const VecArgs& A, const Eval& ev, int grid, LaunchOn st) {
    const size_t lds = vec_lds_bytes(DIM, A.D, A.s);
    hipExtLaunchKernelGGL((k_amplitude_vec<DIM, U, Eval>), dim3(grid), dim3(kVecBlock), lds, st.st, st.start, st.stop, 0, A, ev);
    return hipGetLastError();
}

// Reference actions of the straight line from A.a to A.b (pimc_chunks.hpp).
template <int DIM, class Eval>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2))) k_line_vec(VecArgs A, Eval ev, double* parts) {
    line_part(parts, [&](int level, int k, int N) __attribute__((always_inline)) {
        double qa[1][DIM], qb[1][DIM];
#pragma unroll
        for (int c = 0; c < DIM; ++c) {
            qa[0][c] = A.a[c] + (A.b[c] - A.a[c]) * double(k) / double(N);
            qb[0][c] = A.a[c] + (A.b[c] - A.a[c]) * double(k + 1) / double(N);
        }
        double S = 0.0;
        ev.template eval<1>(level, qa, qb, S);
        return S;
    });
}

template <int DIM, int U, class Eval>
inline int resident_one(size_t lds, int device) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_amplitude_vec<DIM, U, Eval>, kVecBlock, lds) != hipSuccess)
        per_cu = 1;
    int ncu = 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) ncu = 256;
    return (per_cu < 1 ? 1 : per_cu) * ncu;
}

template <int DIM>
inline hipError_t launch_rt(const VecArgs& A, int U, int grid, LaunchOn st) {
    const RadialEvalRT<DIM> ev{A.tab, A.shape, A.stride};
    switch (U) {
        case 1: return launch_one<DIM, 1>(A, ev, grid, st);
        case 2: return launch_one<DIM, 2>(A, ev, grid, st);
        case 3: return launch_one<DIM, 3>(A, ev, grid, st);
        case 4: return launch_one<DIM, 4>(A, ev, grid, st);
        default: return hipErrorInvalidValue;
    }
}

template <int DIM>
inline int resident_rt(int U, size_t lds, int device) {
    switch (U) {
        case 1: return resident_one<DIM, 1, RadialEvalRT<DIM>>(lds, device);
        case 2: return resident_one<DIM, 2, RadialEvalRT<DIM>>(lds, device);
        case 3: return resident_one<DIM, 3, RadialEvalRT<DIM>>(lds, device);
        default: return resident_one<DIM, 4, RadialEvalRT<DIM>>(lds, device);
    }
}

// UMAX: the deepest subtree instantiated by the caller's translation unit (the deepest of all may be
// compiled in a unit of its own).
template <int DIM, int UMAX = poly_subtree_levels(DIM)>
inline hipError_t launch_poly(const VecArgs& A, int U, int grid, LaunchOn st) {
    const PolyEvalRT<DIM> ev{A.tab, A.shape, A.stride};
    switch (U) {
        case 1: return launch_one<DIM, 1>(A, ev, grid, st);
        case 2: return launch_one<DIM, 2>(A, ev, grid, st);
        case 3: return launch_one<DIM, 3>(A, ev, grid, st);
        case 4: if constexpr (UMAX >= 4) return launch_one<DIM, 4>(A, ev, grid, st); break;
        case 5: if constexpr (UMAX >= 5) return launch_one<DIM, 5>(A, ev, grid, st); break;
        case 6: if constexpr (UMAX >= 6) return launch_one<DIM, 6>(A, ev, grid, st); break;
        case 7: if constexpr (UMAX >= 7) return launch_one<DIM, 7>(A, ev, grid, st); break;
        default: break;
    }
    return hipErrorInvalidValue;
}

template <int DIM, int UMAX = poly_subtree_levels(DIM)>
inline int resident_poly(int U, size_t lds, int device) {
    switch (U) {
        case 1: return resident_one<DIM, 1, PolyEvalRT<DIM>>(lds, device);
        case 2: return resident_one<DIM, 2, PolyEvalRT<DIM>>(lds, device);
        case 4: if constexpr (UMAX >= 4) return resident_one<DIM, 4, PolyEvalRT<DIM>>(lds, device); break;
        case 5: if constexpr (UMAX >= 5) return resident_one<DIM, 5, PolyEvalRT<DIM>>(lds, device); break;
        case 6: if constexpr (UMAX >= 6) return resident_one<DIM, 6, PolyEvalRT<DIM>>(lds, device); break;
        case 7: if constexpr (UMAX >= 7) return resident_one<DIM, 7, PolyEvalRT<DIM>>(lds, device); break;
        default: break;
    }
    return resident_one<DIM, 3, PolyEvalRT<DIM>>(lds, device);
}

template <int DIM, int P>
inline hipError_t launch_spec(const VecArgs& A, int p, int grid, LaunchOn st) {
    if constexpr (P <= kMaxP) {
        if (p != P) return launch_spec<DIM, P + 1>(A, p, grid, st);
        const RadialEval<P, DIM> ev{A.tab};
        return launch_one<DIM, kVecU>(A, ev, grid, st);
    } else {
        return hipErrorInvalidValue;
    }
}

template <int DIM, int P>
inline int resident_spec(int p, size_t lds, int device) {
    if constexpr (P <= kMaxP) {
        if (p != P) return resident_spec<DIM, P + 1>(p, lds, device);
        return resident_one<DIM, kVecU, RadialEval<P, DIM>>(lds, device);
    } else {
        return 256;
    }
}

}  // namespace vec
}  // namespace pimc
