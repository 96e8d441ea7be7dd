// Straight-line reference actions of pimc_tables.hpp over the whole range of FP64: one line per problem, the
// library's value and the sum of its slices by Horner, slice after slice.
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "pimc_tables.hpp"

using namespace pimc;

static double slices(const LevelTable& t, double a, double b, int n) {
    const int N = 1 << n;
    double S = 0.0;
    for (int k = 0; k < N; ++k) {
        const double qa = a + (b - a) * double(k) / double(N), qb = a + (b - a) * double(k + 1) / double(N);
        const double mid = 0.5 * (qa + qb), dl = qb - qa, z = dl * dl;
        const double u = t.even ? mid * mid : mid;
        double acc = 0.0;
        size_t end = t.coef.size();
        for (size_t j = t.deg.size(); j-- > 0;) {
            const size_t off = end - size_t(t.deg[j]) - 1;
            double v = t.coef[off];
            for (size_t e = off + 1; e < end; ++e) v = v * u + t.coef[e];
            acc = j + 1 == t.deg.size() ? v : acc * z + v;
            end = off;
        }
        S += acc;
    }
    return S;
}

int main() {
    std::mt19937_64 gen(5);
    std::uniform_real_distribution<double> U(0.0, 1.0);
    auto mag = [&](double lo, double hi) { return std::pow(10.0, lo + (hi - lo) * U(gen)); };
    for (int it = 0; it < 5000; ++it) {
        const bool odd = it % 5 == 0;
        const int p = 1 + it % (odd ? 8 : 18), n = it % 6;
        const double A = mag(-10, 20), g = mag(-10, 20), T = mag(-8, 12), R = mag(-5, 35);
        const double a = it % 7 == 0 ? 0.0 : R * (2.0 * U(gen) - 1.0);
        const double b = it % 3 == 0 ? -a : (it % 4 == 0 ? a : R * (2.0 * U(gen) - 1.0));
        const PolyD V{0.0, odd ? A : 0.0, A / 2.0, 0.0, g / 24.0};
        const Coefficients C = effective_coefficients(V, p);
        const LevelTable t = fold_level(C, !odd, std::ldexp(T, -n), table_xdegrees(C));
        std::printf("%.17g %.17g\n", straight_line_action(t, a, b, n), slices(t, a, b, n));
    }
    return 0;
}
