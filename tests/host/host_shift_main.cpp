// Newton polynomials moved to nearby centres (shift_centres): the moved one has
// the same values, the centres are the ones asked for, and centres that stay
// leave the coefficients as they were, bit for bit.  Built with
// AddressSanitizer and UndefinedBehaviorSanitizer by
// tests/test_host_shift_centres.py.
//
// Bound of the values, in units of 2^-53: coefficient a_t is rewritten once for
// every centre k <= t, each time a product, a sum and the correction's own
// rounding at most as large as the coefficients it is formed from, so the value
// at x is off by at most 4 (m + 2) sum_t |a_t| |pi_t(x)| (values in long double).
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <vector>

#include "ld_internal.h"

int main() {
    int failures = 0;
    for (int m : {1, 2, 3, 8, 40, 81, 150, 300}) {
        const std::vector<double> xi = ld::leja_table(m + 1);
        std::vector<double> d;
        int64_t terms = 0;
        if (ld::divided_differences(0.2, 30.0, m, LD_SVAL_CENTER, 0, d, &terms) != LD_OK) return 2;
        for (double eta : {0x1p-23, 0x1p-24, 0.0}) {
            std::vector<double> c(xi.begin(), xi.begin() + m), to = c, a = d;
            uint64_t s = 1;
            for (double& x : to) {   // within eta of their places, both ways
                s = ld::splitmix_mix(s + 1);
                x += eta * ((double)(s >> 11) * 0x1p-52 - 1.0);
            }
            ld::shift_centres(c, to, a);
            for (int i = 0; i < m; ++i) failures += c[i] != to[i];
            if (eta == 0.0)
                for (int i = 0; i <= m; ++i) failures += a[i] != d[i];
            double worst = 0.0;
            for (int q = 0; q <= 80; ++q) {
                const long double x = -2.0L + 0.05L * q;
                long double u = 0.0L, v = 0.0L, pu = 1.0L, pv = 1.0L, size = 0.0L;
                for (int i = 0; i <= m; ++i) {
                    u += d[i] * pu;
                    v += a[i] * pv;
                    size += std::fabs(a[i] * pv);
                    if (i < m) {
                        pu *= x - xi[i];
                        pv *= x - to[i];
                    }
                }
                const long double off = std::fabs(u - v) / (4.0L * (m + 2) * 0x1p-53L * size);
                if ((double)off > worst) worst = (double)off;
            }
            if (!(worst <= 1.0)) ++failures;
            std::printf("degree %d, eta %g: %.3f of the bound\n", m, eta, worst);
        }
    }
    if (failures) return 1;
    std::printf("centre shifts passed\n");
    return 0;
}
