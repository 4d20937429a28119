// CPU build of the rotation's recurrence factors (paper_2603_17166_amd/csrc/rot_factor.h):
// the largest relative error of G_l(x), l <= lmax, against 128-bit arithmetic
// over every x of some degrees.  Prints "checked <n> error <e>".
#include <quadmath.h>

#include <cstdio>
#include <cstdlib>

#include "rot_factor.h"

int main(int argc, char **argv) {
    if (argc != 2) return 2;
    const int lmax = std::atoi(argv[1]);
    std::vector<double2> w;
    psht::rot_w_table(lmax, w);
    std::vector<__float128> q(lmax + 1, 1);
    for (int n = 1; n <= lmax; ++n) q[n] = q[n - 1] * (__float128)(2 * n - 1) / (__float128)(2 * n);
    long checked = 0;
    double worst = 0.0;
    for (int l = lmax; l >= 0; l -= (l > 64 ? lmax / 16 + 1 : 1))
        for (int x = 0; x <= l; ++x) {
            const int n = (l - x) / 2;
            __float128 c = q[n] * q[x + n] / q[x];
            if ((l - x) & 1) c = 1 / (c * (__float128)((long)(l - x) * (l + x)));
            c = (l & 1) ? c * l * q[l / 2] : c / q[l / 2];
            c *= sqrtq((__float128)(2 * l + 1));
            const double e = (double)fabsq(((__float128)psht::rot_g(w.data(), l, x) - c) / c);
            if (e > worst) worst = e;
            ++checked;
        }
    std::printf("checked %ld error %.3e\n", checked, worst);
    return 0;
}
