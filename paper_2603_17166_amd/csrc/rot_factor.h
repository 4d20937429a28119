// Factors of the rotation's normalised recurrence (see k_rotate.hip):
//   G_l(x) = sqrt(2 l + 1) h_l c_l(x)^2,
// with c_l(x)^2 and h_l ratios of W(n) = (2n-1)!! / (2n)!!:
//   l - x = 2 n:      c_l(x)^2 = W(n) W(x + n) / W(x)
//   l - x = 2 n + 1:  the reciprocal of that (at l - 1), over l^2 - x^2
//   h_{2n} = 1 / W(n),  h_{2n+1} = (2 n + 1) W(n).
// W(n) ~ 1 / sqrt(pi n) lies in the double range at every n, so the ratios are
// taken directly, in double-double: G is the correctly rounded value but for
// about one in 2^40 (an error of 1e-16 in G shows in the rotated coefficients;
// formed from log2(n!) it was 2e-14 at lmax 4096).
#pragma once

#include <cmath>
#include <vector>

#include <hip/hip_runtime.h>

namespace psht {

// W(n) for n = 0..nmax as double-double.  W(n) = W(n - 1) - W(n - 1) / (2 n), the
// rounding of each difference kept in `low`.
inline void rot_w_table(int nmax, std::vector<double2> &w) {
    w.resize((size_t)nmax + 1);
    long double high = 1.0L, low = 0.0L;
    for (int n = 0; n <= nmax; ++n) {
        if (n > 0) {
            const long double d = (high + low) / (2 * (long double)n), t = high - d;
            low += (high - t) - d;
            high = t;
        }
        w[n].x = (double)(high + low);
        w[n].y = (double)((high - w[n].x) + low);
    }
}

// Double-double product and quotient.
__host__ __device__ inline double2 dd_mul(double2 a, double2 b) {
#pragma clang fp contract(off)
    const double p = a.x * b.x;
    const double e = fma(a.x, b.y, fma(a.y, b.x, fma(a.x, b.x, -p)));
    const double hi = p + e;
    return make_double2(hi, e - (hi - p));
}
__host__ __device__ inline double2 dd_div(double2 a, double2 b) {
#pragma clang fp contract(off)
    const double r = 1.0 / b.x, q = a.x * r;
    const double e = fma(-q, b.y, fma(-q, b.x, a.x) + a.y) * r;
    const double hi = q + e;
    return make_double2(hi, e - (hi - q));
}

// G_l(x), 0 <= x <= l, from the table of W(0) .. W(l) or more: one quotient of
// products (a chain of divisions took 2 us more at lmax 64).
__host__ __device__ inline double rot_g(const double2 *w, int l, int x) {
    const int n = (l - x) / 2;
    double2 p = dd_mul(w[n], w[x + n]), q = w[x];
    if ((l - x) & 1) {
        const double2 t = dd_mul(p, make_double2((double)(l - x) * (double)(l + x), 0.0));
        p = q;
        q = t;
    }
    if (l & 1) p = dd_mul(p, dd_mul(make_double2(l, 0.0), w[l / 2]));
    else q = dd_mul(q, w[l / 2]);
    const double a = 2.0 * l + 1.0, s = sqrt(a);
    return dd_mul(dd_div(p, q), make_double2(s, fma(-s, s, a) * (0.5 * s / a))).x;
}

}  // namespace psht
