// Rotation of spherical-harmonic coefficients, points and spin bases into the
// patch frame (Sec. II, step 1: coordinates in which the patch centre is the
// north pole).
//
// R = Rz(alpha) Ry(beta) Rz(gamma) (active rotation, z-y-z Euler angles) moves
// a point n to R n and a field f to f o R^-1.  The coefficients of the moved
// field are
//   a'_lm = exp(-i m alpha) sum_{m'=-l..l} d^l_{m m'}(beta) exp(-i m' gamma) a_lm'
// with a_{l,-m'} = (-1)^m' conj(a_lm') (the reality condition of Sec. I; g and
// c of a spin field each obey it) and d^l the Wigner small-d matrix of
// Appendix A.  The cost is O(lmax^3); the kernels below:
//
// k_rot_prep  tables over (l, k), k = |m'|: the recurrence factor G_l(k) below and
//             b_lk = exp(-i k gamma) a_lk scaled by it; the other sign of m' needs
//             no entry of its own, b_{l,-k} = (-1)^k conj(b_lk).  Zeroes the output.
// k_rot_main  one workgroup per (64 orders m, 16 values of k), lanes along m: each
//             wavefront runs the recurrence in l of d^l_{m,k} and d^l_{m,-k} for 4
//             values of k and adds d b in registers (no reduction over lanes; the
//             b are uniform, scalar loads).  The four wavefronts add up in LDS over
//             8 degrees, which then go to a'_lm with atomics.
//
// Normalised recurrence.  With d^l_{m m'} = h_l c_l(m) c_l(m') y_l and factors
// that obey c_{l+1} c_l A_{l+1} = 1 (A_l(x)^2 = l^2 - x^2, c_x(x) = 1) and
// h_{l+1} h_l = l + 1 (h_0 = 1), the three-term recurrence becomes
//   y_{l+1} = G_l(m) G_l(m') (cos beta - m m' / (l (l + 1))) y_l - y_{l-1},
//   G_l(x) = sqrt(2 l + 1) h_l c_l(x)^2,
// a few multiply-adds a step where the plain form takes six and a square root
// and a division per column.  G is rounded correctly (rot_factor.h), and m / (l (l +
// 1)) and G_l(m) G_l(m') once each before they are used: the recurrence is then at
// least as accurate as the plain form (largest error of d^l against 128 bits over
// 100 to 300 columns, plain / this, in 1e-15: beta 1.1, lmax 256 0.5 / 0.7, 1024
// 1.4 / 0.7, 4096 1.0 / 1.2; beta 0.1, lmax 1024 13 / 10, 4096 14 / 16; root mean
// square over the columns 3 to 25 % below).  With G from log2(n!) it was 5.6 at
// beta 1.1, lmax 4096.
//
// Bound by the vector instructions (13 FP64 ones per degree, order and pair of
// signs, as many again for broadcasts, sums and the flush: 62 % of the busy
// cycles) and by the atomics (without them 0.74 ms of the 1.6 ms that separate
// atomics for Re and Im took at lmax 1024; 128 consecutive bytes per order and
// flush: 0.97 ms).  us per call, before (8 orders x 128 columns per wavefront,
// summed over lanes at every degree) / now: lmax 64, two components 137 / 63;
// lmax 256, one component 355 / 136; lmax 1024, two components 2031 / 866; lmax
// 2048, two components 9218 / 5860.  Eight wavefronts per workgroup: 800 at lmax
// 1024, but 76, 172 and 6220 at the other sizes.
// k_rot_points, k_spin_phase  points and the spin basis angle.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>

#include "lane_ops.h"
#include "leg_common.h"
#include "psht_internal.h"
#include "rot_factor.h"

namespace psht {

constexpr int kRotPairs = 4;                  // values of k = |m'| per wavefront
constexpr int kRotWaves = 4;                  // wavefronts per workgroup
constexpr int kRotCols = kRotPairs * kRotWaves;  // values of k per workgroup
constexpr int kRotSteps = 8;                  // degrees between two flushes of the sums

__device__ inline int64_t rot_alm_index(int lmax, int l, int m) { return (int64_t)m * (2 * lmax + 1 - m) / 2 + l; }

// exp(-i k x) for an integer k: the product k x is split into hi + lo exactly
// (fma), so that its rounding does not enter the phase.
__device__ inline double2 phase_neg(int k, double x) {
    const double hi = (double)k * x;
    const double lo = fma((double)k, x, -hi);
    double s, c;
    sincos(hi, &s, &c);
    return make_double2(c - s * lo, -(s + c * lo));
}

// Double-double difference a - b (two-sum on the high parts).
__device__ inline double2 dd_sub(double2 a, double2 b) {
    const double s = a.x - b.x;
    const double bb = s - a.x;
    const double e = (a.x - (s - bb)) + (-b.x - bb);
    const double t = e + (a.y - b.y);
    const double hi = s + t;
    return make_double2(hi, t - (hi - s));
}

struct RotArgs {
    const double2 *alm;   // input [nc][nalm]
    double *B;            // [lmax + 1][lmax + 1][2 nc]: (l, k, Re and Im of each component)
    double *G;            // [lmax + 1][lmax + 1]: G_l(x), zero for x > l
    double *out;          // output [nc][nalm] complex, accumulated
    const double2 *lf;    // log2(n!) as double-double, n = 0..2 lmax
    const double2 *w;     // W(n) as double-double, n = 0..lmax (rot_factor.h)
    int lmax;
    int64_t nalm;
    double alpha, gamma, cb, hc, hs;  // cos beta, cos(beta/2), sin(beta/2)
};

template <int NC> __global__ __launch_bounds__(256) void k_rot_prep(RotArgs A) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    const int l = blockIdx.y;
    if (k > A.lmax) return;
    const int64_t row = (int64_t)l * (A.lmax + 1) + k;
    const double g = k <= l ? rot_g(A.w, l, k) : 0.0;
    const double2 e = phase_neg(k, A.gamma);
    const double sc = sqrt(g / (2.0 * l + 1.0));  // (d b) / (y b') = sqrt(G_l(m)) sc
    A.G[row] = g;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        double2 v = make_double2(0.0, 0.0);
        if (k <= l) {
            const int64_t i = (int64_t)c * A.nalm + rot_alm_index(A.lmax, l, k);
            double2 a = A.alm[i];
            if (k == 0) a.y = 0.0;
            v = make_double2((e.x * a.x - e.y * a.y) * sc, (e.x * a.y + e.y * a.x) * sc);
            A.out[2 * i] = A.out[2 * i + 1] = 0.0;
        }
        A.B[2 * (row * NC + c)] = v.x;
        A.B[2 * (row * NC + c) + 1] = v.y;
    }
}

// lmax = 0: the monopole does not turn
__global__ void k_rot_monopole(const double2 *in, double *out, int nc) {
    if ((int)threadIdx.x < nc) {
        out[2 * threadIdx.x] = in[threadIdx.x].x;
        out[2 * threadIdx.x + 1] = 0.0;
    }
}

// Seed d^{l0}_{m m'}(beta), l0 = max(m, |m'|), m >= 0, from the single
// surviving term of the explicit sum at the lowest degree:
//   m >= |m'|:  (-1)^(m-m') sqrt(C(2m, m+m'))  c^(m+m')  s^(m-m')
//   m' > m:                 sqrt(C(2m', m'+m)) c^(m'+m)  s^(m'-m)
//   -m' > m:    (-1)^(m+l0) sqrt(C(2l0, l0+m)) c^(l0-m)  s^(l0+m)
// (c = cos(beta/2), s = sin(beta/2)), returned as stored * 2^(512 k), k <= 0.
// The binomial comes from log2(n!) in double-double, the powers by binary
// powering with a separate exponent.
__device__ inline void rot_seed(const RotArgs &A, int m, int mp, double &stored, int &k) {
    const int am = mp < 0 ? -mp : mp;
    int j, x, pc, ps;
    bool neg;
    if (m >= am) {
        j = m;
        x = mp;
        pc = m + mp;
        ps = m - mp;
        neg = ((m - mp) & 1) != 0;
    } else if (mp > 0) {
        j = mp;
        x = m;
        pc = mp + m;
        ps = mp - m;
        neg = false;
    } else {
        j = am;
        x = m;
        pc = j - m;
        ps = j + m;
        neg = ((m + j) & 1) != 0;
    }
    if ((pc > 0 && A.hc == 0.0) || (ps > 0 && A.hs == 0.0)) {
        stored = 0.0;
        k = 0;
        return;
    }
    if (A.hs < 0.0 && (ps & 1)) neg = !neg;
    const double2 L = dd_sub(dd_sub(A.lf[2 * j], A.lf[j + x]), A.lf[j - x]);
    const double half_hi = 0.5 * L.x, half_lo = 0.5 * L.y;
    const double eb = floor(half_hi);
    const double mb = exp2((half_hi - eb) + half_lo);
    const XDbl pcx = xd_pow(fabs(A.hc), pc), psx = xd_pow(fabs(A.hs), ps);
    int e1;
    const double mant = frexp(mb * pcx.m * psx.m, &e1);
    xd_split(neg ? -mant : mant, (int)eb + pcx.e + psx.e + e1, stored, k);
}

// Renormalisation of a scaled pair (true value = stored * 2^(512 k), k <= 0):
// once the stored value passes 2^200 both values are scaled by 2^-512.
__device__ inline void rot_rescale(double &cur, double &prev, int &k) {
    const bool big = (k < 0) && (fabs(cur) > PSHT_RESCALE_HI);
    const double f = big ? PSHT_RESCALE_FACTOR : 1.0;
    cur *= f;
    prev *= f;
    k += big ? 1 : 0;
}

// f(std::integral_constant<int, 0>) ... f(std::integral_constant<int, N - 1>)
template <int N, typename Fn, int I = 0> __device__ inline void rot_unroll(const Fn &f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>());
        rot_unroll<N, Fn, I + 1>(f);
    }
}

// Uniform values of one degree and wavefront as they lie in LDS, whole rows of 16 doubles:
// b (2 nc per pair), G_l(k) per pair.  Each 16-lane row reads them
// one per lane and broadcasts.
template <int NC> struct RotRow {
    static constexpr int g = 2 * NC * kRotPairs, size = (g + kRotPairs + 15) / 16 * 16;
};

// Barrier for LDS only: the loads and the atomics in flight are not waited for.
__device__ inline void rot_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The states of one wavefront.
struct RotWave {
    // y of k and (-1)^k y of -k, with the previous ones
    double yp[kRotPairs], ypp[kRotPairs], ym[kRotPairs], ymp[kRotPairs];
    int kp[kRotPairs], km[kRotPairs];                                     // their scales
};

// Degrees lb .. lb + nsteps - 1.  MODE 2: every state has started and has scale 0.
// MODE 1: any.  MODE 3: all started, some scaled.  MODE 0: all started, none
// contributes (scaled, or zero): recurrence only.
// uni, gms, qms: this wavefront's uniform rows, G_l(m) and m / (l (l + 1)) of
// the chunk.
template <int NC, int MODE>
__device__ inline void rot_steps(RotWave &w, double *acc, int acc_stride, const double *uni, int uni_stride,
                                 const double *gms, const double *qms, int lb, int nsteps, int m, int kw, int lane,
                                 double cb) {
    typedef RotRow<NC> Row;
#pragma unroll 1
    for (int u = 0; u < nsteps; ++u) {
        const int l = lb + u;
        double x[Row::size / 16];
#pragma unroll
        for (int i = 0; i < Row::size / 16; ++i) x[i] = uni[u * uni_stride + 16 * i + (lane & 15)];
        const double gm = gms[u * 64 + lane], qm = qms[u * 64 + lane];
        double re[NC], im[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) re[c] = im[c] = 0.0;
        rot_unroll<kRotPairs>([&](auto P) {
            constexpr int p = decltype(P)::value;
            const int k = kw + p;
            const double g = row_bcast<(Row::g + p) % 16>(x[(Row::g + p) / 16]);
            const bool on = MODE != 1 || l >= max(m, k);
            if (MODE != 0) {
                double a = w.yp[p], b = w.ym[p];
                if (MODE == 1 || MODE == 3) {
                    a = on && w.kp[p] == 0 ? a : 0.0;
                    b = on && w.km[p] == 0 ? b : 0.0;
                }
                const double s = a + b, d = a - b;
                rot_unroll<NC>([&](auto Cc) {
                    constexpr int c = decltype(Cc)::value, i = 2 * NC * p + 2 * c;
                    re[c] = fma(s, row_bcast<i % 16>(x[i / 16]), re[c]);
                    im[c] = fma(d, row_bcast<(i + 1) % 16>(x[i / 16]), im[c]);
                });
            }
            const double gg = gm * g;
            const double tp = fma(-qm, (double)k, cb) * gg, tm = fma(qm, (double)k, cb) * gg;
            const double np = fma(tp, w.yp[p], -w.ypp[p]), nm = fma(tm, w.ym[p], -w.ymp[p]);
            // a state that has not started keeps its seed, with a previous value of zero
            w.ypp[p] = on ? w.yp[p] : 0.0;
            w.ymp[p] = on ? w.ym[p] : 0.0;
            w.yp[p] = on ? np : w.yp[p];
            w.ym[p] = on ? nm : w.ym[p];
        });
        if (MODE != 0) {
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                atomicAdd(acc + u * acc_stride + (2 * c) * 64 + lane, re[c]);
                atomicAdd(acc + u * acc_stride + (2 * c + 1) * 64 + lane, im[c]);
            }
        }
    }
}

template <int NC> __global__ __launch_bounds__(64 * kRotWaves) void k_rot_main(RotArgs A) {
    // 8 doubles between the rows of two degrees: the flush reads 8 of them side by side
    constexpr int kStride = 2 * NC * 64 + 8;
    typedef RotRow<NC> Row;
    constexpr int kUni = kRotWaves * Row::size, kThreads = 64 * kRotWaves;
    __shared__ double acc[kRotSteps * kStride];
    __shared__ double uni[kRotSteps * kUni];
    // G_l(m); its root, read by the flush while the next is stored
    __shared__ double gms[kRotSteps * 64], sqg[2][kRotSteps * 64];
    __shared__ double qms[kRotSteps * 64];  // m / (l (l + 1))
    __shared__ double2 phase[64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lmax = A.lmax, n = lmax + 1;
    const int m0 = blockIdx.x * 64, m = m0 + lane;
    const int kw = blockIdx.y * kRotCols + wave * kRotPairs;
    const int first = max(m0, (int)blockIdx.y * kRotCols);  // a multiple of 8
    if (first > lmax) return;

    RotWave w;
#pragma unroll
    for (int p = 0; p < kRotPairs; ++p) {
        w.yp[p] = w.ypp[p] = w.ym[p] = w.ymp[p] = 0.0;
        w.kp[p] = w.km[p] = 0;
    }
#pragma unroll 1
    for (int i = 0; i < 2 * kRotPairs; ++i) {
        const int k = kw + (i >> 1);
        double v = 0.0;
        int s = 0;
        if (m <= lmax && k <= lmax && !(k == 0 && (i & 1))) {
            rot_seed(A, m, (i & 1) ? -k : k, v, s);
            const int l0 = max(m, k);
            v *= sqrt((2.0 * l0 + 1.0) / (A.G[(int64_t)l0 * n + m] * A.G[(int64_t)l0 * n + k]));
            if ((i & 1) && (k & 1)) v = -v;
        }
#pragma unroll
        for (int p = 0; p < kRotPairs; ++p) {
            if (i == 2 * p) w.yp[p] = v, w.kp[p] = s;
            if (i == 2 * p + 1) w.ym[p] = v, w.km[p] = s;
        }
    }
    // flush: value i = tid + h kThreads is part i mod 2 (Re, Im) of degree (i / 2) mod
    // 8 of order m0 + i / 16: each order's 8 degrees are 128 consecutive bytes
    constexpr int kFlush = 16 * 64 / kThreads;
    if (tid < 64) phase[tid] = phase_neg(m0 + tid, A.alpha);
    for (int i = tid; i < kRotSteps * kStride; i += kThreads) acc[i] = 0.0;

    // The uniform values and the G_l(m) of a chunk of degrees are read from memory
    // while the chunk before it is computed: one degree at a time, every step
    // waited for memory (1.8 us a step).
    constexpr int kNU = (kRotSteps * kUni + kThreads - 1) / kThreads, kNG = kRotSteps * 64 / kThreads;
    double un[kNU], gn[kNG];
    const int k0 = blockIdx.y * kRotCols;
    auto fetch = [&](int lb) {
#pragma unroll
        for (int q = 0; q < kNU; ++q) {
            const int i = tid + q * kThreads, j = i % Row::size, l = min(lb + i / kUni, lmax);
            const int kb = k0 + (i / Row::size) % kRotWaves * kRotPairs;
            const int p = j < Row::g ? j / (2 * NC) : j - Row::g;
            const int64_t row = (int64_t)l * n + min(kb + p, lmax);
            double v = 0.0;
            if (j < Row::g) v = A.B[row * (2 * NC) + j % (2 * NC)];
            else if (j < Row::size) v = A.G[row];
            un[q] = v;
        }
#pragma unroll
        for (int q = 0; q < kNG; ++q) {
            const int i = tid + q * kThreads;
            gn[q] = A.G[(int64_t)min(lb + i / 64, lmax) * n + min(m0 + i % 64, lmax)];
        }
    };
    auto store = [&](int buf, int lb) {
#pragma unroll
        for (int q = 0; q < kNU; ++q)
            if (tid + q * kThreads < kRotSteps * kUni) uni[tid + q * kThreads] = un[q];
#pragma unroll
        for (int q = 0; q < kNG; ++q) {
            const int i = tid + q * kThreads, l = lb + i / 64;
            gms[i] = gn[q];
            sqg[buf][i] = sqrt(gn[q]);
            qms[i] = l ? (double)(m0 + i % 64) / ((double)l * (double)(l + 1)) : 0.0;
        }
    };
    fetch(first);
    store((first / kRotSteps) & 1, first);
    __syncthreads();

    // the last first degree of the wavefront
    const int started = max(min(m0 + 63, lmax), min(kw + kRotPairs - 1, lmax));
#pragma unroll 1
    for (int lb = first; lb <= lmax; lb += kRotSteps) {
        const int nsteps = min(kRotSteps, lmax + 1 - lb);
        const int cur = (lb / kRotSteps) & 1;
        fetch(lb + kRotSteps);
        if (kw <= lmax && lb + nsteps > kw) {
            bool scaled = false, live = false;
#pragma unroll
            for (int p = 0; p < kRotPairs; ++p) {
                scaled |= w.kp[p] < 0 || w.km[p] < 0;
                live |= (w.kp[p] == 0 && w.yp[p] != 0.0) || (w.km[p] == 0 && w.ym[p] != 0.0);
                // an underflowed pair of zeros may still wait for its previous value
                live |= (w.kp[p] == 0 && w.ypp[p] != 0.0) || (w.km[p] == 0 && w.ymp[p] != 0.0);
            }
            const bool mixed = lb < started || __any(scaled);
            auto steps = [&](auto mode) {
                rot_steps<NC, decltype(mode)::value>(w, acc, kStride, uni + wave * Row::size, kUni, gms, qms, lb,
                                                     nsteps, m, kw, lane, A.cb);
            };
            // a value of b that is not finite reaches every order of its degree, also
            // those that nothing else contributes to
            auto bad_b = [&] {
                bool bad = false;
#pragma unroll
                for (int q = 0; q < kRotSteps * Row::size / 64; ++q) {
                    const int i = q * 64 + lane;
                    bad |= !isfinite(uni[i / Row::size * kUni + wave * Row::size + i % Row::size]);
                }
                return bad;
            };
            if (!mixed) steps(std::integral_constant<int, 2>());
            else if (lb < started) steps(std::integral_constant<int, 1>());
            else if (__any(live || bad_b())) steps(std::integral_constant<int, 3>());
            else steps(std::integral_constant<int, 0>());
            if (mixed) {
#pragma unroll
                for (int p = 0; p < kRotPairs; ++p) {
                    rot_rescale(w.yp[p], w.ypp[p], w.kp[p]);
                    rot_rescale(w.ym[p], w.ymp[p], w.km[p]);
                }
            }
        }
        rot_barrier();
        const int fu = (tid >> 1) & (kRotSteps - 1), l = lb + fu;
#pragma unroll
        for (int h = 0; h < kFlush; ++h) {
            const int j = (tid + h * kThreads) / 16;
            const bool in = l <= lmax && m0 + j <= l;
            const double sc = in ? sqg[cur][fu * 64 + j] : 0.0;
            const double2 ph = phase[j];
            const double pr = (tid & 1) ? ph.y : ph.x, pi = (tid & 1) ? ph.x : -ph.y;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                // both lanes of a value read before either clears
                double *src = acc + fu * kStride + 2 * c * 64 + j;
                const double re = src[0], im = src[64];
                src[64 * (tid & 1)] = 0.0;
                if (in && (re != 0.0 || im != 0.0))
                    atomicAdd(A.out + 2 * ((int64_t)c * A.nalm + rot_alm_index(lmax, l, m0 + j)) + (tid & 1),
                              (pr * re + pi * im) * sc);
            }
        }
        store(cur ^ 1, lb + kRotSteps);
        rot_barrier();
    }
}

// Points: n' = R n; psi from the rotated basis vector R e_theta(n) to
// e_theta(n'), towards e_phi(n').
__global__ __launch_bounds__(256) void k_rot_points(int64_t n, RotMatrix R, const double *theta, const double *phi,
                                                    double *theta_out, double *phi_out, double *psi_out) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    double st, ct, sp, cp;
    sincos(theta[i], &st, &ct);
    sincos(phi[i], &sp, &cp);
    const double v[3] = {st * cp, st * sp, ct};
    const double e[3] = {ct * cp, ct * sp, -st};
    double w[3], f[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        w[r] = R.r[r][0] * v[0] + R.r[r][1] * v[1] + R.r[r][2] * v[2];
        f[r] = R.r[r][0] * e[0] + R.r[r][1] * e[1] + R.r[r][2] * e[2];
    }
    const double rho = sqrt(w[0] * w[0] + w[1] * w[1]);
    const double t2 = atan2(rho, w[2]);
    double p2 = atan2(w[1], w[0]);
    if (p2 < 0.0) p2 += 2.0 * M_PI;
    if (p2 >= 2.0 * M_PI) p2 = 0.0;
    double st2, ct2, sp2, cp2;
    sincos(t2, &st2, &ct2);
    sincos(p2, &sp2, &cp2);
    const double along_t = f[0] * ct2 * cp2 + f[1] * ct2 * sp2 - f[2] * st2;
    const double along_p = -f[0] * sp2 + f[1] * cp2;
    theta_out[i] = t2;
    phi_out[i] = p2;
    psi_out[i] = atan2(along_p, along_t);
}

template <typename T>
__global__ __launch_bounds__(256) void k_spin_phase(int64_t n, double ks, const double *psi, T *map) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    double s, c;
    sincos(ks * psi[i], &s, &c);
    const double xr = map[2 * i], xi = map[2 * i + 1];
    map[2 * i] = (T)(c * xr - s * xi);
    map[2 * i + 1] = (T)(c * xi + s * xr);
}

hipError_t launch_rotate_alm(int lmax, int nc, double alpha, double beta, double gamma, const void *alm_in,
                             void *alm_out, void *ws, const double2 *lf, const double2 *w, hipStream_t st) {
    RotArgs A;
    A.alm = (const double2 *)alm_in;
    // B and G: (nc 16 + 8)(lmax + 1)^2 bytes, within the workspace's nc 16 (lmax + 1)(2 lmax + 1) from lmax = 1 on
    A.B = (double *)ws;
    A.G = A.B + 2 * (int64_t)nc * (lmax + 1) * (lmax + 1);
    A.out = (double *)alm_out;
    A.lf = lf;
    A.w = w;
    A.lmax = lmax;
    A.nalm = (int64_t)(lmax + 1) * (lmax + 2) / 2;
    A.alpha = alpha;
    A.gamma = gamma;
    A.cb = cos(beta);
    A.hc = cos(0.5 * beta);
    A.hs = sin(0.5 * beta);
    if (lmax == 0) {
        k_rot_monopole<<<1, 64, 0, st>>>(A.alm, A.out, nc);
        return hipGetLastError();
    }
    const dim3 prep((lmax + 256) / 256, lmax + 1), grid((lmax + 64) / 64, (lmax + kRotCols) / kRotCols);
    if (nc == 2) {
        k_rot_prep<2><<<prep, 256, 0, st>>>(A);
        k_rot_main<2><<<grid, 64 * kRotWaves, 0, st>>>(A);
    } else {
        k_rot_prep<1><<<prep, 256, 0, st>>>(A);
        k_rot_main<1><<<grid, 64 * kRotWaves, 0, st>>>(A);
    }
    return hipGetLastError();
}

hipError_t launch_rotate_points(int64_t n, const RotMatrix &R, const double *theta, const double *phi,
                                double *theta_out, double *phi_out, double *psi_out, hipStream_t st) {
    if (n == 0) return hipSuccess;
    k_rot_points<<<dim3((unsigned)((n + 255) / 256)), 256, 0, st>>>(n, R, theta, phi, theta_out, phi_out, psi_out);
    return hipGetLastError();
}

hipError_t launch_spin_phase(int64_t n, double ks, int fp32, const double *psi, void *map, hipStream_t st) {
    if (n == 0) return hipSuccess;
    const dim3 grid((unsigned)((n + 255) / 256));
    if (fp32) k_spin_phase<float><<<grid, 256, 0, st>>>(n, ks, psi, (float *)map);
    else k_spin_phase<double><<<grid, 256, 0, st>>>(n, ks, psi, (double *)map);
    return hipGetLastError();
}

}  // namespace psht
