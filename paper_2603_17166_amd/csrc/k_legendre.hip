// Ring Legendre (Wigner-d) step of the partial-sky transform on gfx950.
//
// Synthesis: for every order m and every ring j with m <= mmax_j,
//   F_j(+m) = -          sum_l (g_lm + i c_lm)             lambda+_lm(theta_j)
//   F_j(-m) = -(-1)^s    sum_l (conj g_lm + i conj c_lm)   lambda-_lm(theta_j)
// so that f(theta_j, phi) = sum_m F_j(m) e^{i m phi} is the map of eq. syn on
// the ring (reality condition a_{l,-m} = (-1)^m conj(a_lm), Sec. I).  This is
// the step whose cost dominates the method (Sec. II.A); only rings inside the
// apodized cap are evaluated and orders well above lmax sin(theta_j) are
// dropped (polar optimization).
//
// Adjoint: the exact transpose,
//   A_lm = sum_j lambda+_lm(theta_j) F'_j(m),  B_lm = sum_j lambda-_lm(theta_j) conj F'_j(-m),
//   g~_lm = -(A + (-1)^s B)/2,  c~_lm = (i/2)(A - (-1)^s B)   (Sec. I, adjoint).
//
// Work decomposition.  The active rings of an order m come in bands of 64
// consecutive rings, one ring per lane.  Below the turning point l sin(theta) ~ m
// the lambda of a ring fall off faster than exponentially towards l = m, so a
// band starts at the first degree (on a grid of 32) at which any of its rings
// reaches 2^-64 (kLegStartExp): the terms left out lie below the rounding of the
// sums.  The recurrence of each band starts from a state stored at plan time
// (mu_l, mu_{l-1}; in the double range, see k_leg_states), so the kernels carry
// no exponents.  A wave holds several bands (registers) and takes them in one
// after the other as l passes their starts.  At lmax 4096 (35 degree cap) the
// bands start at 0.73 of the (ring, m, l) triples of l >= m, at lmax 2048 0.78.
// Two things need more than that:
//  - at spins in the hundreds the weaker sign of a ring can lie below the double
//    range where its band starts and matter later: the synthesis of such plans
//    takes every band's next stored state in as l passes it (synth_run);
//  - values that are not finite are looked for among the terms left out, from the
//    degree on at which a ring of the order reaches 2^-312, and put into the
//    results: coefficients by the synthesis, ring values by the adjoint.
//
// The per-(l, m) recurrence coefficients and coefficient combinations are
// wave-uniform: they are staged through LDS one chunk of 32 degrees ahead.
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "lane_ops.h"
#include "leg_common.h"
#include "psht_internal.h"

namespace psht {

struct LegArgs {
    const LegBand *bands;  // sorted by start degree within each order
    const double2 *st_p, *st_m;  // stored states {mu_l, mu_{l-1}} of the + and - functions
    int seg;               // degrees between stored states
    const double4 *coef;  // {-A, A + B, A - B, P} per (l, m)
    const double *kmant;
    const int32_t *kexp;
    const double *ring_y, *ring_ch, *ring_sh;
    int nring, lmax, spin, mmax;
    int64_t nalm;
    const char *alm_in;  // synthesis input of map 0: g_lm then c_lm, complex [nalm] each
    char *alm_out;       // adjoint output of map 0, complex [2][nalm]
    char *F;             // complex [2 mmax + 1][nring] of map 0: synthesis output / adjoint input
    int64_t alm_stride, F_stride;  // bytes between the coefficients / the F (workspaces) of consecutive maps
    int nmaps;
    double mscale;     // extra factor on the inputs (synthesis) or outputs (adjoint) of order m >= 1
};

// The coefficient stream of one order m ({-A, A+B, A-B, P} and, for the
// synthesis, the combinations Q) is staged in chunks of kStage degrees: by the
// synthesis through LDS, every lane loading 32-byte entries of the next chunk
// (coalesced) while the current chunk is computed from wave-uniform (broadcast)
// LDS reads.
constexpr int kStage = 32;

// The synthesis multiplies lambda+ by P (g + i c) and lambda- by P (conj g +
// i conj c) (Sec. I, with lambda_l = P_l mu_l): the four real combinations
// P {g_r - c_i, g_i + c_r, g_r + c_i, c_r - g_i} of order m at degree l
// (coefficient index k), with the imaginary parts of the m = 0 coefficients
// dropped and the inputs of order m >= 1 scaled by mscale.
__device__ inline double4 synth_combo(const double2 *g, const double2 *c, double P, int64_t k, int m,
                                      double mscale) {
    double2 a = g[k], b = c[k];
    if (m == 0) {
        a.y = 0.0;
        b.y = 0.0;
    } else {
        P *= mscale;
    }
    return make_double4((a.x - b.y) * P, (a.y + b.x) * P, (a.x + b.y) * P, (b.x - a.y) * P);
}

// Staged chunk of the synthesis: the recurrence table and the coefficient
// combinations of NM maps (one spare entry: the loop reads one step ahead).
template <int NM> struct SynthChunk {
    double4 T[kStage + 1], Q[NM][kStage + 1];
};

// Recurrence values of up to RMAX bands (one ring per lane and band).
template <int RMAX> struct BandState {
    double y[RMAX], up[RMAX], upp[RMAX], um[RMAX], ump[RMAX];
};

// Ring of this lane in a band; -1: none.
__device__ inline int band_ring(const LegBand &b, int lane) { return (b.mask >> lane) & 1 ? b.jb + lane : -1; }

// Degree at which a band enters an item that starts at la, and its state there:
// its own start, or the state stored for the segment start la above it.
__device__ inline int band_enter(const LegBand &b, int la) { return b.bs > la ? b.bs : la; }
__device__ inline int64_t band_state(const LegBand &b, int la, int l0, int seg, int lane) {
    const int k = b.bs >= la ? 0 : (la - l0) / seg - (b.bs - l0) / seg;
    return ((int64_t)b.blk + k) * 64 + lane;
}

// Loads a band's state into slot r (zero until then).  The slots are filled one
// chunk before the band enters, so that the loads are in flight meanwhile.
template <int RMAX, bool SPIN>
__device__ inline void band_load(const LegArgs &a, int r, int j, int64_t q, BandState<RMAX> &S) {
    if (j >= 0) {
        const double2 v = a.st_p[q];
        S.y[r] = a.ring_y[j];
        S.up[r] = v.x;
        S.upp[r] = v.y;
        if (SPIN) {
            const double2 w = a.st_m[q];
            S.um[r] = w.x;
            S.ump[r] = w.y;
        }
    }
}

// The first R bands and NM maps over n steps (a multiple of 4) of a staged
// chunk: accumulate lambda_l into the ring sums, then advance the recurrence.
// The coefficients of step t + 1 are read while step t computes; within a step
// the independent work comes first (step coefficients (A +/- B) - A y of every
// ring, accumulations), the dependent updates last.  Entries past the item's
// last degree are zero: their steps add nothing.
template <int R, int RMAX, int NM, bool SPIN>
__device__ inline void synth_chunk(BandState<RMAX> &S, double4 (*f)[RMAX], const SynthChunk<NM> &b, int n) {
    double4 q[NM];
#pragma unroll
    for (int k = 0; k < NM; ++k) q[k] = b.Q[k][0];
    double3 tc = make_double3(b.T[0].x, b.T[0].y, b.T[0].z);
#pragma unroll 1
    for (int t4 = 0; t4 < n; t4 += 4)
#pragma unroll
    for (int t = t4; t < t4 + 4; ++t) {
        double4 qn[NM];
#pragma unroll
        for (int k = 0; k < NM; ++k) qn[k] = b.Q[k][t + 1];
        const double3 tn = make_double3(b.T[t + 1].x, b.T[t + 1].y, b.T[t + 1].z);
        __builtin_amdgcn_sched_barrier(0);
        double cpl[R], cmi[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            cpl[r] = fma(tc.x, S.y[r], tc.y);
            if (SPIN) cmi[r] = fma(tc.x, S.y[r], tc.z);
        }
#pragma unroll
        for (int k = 0; k < NM; ++k)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const double vm = SPIN ? S.um[r] : S.up[r];
                f[k][r].x = fma(q[k].x, S.up[r], f[k][r].x);
                f[k][r].y = fma(q[k].y, S.up[r], f[k][r].y);
                f[k][r].z = fma(q[k].z, vm, f[k][r].z);
                f[k][r].w = fma(q[k].w, vm, f[k][r].w);
            }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double np = fma(cpl[r], S.up[r], -S.upp[r]);
            S.upp[r] = S.up[r];
            S.up[r] = np;
            if (SPIN) {
                const double nm = fma(cmi[r], S.um[r], -S.ump[r]);
                S.ump[r] = S.um[r];
                S.um[r] = nm;
            }
        }
#pragma unroll
        for (int k = 0; k < NM; ++k) q[k] = qn[k];
        tc = tn;
    }
}

// Synthesis: one wave per item, the degrees [la, lb) of order m for up to RMAX
// bands.  Segment 0 of an order, and for each band the segment it starts in,
// writes F; later segments write the partial copy of F of their segment
// (k part_stride bytes after F), which k_synth_parts_sum then adds into F.
// RMAX = 4 reads each staged coefficient once for four bands: 18 cycles of the
// CU's LDS pipe per step (four 16-byte broadcasts at 4.4 cycles) against 32 FMAs
// (39 cycles over the four SIMDs); with two bands the two are level and neither
// overlaps fully.
struct SynthArgs {
    LegArgs a;
    const SynthItem *items;
    int nitems;
    int64_t part_stride;  // bytes from F to the copy of segment 1, and on to the next ones
};

// What a wave of the synthesis works on.
template <int NM> struct SynthWave {
    const LegArgs &a;
    const LegBand *bands;  // of the item
    const double4 *T4;
    SynthChunk<NM> *buf;   // two chunks
    int64_t base;
    int m, l0, la, lb, nb, lane, map0;
};

// Loads one chunk's entries from degree c (zero from the item's end on): lanes
// 0..31 and 32..63 take an entry array each per round, the table first (round
// 0, lower half), then the maps' combinations.
template <int NM> struct SynthStage {
    static constexpr int N = (NM + 2) / 2;
    double4 v[N];
    __device__ inline void load(const SynthWave<NM> &w, int c) {
        const int l = c + (w.lane & 31), half = w.lane >> 5;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int k = 2 * i + half - 1;  // map; -1: the table
            v[i] = make_double4(0.0, 0.0, 0.0, 0.0);
            if (l < w.lb && k < NM && w.map0 + k < w.a.nmaps) {
                const double4 T = w.T4[l];
                if (k < 0) {
                    v[i] = T;
                } else {
                    const double2 *g = reinterpret_cast<const double2 *>(w.a.alm_in + (w.map0 + k) * w.a.alm_stride);
                    v[i] = synth_combo(g, g + w.a.nalm, T.w, w.base + l, w.m, w.a.mscale);
                }
            }
        }
    }
    __device__ inline void store(SynthChunk<NM> &b, int lane) const {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int k = 2 * i + (lane >> 5) - 1;
            if (k < 0) b.T[lane & 31] = v[i];
            else if (k < NM) b.Q[k][lane & 31] = v[i];
        }
    }
};

// The chunks from c while R bands have entered, then those with one more (one
// loop per R, so that the bands stay in their registers).  The next band is
// loaded during the last chunk before it enters.  RELOAD: the bands take in the
// state stored for each segment start they pass, since the one they entered with
// may have lost a value that matters from there on (k_leg_states).
template <int R, int RMAX, int NM, bool SPIN, bool RELOAD>
__device__ __forceinline__ void synth_run(const SynthWave<NM> &w, BandState<RMAX> &S, double4 (*f)[RMAX], int c,
                                          int slot) {
    const bool more = R < RMAX && R < w.nb;
    const int cend = more ? min(band_enter(w.bands[R], w.la), w.lb) : w.lb;
    auto load = [&] {
        const LegBand b = w.bands[R];
        band_load<RMAX, SPIN>(w.a, R, band_ring(b, w.lane), band_state(b, w.la, w.l0, w.a.seg, w.lane), S);
    };
    if constexpr (R < RMAX)
        if (more && c >= cend) load();  // enters with the one before
    if constexpr (R > 0) {
#pragma unroll 1
        for (; c < cend; c += kStage) {
            SynthStage<NM> next;
            const bool has_next = c + kStage < w.lb;
            if (has_next) next.load(w, c + kStage);
            if constexpr (R < RMAX)
                if (more && c + kStage >= cend) load();
            if constexpr (RELOAD)
                if (((c - w.l0) & (w.a.seg - 1)) == 0) {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const LegBand b = w.bands[r];
                        if (c > band_enter(b, w.la))
                            band_load<RMAX, SPIN>(w.a, r, band_ring(b, w.lane),
                                                  band_state(b, c, w.l0, w.a.seg, w.lane), S);
                    }
                }
            synth_chunk<R, RMAX, NM, SPIN>(S, f, w.buf[slot], min(kStage, (w.lb - c + 3) & ~3));
            if (has_next) next.store(w.buf[slot ^ 1], w.lane);
            __syncthreads();
            slot ^= 1;
        }
    }
    if constexpr (R < RMAX) {
        if (c < w.lb) synth_run<R + 1, RMAX, NM, SPIN, RELOAD>(w, S, f, c, slot);
    }
}

// Whether a coefficient combination of the degrees [from, to) is not finite, by
// map (bit k), in every lane: two rounds of loads in flight.
template <int NM> __device__ inline unsigned synth_non_finite(const SynthWave<NM> &w, int from, int to) {
    bool bad[NM] = {};
    for (int l0 = from; l0 < to; l0 += 128) {
        double4 q[2][NM];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int k = 0; k < NM; ++k) {
                const int l = min(l0 + 64 * i + w.lane, to - 1);
                const int map = min(w.map0 + k, w.a.nmaps - 1);
                const double2 *g = reinterpret_cast<const double2 *>(w.a.alm_in + map * w.a.alm_stride);
                q[i][k] = synth_combo(g, g + w.a.nalm, 1.0, w.base + l, w.m, 1.0);
            }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int k = 0; k < NM; ++k) {
                const double4 v = q[i][k];
                bad[k] |= !(isfinite(v.x) && isfinite(v.y) && isfinite(v.z) && isfinite(v.w));
            }
    }
    unsigned mask = 0;
#pragma unroll
    for (int k = 0; k < NM; ++k) mask |= __any(bad[k]) ? 1u << k : 0u;
    return mask;
}

// Maps NM blockIdx.y .. + NM - 1 share the recurrence.
template <int RMAX, int NM, bool SPIN, bool RELOAD = false>
__global__ __launch_bounds__(64) void k_leg_synth(SynthArgs A) {
    __shared__ SynthChunk<NM> buf[2];
    const LegArgs &a = A.a;
    if ((int)blockIdx.x >= A.nitems) return;
    const SynthItem it = A.items[blockIdx.x];
    if (it.nb <= 0) return;
    const int m = it.m, s = a.spin, lane = threadIdx.x;
    const LegBand *bands = a.bands + it.b0;
    const int64_t base = (int64_t)m * (2 * a.lmax + 1 - m) / 2;
    const SynthWave<NM> w{a, bands, a.coef + base, buf, base, m, m > s ? m : s, it.la, it.lb, it.nb, lane,
                          (int)blockIdx.y * NM};

    BandState<RMAX> S;
    double4 f[NM][RMAX];  // sums of the +m and -m coefficients {Re, Im, Re, Im}
#pragma unroll
    for (int r = 0; r < RMAX; ++r) {
        S.y[r] = S.up[r] = S.upp[r] = S.um[r] = S.ump[r] = 0.0;
#pragma unroll
        for (int k = 0; k < NM; ++k) f[k][r] = make_double4(0.0, 0.0, 0.0, 0.0);
    }
    const int c = band_enter(bands[0], it.la);
    unsigned poison = 0;
    {
        SynthStage<NM> first;
        first.load(w, c);
        // the terms that the order leaves out, in one of its items (a value that is
        // not finite in one ring spreads to the whole map)
        if (it.live < it.start) poison = synth_non_finite<NM>(w, it.live, it.start);
        first.store(buf[0], lane);
    }
    __syncthreads();
    synth_run<0, RMAX, NM, SPIN, RELOAD>(w, S, f, c, 0);

    const double sgn_neg = (s & 1) ? 1.0 : -1.0;  // -(-1)^s
    const int64_t op = (int64_t)(a.mmax + m) * a.nring, om = (int64_t)(a.mmax - m) * a.nring;
#pragma unroll
    for (int k = 0; k < NM; ++k) {
        if (w.map0 + k >= a.nmaps) break;
#pragma unroll
        for (int r = 0; r < RMAX; ++r) {
            if (r >= it.nb) break;
            const LegBand b = bands[r];
            const int j = band_ring(b, lane);
            const bool first = b.bs >= it.la;  // the band starts in this segment
            double2 *F = reinterpret_cast<double2 *>(a.F + (w.map0 + k) * a.F_stride +
                                                     (first ? 0 : (int64_t)it.part * A.part_stride));
            if (r == 0 && ((poison >> k) & 1)) f[k][r].x = f[k][r].y = f[k][r].z = f[k][r].w = NAN;
            if (j >= 0) {
                F[op + j] = make_double2(-f[k][r].x, -f[k][r].y);
                if (m != 0) F[om + j] = make_double2(sgn_neg * f[k][r].z, sgn_neg * f[k][r].w);
            }
        }
    }
}

// F(m)[j] += the partials of the segments after the one the ring's band starts
// in, for every written entry (|m| <= ring_mmax[j] and order |m| has degrees);
// order |m| has ceil((lmax + 1 - max(|m|, s)) / S) segments.  One thread per
// entry of F, rings contiguous.
__global__ __launch_bounds__(256) void k_synth_parts_sum(char *F0, int64_t F_stride, int64_t part_stride,
                                                         const LegOrder *orders, const int32_t *band_bs,
                                                         const int32_t *ring_mmax, int nring, int mmax, int lmax,
                                                         int spin, int S) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t n = (int64_t)(2 * mmax + 1) * nring;
    if (e >= n) return;
    const int mi = (int)(e / nring), j = (int)(e - (int64_t)mi * nring);
    const int m = mi >= mmax ? mi - mmax : mmax - mi;
    const int l0 = m > spin ? m : spin;
    if (l0 > lmax || ring_mmax[j] < m) return;
    const LegOrder o = orders[m];
    const int k0 = (band_bs[o.band0 + ((o.last - j) >> 6)] - l0) / S;
    const int nseg = (lmax + 1 - l0 + S - 1) / S;
    if (nseg < k0 + 2) return;
    char *Fc = F0 + blockIdx.y * F_stride;
    double2 *F = reinterpret_cast<double2 *>(Fc);
    double2 acc = F[e];
    for (int k = k0 + 1; k < nseg; ++k) {
        const double2 v = reinterpret_cast<const double2 *>(Fc + k * part_stride)[e];
        acc.x += v.x;
        acc.y += v.y;
    }
    F[e] = acc;
}

// ---------------------------------------------------------------- adjoint
//
// An item sums the degrees [la, lb) of order m over every active ring of the
// order (or one group of its bands, see AdjArgs::accumulate): G waves hold the
// bands in turn (band i in wave i mod G), up to RMAX each, and take them in as
// l passes their starts.  Beyond its FMAs the adjoint pays for reducing each
// degree's four sums (Re and Im of A and B) over the 64 lanes, whatever the
// number of bands a lane holds: hence up to eight bands per lane, and the
// reduction goes through LDS.  Four degrees at a time, each lane writes its
// sums as two 16-byte values per degree and reads back eight lanes' values of
// one (degree, sum) pair: 7 complex additions per lane for 4 degrees, against
// 13 instructions per degree (of which 6 half-rate permlane swaps) for a
// transposed butterfly in registers.  The reads are consumed one step later,
// so that their latency overlaps the next degree's FMAs.  Once per chunk of 32
// degrees one wave adds the eight partial sums of every wave and writes each
// output once, coalesced, with a plain store (no atomics, no prior clear).
// Waves of an item meet only there.

// double2 per (degree, sum) row of 64 lanes: with rows half of the banks apart,
// lane i's read of entry (i >> 3, i & 7) has the bank of a contiguous read (at
// 66, four tenths of the LDS cycles were conflicts)
constexpr int kRedRow = 72;
constexpr int kRed1 = 8 * kRedRow, kRed2 = 8 * 64;  // a wave's reduction areas (double2): 4 degrees; 32 degrees

struct AdjArgs {
    LegArgs a;
    const AdjItem *items;
    int nitems;
    bool accumulate;  // band groups: add into the (cleared) output instead of storing
};

// Recurrence coefficients of 16 degrees, degree c + i in lane i of every
// 16-lane row: a step takes its own with three row broadcasts, which leaves the
// LDS pipe to the reduction (as LDS broadcasts they took a quarter of it).
struct RowCoef {
    double x, y, z;
};
__device__ inline RowCoef row_coef(const double4 *T4, int c, int lmax, int lane) {
    const int l = min(c + (lane & 15), lmax);
    return RowCoef{T4[l].x, T4[l].y, T4[l].z};
}

// The first R bands over the 4 nblk <= 32 degrees from c, whose coefficients
// are in T and then Tn (both move on by the degrees taken); block b's partial
// sums (lane 8 (2 u + pair) + h: step u, A or B, lanes h mod 8) go to red2[b].
// A block is read back in two groups of four values, after its last step and
// after the next block's first one.
template <int R, int RMAX, bool SPIN>
__device__ inline void adj_chunk(BandState<RMAX> &S, const double *fpr, const double *fpi, const double *fmr,
                                 const double *fmi, RowCoef &T, RowCoef &Tn, const double4 *T4, int c, int lmax,
                                 double2 *red1, double2 *red2, int nblk, int lane) {
    const double2 *rd = red1 + (lane >> 3) * kRedRow + (lane & 7);
    double2 v[4], p;
    auto sum4 = [&] {
        return make_double2((v[0].x + v[1].x) + (v[2].x + v[3].x), (v[0].y + v[1].y) + (v[2].y + v[3].y));
    };
    auto read4 = [&](int i0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = rd[8 * (i0 + i)];
    };
    auto step = [&](auto U, int b) {
        constexpr int u = decltype(U)::value & 3;
        const double tx = row_bcast<decltype(U)::value>(T.x), ty = row_bcast<decltype(U)::value>(T.y),
                     tz = SPIN ? row_bcast<decltype(U)::value>(T.z) : 0.0;
        double pa_r = 0.0, pa_i = 0.0, pb_r = 0.0, pb_i = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double vp = S.up[r], vm = SPIN ? S.um[r] : S.up[r];
            pa_r = fma(vp, fpr[r], pa_r);
            pa_i = fma(vp, fpi[r], pa_i);
            pb_r = fma(vm, fmr[r], pb_r);
            pb_i = fma(vm, fmi[r], pb_i);
            const double np = fma(fma(tx, S.y[r], ty), vp, -S.upp[r]);
            S.upp[r] = vp;
            S.up[r] = np;
            if (SPIN) {
                const double nm = fma(fma(tx, S.y[r], tz), vm, -S.ump[r]);
                S.ump[r] = vm;
                S.um[r] = nm;
            }
        }
        if (u == 0 && b > 0) {
            p = sum4();
            read4(4);  // before this step's writes to the same rows (LDS runs in program order)
        }
        if (u == 1 && b > 0) {
            const double2 q = sum4();
            red2[(b - 1) * 64 + lane] = make_double2(p.x + q.x, p.y + q.y);
        }
        red1[2 * u * kRedRow + lane] = make_double2(pa_r, pa_i);
        red1[(2 * u + 1) * kRedRow + lane] = make_double2(pb_r, pb_i);
        __builtin_amdgcn_sched_barrier(0);
        if (u == 3) {
            read4(0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
#pragma unroll 1
    for (int b = 0; b < nblk; b += 2) {
        step(std::integral_constant<int, 0>(), b);
        step(std::integral_constant<int, 1>(), b);
        step(std::integral_constant<int, 2>(), b);
        step(std::integral_constant<int, 3>(), b);
        if (b + 1 < nblk) {
            step(std::integral_constant<int, 4>(), b + 1);
            step(std::integral_constant<int, 5>(), b + 1);
            step(std::integral_constant<int, 6>(), b + 1);
            step(std::integral_constant<int, 7>(), b + 1);
        }
        if (b & 2) {
            T = Tn;
            Tn = row_coef(T4, c + 4 * b + 24, lmax, lane);
        } else {
            T.x = row_rotate8(T.x);
            T.y = row_rotate8(T.y);
            if (SPIN) T.z = row_rotate8(T.z);
        }
    }
    p = sum4();
    read4(4);
    const double2 q = sum4();
    red2[(nblk - 1) * 64 + lane] = make_double2(p.x + q.x, p.y + q.y);
}

// Barrier of an item's waves for LDS data only: waits for this wave's LDS
// operations, not for its outstanding global loads (the next coefficients stay
// in flight across the barrier), then s_barrier.  A wave that holds its item
// alone needs neither: its LDS operations run in program order, and only the
// compiler has to keep it.
__device__ inline void lds_barrier(bool alone) {
    asm volatile("" ::: "memory");
    if (!alone) {
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0); vmcnt and expcnt not waited for
        __builtin_amdgcn_s_barrier();
    }
    asm volatile("" ::: "memory");
}

// Zero outputs of order m for l in [l_from, l_to), by thread i of n.
__device__ inline void adj_zero_range(const LegArgs &a, double *dst, int64_t base, int l_from, int l_to, int i, int n) {
    double2 *out = reinterpret_cast<double2 *>(dst);
    for (int l = l_from + i; l < l_to; l += n) {
        out[base + l] = make_double2(0.0, 0.0);
        out[a.nalm + base + l] = make_double2(0.0, 0.0);
    }
}

// What an item's wave works on.
struct AdjWave {
    const LegArgs &a;
    const LegBand *bands;  // of the item
    const double4 *T4;
    const double2 *Fp, *Fm;
    double *out;  // complex [2][nalm]
    double2 *red1, *red2, *red2all;
    int64_t base;
    int m, l0, la, lb, nb, G, wave, lane;
    bool accumulate;
};

// The wave's band i of the item into slot r.
template <int RMAX, bool SPIN>
__device__ __forceinline__ void adj_load(const AdjWave &w, int r, int i, BandState<RMAX> &S, double *fpr, double *fpi,
                                         double *fmr, double *fmi) {
    const LegBand b = w.bands[i];
    const int j = band_ring(b, w.lane);
    band_load<RMAX, SPIN>(w.a, r, j, band_state(b, w.la, w.l0, w.a.seg, w.lane), S);
    if (j >= 0) {
        const double2 vp = w.Fp[j], vm = w.Fm[j];
        fpr[r] = vp.x;
        fpi[r] = vp.y;
        fmr[r] = vm.x;
        fmi[r] = vm.y;
    }
}

// Adds the eight partials of every wave of the chunk from c and writes its n
// degrees: lane 2 t + pair holds A or B of step t (rotated start: the lanes of
// one LDS phase read distinct banks), the lane pair exchanges them and writes
// g~ and c~.  P: that of degree c + t.
__device__ __forceinline__ void adj_write(const AdjWave &w, int c, int n, double P) {
    double sr = 0.0, si = 0.0;
    for (int g = 0; g < w.G; ++g) {
        const double2 *r2 = w.red2all + g * kRed2 + w.lane * 8;
#pragma unroll
        for (int h = 0; h < 8; ++h) {
            const double2 v = r2[(h + (w.lane >> 1)) & 7];
            sr += v.x;
            si += v.y;
        }
    }
    if (w.lane & 1) si = -si;  // B sums conj F'(-m)
    const double orr = quad_xor1(sr), oi = quad_xor1(si);
    const int t = w.lane >> 1;
    if (t >= n) return;
    const double sgn_s = (w.a.spin & 1) ? -1.0 : 1.0;
    const double hP = (w.m == 0 ? 0.5 : 0.5 * w.a.mscale) * P;
    double2 val;
    double *dst = w.out + 2 * (w.base + c + t);
    // Im g~_l0 and Im c~_l0 vanish (reality condition)
    if ((w.lane & 1) == 0) {  // g~ = -hP (A + (-1)^s B)
        val.x = -hP * (sr + sgn_s * orr);
        val.y = w.m == 0 ? 0.0 : -hP * (si + sgn_s * oi);
    } else {  // c~ = i hP (A - (-1)^s B)
        val.x = -hP * (oi - sgn_s * si);
        val.y = w.m == 0 ? 0.0 : hP * (orr - sgn_s * sr);
        dst += 2 * w.a.nalm;
    }
    if (w.accumulate) {
        atomicAdd(dst, val.x);
        atomicAdd(dst + 1, val.y);
    } else {
        *reinterpret_cast<double2 *>(dst) = val;
    }
}

// The chunks from c while the wave has R bands, then those with one more.  The
// next band is loaded during the last chunk before it enters.  (One loop per R:
// a switch over R inside a common loop shuffled the bands between registers
// and scratch at every chunk, a fifth of all instructions.)
template <int R, int RMAX, bool SPIN>
__device__ __forceinline__ void adj_run(const AdjWave &w, BandState<RMAX> &S, double *fpr, double *fpi, double *fmr,
                                        double *fmi, RowCoef &T, RowCoef &Tn, int c) {
    const int i = R * w.G + w.wave;  // the wave's next band
    const bool more = R < RMAX && i < w.nb;
    const int cend = more ? min(band_enter(w.bands[i], w.la), w.lb) : w.lb;
    const int lmax = w.a.lmax;
    if constexpr (R < RMAX)
        if (more && c >= cend) adj_load<RMAX, SPIN>(w, R, i, S, fpr, fpi, fmr, fmi);  // enters with the one before
#pragma unroll 1
    for (; c < cend; c += kStage) {
        // P of the degree whose outputs this lane may write
        const double P = w.T4[min(c + (w.lane >> 1), lmax)].w;
        if constexpr (R < RMAX)
            if (more && c + kStage >= cend) adj_load<RMAX, SPIN>(w, R, i, S, fpr, fpi, fmr, fmi);
        const int n = min(kStage, w.lb - c), nblk = (n + 3) >> 2;
        if constexpr (R == 0) {
            for (int b = 0; b < nblk; ++b) w.red2[b * 64 + w.lane] = make_double2(0.0, 0.0);
            T = row_coef(w.T4, c + kStage, lmax, w.lane);
            Tn = row_coef(w.T4, c + kStage + 16, lmax, w.lane);
        } else {
            adj_chunk<R, RMAX, SPIN>(S, fpr, fpi, fmr, fmi, T, Tn, w.T4, c, lmax, w.red1, w.red2, nblk, w.lane);
        }
        lds_barrier(w.G == 1);
        if (w.G == 1 || (((c - w.la) / kStage) & (w.G - 1)) == w.wave) adj_write(w, c, n, P);
        lds_barrier(w.G == 1);
    }
    if constexpr (R < RMAX) {
        if (c < w.lb) adj_run<R + 1, RMAX, SPIN>(w, S, fpr, fpi, fmr, fmi, T, Tn, c);
    }
}

// A workgroup of wg waves (1, 2 or 4) holds one item of wg waves, or wg items
// of one wave each (orders or segments with at most RMAX started bands: more
// bands per wave, no barriers).
template <bool SPIN, int RMAX>
__device__ inline void adj_item(const AdjArgs &A, int w0) {
    extern __shared__ __align__(16) double2 redbase[];  // per wave: kRed1, then kRed2 of every wave
    const LegArgs &a = A.a;
    const int wg = blockDim.x >> 6, lane = threadIdx.x & 63;
    if ((int)blockIdx.x * wg + w0 >= A.nitems) return;
    const AdjItem it = A.items[blockIdx.x * wg + w0];
    const int G = it.waves, wave = G == 1 ? 0 : w0;
    const int m = it.m, s = a.spin, lmax = a.lmax;
    const int l0 = m > s ? m : s;
    const int64_t base = (int64_t)m * (2 * lmax + 1 - m) / 2;
    const LegBand *bands = a.bands + it.b0;
    const int la = max(it.la, l0);
    const int c0 = it.nb > 0 ? band_enter(bands[0], la) : it.lb;
    double *out = reinterpret_cast<double *>(a.alm_out + blockIdx.y * a.alm_stride);
    // no ring has started (or l < s)
    if (!A.accumulate) adj_zero_range(a, out, base, it.la, min(c0, it.lb), 64 * wave + lane, 64 * G);
    if (it.nb <= 0) return;
    double2 *red2 = redbase + wg * kRed1 + w0 * kRed2;
    const double2 *F = reinterpret_cast<const double2 *>(a.F + blockIdx.y * a.F_stride);
    const double4 *T4 = a.coef + base;
    const AdjWave w{a,    bands, T4, F + (int64_t)(a.mmax + m) * a.nring, F + (int64_t)(a.mmax - m) * a.nring,
                    out,  redbase + w0 * kRed1, red2, red2 - wave * kRed2, base, m, l0, la, it.lb, it.nb, G, wave, lane,
                    A.accumulate};
    BandState<RMAX> S;
    double fpr[RMAX], fpi[RMAX], fmr[RMAX], fmi[RMAX];
#pragma unroll
    for (int r = 0; r < RMAX; ++r) {
        S.y[r] = S.up[r] = S.upp[r] = S.um[r] = S.ump[r] = 0.0;
        fpr[r] = fpi[r] = fmr[r] = fmi[r] = 0.0;
    }
    RowCoef T = row_coef(T4, c0, lmax, lane), Tn = row_coef(T4, c0 + 16, lmax, lane);
    adj_run<0, RMAX, SPIN>(w, S, fpr, fpi, fmr, fmi, T, Tn, c0);
}

// The item's outputs in [live, start), whose terms adj_item left out: NaN in place
// of the zeros it wrote where the order's ring values are not finite (each thread
// overwrites its own).  After the sums and from the item again, with the lane from
// mbcnt: what it needs would otherwise be held in registers through them (k_leg_adj8
// spills).  One ring stands for the order: the transforms before spread a value
// that is not finite over all of them.
__device__ inline void adj_non_finite(const AdjArgs &A, int w0) {
    const LegArgs &a = A.a;
    const int64_t at = (int64_t)blockIdx.x * (blockDim.x >> 6) + w0;
    if (at >= A.nitems) return;
    const AdjItem it = A.items[at];
    const int from = max(it.live, it.la), to = min(it.start, it.lb);
    if (from >= to) return;
    const double2 *F = reinterpret_cast<const double2 *>(a.F + blockIdx.y * a.F_stride) + it.ring;
    const double2 vp = F[(int64_t)(a.mmax + it.m) * a.nring], vm = F[(int64_t)(a.mmax - it.m) * a.nring];
    if (isfinite(vp.x) && isfinite(vp.y) && isfinite(vm.x) && isfinite(vm.y)) return;
    const int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    double2 *out = reinterpret_cast<double2 *>(a.alm_out + blockIdx.y * a.alm_stride) +
                   (int64_t)it.m * (2 * a.lmax + 1 - it.m) / 2;
    for (int l = it.la + (it.waves > 1 ? 64 * w0 : 0) + lane; l < to; l += 64 * it.waves)
        if (l >= from) out[l] = out[a.nalm + l] = make_double2(NAN, it.m ? NAN : 0.0);
}

template <bool SPIN>
__global__ __launch_bounds__(256, 2) void k_leg_adj8(AdjArgs A) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    adj_item<SPIN, 8>(A, wave);
    adj_non_finite(A, wave);
}
template <bool SPIN>
__global__ __launch_bounds__(256, 2) void k_leg_adj4(AdjArgs A) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    adj_item<SPIN, 4>(A, wave);
    adj_non_finite(A, wave);
}

// ------------------------------------------------------- starts and states

// Plan time, one wave per band: the degree l0 + 32 i of the chunk in which a
// ring of the band first has |lambda+-| >= 2^kLegStartExp (at most the last
// chunk of the order), and the degree l0 + 8 i from which on one has a value
// in the unscaled range (at or above 2^-312, or a seed above 2^-600).
template <bool SPIN>
__global__ __launch_bounds__(64) void k_leg_starts(LegArgs a, const LegBand *bands, int nbands, int32_t *bs,
                                                   int32_t *live) {
    if ((int)blockIdx.x >= nbands) return;
    const LegBand b = bands[blockIdx.x];
    const int lane = threadIdx.x, m = b.order, s = a.spin, lmax = a.lmax;
    const int l0 = m > s ? m : s;
    const int j = band_ring(b, lane);
    const bool act = j >= 0;
    const double thr = ldexp(1.0, kLegStartExp);
    double y = 0.0, up = 0.0, um = 0.0, upp = 0.0, ump = 0.0;
    int kp = 0, km = 0;
    if (act) {
        y = a.ring_y[j];
        leg_seed(a.kmant[m], a.kexp[m], m, s, a.ring_ch[j], a.ring_sh[j], up, kp, um, km);
    }
    const double4 *T4 = a.coef + (int64_t)m * (2 * lmax + 1 - m) / 2;
    auto unscaled = [&] { return __any(act && (kp == 0 || (SPIN && km == 0))); };
    int c = l0, from = -1;
    for (; c + kStage <= lmax; c += kStage) {
        bool hit = false;
        if (from < 0 && unscaled()) from = c;
#pragma unroll 8
        for (int t = 0; t < kStage; ++t) {
            const double4 f = T4[c + t];
            hit |= kp == 0 && fabs(f.w * up) >= thr;
            double n = fma(fma(f.x, y, f.y), up, -upp);
            upp = up;
            up = n;
            if (SPIN) {
                hit |= km == 0 && fabs(f.w * um) >= thr;
                n = fma(fma(f.x, y, f.z), um, -ump);
                ump = um;
                um = n;
            }
            if ((t & 7) == 7) {  // 8 steps grow a value by far less than the headroom above 2^200
                leg_rescale(up, upp, kp);
                if (SPIN) leg_rescale(um, ump, km);
                if (from < 0 && unscaled()) from = c + t + 1;
            }
        }
        if (__any(hit)) break;
    }
    if (lane == 0) {
        bs[blockIdx.x] = c;
        live[blockIdx.x] = from < 0 || from > c ? c : from;
    }
}

// Plan time, one wave per band: stores the state (mu_l, mu_{l-1}) of both signs
// at the band's start bs and at every segment start l0 + k seg above it (in
// blocks of 64 from blk).  The values are stored in the double range: a value
// below 2^-960 there (a ring far inside its band, or the weaker sign at high
// spin) would lose digits.  lost[0] counts the rings in which such a value grows
// past the start threshold before the next stored state: the adjoint's items,
// which run from one stored state to the next, then need shorter segments.
// lost[1] counts those in which it does so at any later degree: the items of the
// synthesis run over several stored states, up to lmax (the plain list), and
// then have to take them in on the way.
template <bool SPIN>
__global__ __launch_bounds__(64) void k_leg_states(LegArgs a, int nbands, double2 *st_p, double2 *st_m,
                                                   int32_t *lost) {
    if ((int)blockIdx.x >= nbands) return;
    const LegBand w = a.bands[blockIdx.x];
    const int lane = threadIdx.x, m = w.order, s = a.spin, lmax = a.lmax;
    const int l0 = m > s ? m : s;
    const int j = band_ring(w, lane);
    const bool act = j >= 0;
    const double thr = ldexp(1.0, kLegStartExp), low = ldexp(1.0, -960);
    double y = 0.0, up = 0.0, um = 0.0, upp = 0.0, ump = 0.0;
    int kp = 0, km = 0;
    if (act) {
        y = a.ring_y[j];
        leg_seed(a.kmant[m], a.kexp[m], m, s, a.ring_ch[j], a.ring_sh[j], up, kp, um, km);
    }
    const double4 *T4 = a.coef + (int64_t)m * (2 * lmax + 1 - m) / 2;
    const int lsteps = lmax - l0;
    bool lp = false, lm = false, bad = false;       // since the last stored state
    bool anyp = false, anym = false, late = false;  // since any
    // l advances in steps of 32 between the points that may store (bs and the
    // segment starts are multiples of 32 from l0); seg is a multiple of 64
    int64_t q = (int64_t)w.blk * 64 + lane;
    const int klast = lsteps / a.seg;
    for (int c = l0; c <= lmax; c += kStage) {
        if (c == w.bs || (c > w.bs && (c - l0) % a.seg == 0)) {
            const double vp = ldexp(up, kScaleStep * kp), vm = SPIN ? ldexp(um, kScaleStep * km) : vp;
            st_p[q] = make_double2(vp, ldexp(upp, kScaleStep * kp));
            lp = up != 0.0 && fabs(vp) < low;
            if (SPIN) {
                st_m[q] = make_double2(vm, ldexp(ump, kScaleStep * km));
                lm = um != 0.0 && fabs(vm) < low;
            }
            anyp |= lp;
            anym |= lm;
            q += 64;
        }
        if (c > w.bs && c - l0 >= klast * a.seg && !(anyp || anym)) break;
        const int n = min(kStage, lmax + 1 - c);
#pragma unroll 8
        for (int t = 0; t < n; ++t) {
            const double4 f = T4[c + t];
            const bool on = kp == 0 && fabs(f.w * up) >= thr;
            bad |= lp && on;
            late |= anyp && on;
            double v = fma(fma(f.x, y, f.y), up, -upp);
            upp = up;
            up = v;
            if (SPIN) {
                const bool om = km == 0 && fabs(f.w * um) >= thr;
                bad |= lm && om;
                late |= anym && om;
                v = fma(fma(f.x, y, f.z), um, -ump);
                ump = um;
                um = v;
            }
            if ((t & 7) == 7) {
                leg_rescale(up, upp, kp);
                if (SPIN) leg_rescale(um, ump, km);
            }
        }
    }
    if (bad) atomicAdd(lost, 1);
    if (late) atomicAdd(lost + 1, 1);
}

static LegArgs leg_args(const psht_plan_s &p, const void *alm_in, void *alm_out, void *F, const MapBatch &mb) {
    const Geometry &g = p.g;
    LegArgs a;
    a.bands = p.d_bands;
    a.st_p = reinterpret_cast<const double2 *>(p.d_st_p);
    a.st_m = reinterpret_cast<const double2 *>(p.d_st_m);
    a.seg = p.adj_seg;
    a.coef = reinterpret_cast<const double4 *>(p.leg->d_coef);
    a.kmant = p.leg->d_kmant;
    a.kexp = p.leg->d_kexp;
    a.ring_y = p.d_ring_y;
    a.ring_ch = p.d_ring_ch;
    a.ring_sh = p.d_ring_sh;
    a.nring = g.nring;
    a.lmax = g.lmax;
    a.spin = g.spin;
    a.mmax = g.mmax;
    a.nalm = (int64_t)(g.lmax + 1) * (g.lmax + 2) / 2;
    a.alm_in = static_cast<const char *>(alm_in);
    a.alm_out = static_cast<char *>(alm_out);
    a.F = static_cast<char *>(F);
    a.alm_stride = 2 * 16 * a.nalm;
    a.F_stride = mb.ws_stride;
    a.nmaps = mb.n;
    a.mscale = 1.0;
    return a;
}

// Bands per wave of the synthesis: PSHT_LEG_R (1, 2 or 4) fixes it for tuning
// runs; without it 0, and the plan chooses by the size of its work list.
int leg_bands_per_wave() {
    static const int r = [] {
        const char *e = getenv("PSHT_LEG_R");
        const int v = e ? atoi(e) : 0;
        return v == 1 || v == 2 || v == 4 ? v : 0;
    }();
    return r;
}

template <int R, int NM>
static void leg_synth_run(const SynthArgs &A, int spin, hipStream_t st) {
    const dim3 grid(A.nitems, (A.a.nmaps + NM - 1) / NM), block(64);
    if (spin) {
        hipLaunchKernelGGL((k_leg_synth<R, NM, true>), grid, block, 0, st, A);
    } else {
        if constexpr (NM <= 2) hipLaunchKernelGGL((k_leg_synth<R, NM, false>), grid, block, 0, st, A);
    }
}

// NM maps per wave share the recurrence (4 of the 8 FMAs per ring, degree and
// map with a spin; 2 of 6 without): 6 FMAs per map with two maps, 5 with four.
// Four fit the registers beside two bands (210 VGPRs) and pay with a spin only
// (lmax 2048, 8 maps, us per map: spin 2 on a 34-degree cap 128 against 145 with
// two; spin 0 on 20 degrees 58 against 60, on fewer maps slower); with four
// bands they leave one wave per SIMD (lmax 4096: 915 against 822 with two).
template <int R>
static hipError_t leg_synth_maps(SynthArgs A, int spin, hipStream_t st) {
    LegArgs &a = A.a;
    const int total = a.nmaps;
    for (int done = 0; done < total; done += a.nmaps) {
        const int left = total - done;
        if constexpr (R <= 2) {
            if (spin && left >= 3) {  // whole groups of four; three left over fill a group but for one
                a.nmaps = left % 4 == 3 ? left : left / 4 * 4;
                leg_synth_run<R, 4>(A, spin, st);
                a.alm_in += a.nmaps * a.alm_stride;
                a.F += a.nmaps * a.F_stride;
                continue;
            }
        }
        a.nmaps = left;
        if (left >= 2) leg_synth_run<R, 2>(A, spin, st);
        else leg_synth_run<R, 1>(A, spin, st);
    }
    return hipGetLastError();
}

static hipError_t leg_synth_list(const psht_plan_s &p, SynthArgs &A, const SynthItem *items, int nitems, int R,
                                 hipStream_t st) {
    if (nitems == 0) return hipSuccess;
    A.items = items;
    A.nitems = nitems;
    if (p.syn_reload) {
        // one kernel for such plans (lists of at most two bands, one map per wave)
        const dim3 grid(nitems, A.a.nmaps), block(64);
        if (p.g.spin)
            hipLaunchKernelGGL((k_leg_synth<kSynthReloadBands, 1, true, true>), grid, block, 0, st, A);
        else
            hipLaunchKernelGGL((k_leg_synth<kSynthReloadBands, 1, false, true>), grid, block, 0, st, A);
        return hipGetLastError();
    }
    if (R == 4) return leg_synth_maps<4>(A, p.g.spin, st);
    if (R == 2) return leg_synth_maps<2>(A, p.g.spin, st);
    return leg_synth_maps<1>(A, p.g.spin, st);
}

hipError_t launch_leg_synth(const psht_plan_s &p, const void *alm, void *F, bool segments, const MapBatch &mb,
                            double mscale, hipStream_t st) {
    SynthArgs A;
    A.a = leg_args(p, alm, nullptr, F, mb);
    A.a.mscale = mscale;
    A.part_stride = (int64_t)p.ws_F;
    const bool multi = mb.n >= 3;
    const int seg = !segments ? 0 : multi && p.syn_seg > 0 ? p.multi_seg : p.syn_seg;
    if (seg == 0) return leg_synth_list(p, A, p.d_leg_items, p.n_leg_items, p.leg_r, st);
    const hipError_t e = multi ? leg_synth_list(p, A, p.d_multi_items, p.n_multi_items, p.multi_r, st)
                               : leg_synth_list(p, A, p.d_syn_items, p.n_syn_items, p.syn_r, st);
    if (e != hipSuccess || p.syn_parts == 0) return e;
    const int64_t n = (int64_t)(2 * p.g.mmax + 1) * p.g.nring;
    hipLaunchKernelGGL(k_synth_parts_sum, dim3((unsigned)((n + 255) / 256), mb.n), dim3(256), 0, st,
                       static_cast<char *>(F), mb.ws_stride, (int64_t)p.ws_F, p.d_orders, p.d_band_bs, p.d_ring_mmax,
                       p.g.nring, p.g.mmax, p.g.lmax, p.g.spin, seg);
    return hipGetLastError();
}

hipError_t launch_leg_starts(const psht_plan_s &p, const LegBand *bands, int nbands, int32_t *bs, int32_t *live,
                             hipStream_t st) {
    if (nbands == 0) return hipSuccess;
    const LegArgs a = leg_args(p, nullptr, nullptr, nullptr, MapBatch());
    if (p.g.spin) hipLaunchKernelGGL(k_leg_starts<true>, dim3(nbands), dim3(64), 0, st, a, bands, nbands, bs, live);
    else hipLaunchKernelGGL(k_leg_starts<false>, dim3(nbands), dim3(64), 0, st, a, bands, nbands, bs, live);
    return hipGetLastError();
}

hipError_t launch_leg_states(const psht_plan_s &p, int nbands, int32_t *lost, hipStream_t st) {
    if (nbands == 0) return hipSuccess;
    const LegArgs a = leg_args(p, nullptr, nullptr, nullptr, MapBatch());
    double2 *sp = reinterpret_cast<double2 *>(p.d_st_p), *sm = reinterpret_cast<double2 *>(p.d_st_m);
    if (p.g.spin)
        hipLaunchKernelGGL(k_leg_states<true>, dim3(nbands), dim3(64), 0, st, a, nbands, sp, sm, lost);
    else
        hipLaunchKernelGGL(k_leg_states<false>, dim3(nbands), dim3(64), 0, st, a, nbands, sp, sm, lost);
    return hipGetLastError();
}

template <typename K>
static hipError_t leg_adjoint_run(K kern, const psht_plan_s &p, const AdjArgs &A, hipStream_t st) {
    const size_t lds = sizeof(double2) * (size_t)p.adj_waves * (kRed1 + kRed2);
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(p.n_adj_items / p.adj_waves, A.a.nmaps), dim3(64 * p.adj_waves), lds, st, A);
    return hipGetLastError();
}

hipError_t launch_leg_adjoint(const psht_plan_s &p, const void *F, void *alm, const MapBatch &mb, double mscale,
                              hipStream_t st) {
    const int64_t nalm = (int64_t)(p.g.lmax + 1) * (p.g.lmax + 2) / 2;
    if (p.adj_accumulate) {
        const hipError_t e = launch_fill_zero(alm, (size_t)nalm * 2 * 16 * mb.n, st);
        if (e != hipSuccess) return e;
    }
    if (p.n_adj_items == 0) return hipSuccess;
    AdjArgs A;
    A.a = leg_args(p, nullptr, alm, const_cast<void *>(F), mb);
    A.a.mscale = mscale;
    A.items = p.d_adj_items;
    A.nitems = p.n_adj_items;
    A.accumulate = p.adj_accumulate;
    if (p.adj_rmax <= 4)
        return p.g.spin ? leg_adjoint_run(k_leg_adj4<true>, p, A, st) : leg_adjoint_run(k_leg_adj4<false>, p, A, st);
    return p.g.spin ? leg_adjoint_run(k_leg_adj8<true>, p, A, st) : leg_adjoint_run(k_leg_adj8<false>, p, A, st);
}

}  // namespace psht
