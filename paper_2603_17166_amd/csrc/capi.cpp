// C ABI of libpsht (declared in include/psht.h): argument validation, plan
// construction (point statistics, geometry, tables, point sort), workspace
// layout and the stage sequences of synthesis and adjoint synthesis.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <vector>
#include <new>
#include <string>
#include <tuple>

#include "leg_common.h"
#include "nufft_index.h"
#include "psht_internal.h"
#include "rot_factor.h"

namespace {

thread_local std::string g_last_error;

psht_status fail(psht_status code, const std::string &msg) {
    g_last_error = msg;
    return code;
}

psht_status fail(const psht::Error &e) { return fail(e.code, e.msg); }

psht_status device_fail(hipError_t e, const char *what) {
    return fail(e == hipErrorOutOfMemory ? PSHT_ERR_NOMEM : PSHT_ERR_DEVICE,
                std::string(what) + ": " + hipGetErrorString(e));
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

template <typename T> bool dalloc(psht_plan_s &p, T *&ptr, size_t count) {
    void *raw = nullptr;
    size_t bytes = std::max<size_t>(count, 1) * sizeof(T);
    if (hipMalloc(&raw, bytes) != hipSuccess) return false;
    p.allocations.push_back(raw);
    p.resident += bytes;
    ptr = static_cast<T *>(raw);
    return true;
}

// Synchronous upload: the host vectors are temporaries of plan creation.
template <typename T> bool upload(psht_plan_s &p, T *&ptr, const std::vector<T> &host, hipStream_t) {
    if (!dalloc(p, ptr, host.size())) return false;
    if (host.empty()) return true;
    return hipMemcpy(ptr, host.data(), host.size() * sizeof(T), hipMemcpyHostToDevice) == hipSuccess;
}

void free_plan(psht_plan_s *p) {
    if (!p) return;
    for (auto &e : p->pending) {
        (void)hipEventDestroy(e.second.first);
        (void)hipEventDestroy(e.second.second);
    }
    for (hipEvent_t e : p->event_pool) (void)hipEventDestroy(e);
    for (void *a : p->allocations) (void)hipFree(a);
    delete p;
}

hipEvent_t take_event(psht_plan_s &p) {
    if (!p.event_pool.empty()) {
        hipEvent_t e = p.event_pool.back();
        p.event_pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}

// Runs one stage launch, bracketed by timing events when timing is on.
template <typename Fn> hipError_t timed(psht_plan_s &p, int stage, hipStream_t st, Fn fn) {
    if (!((p.timing >> stage) & 1u)) return fn();
    hipEvent_t a = take_event(p), b = take_event(p);
    if (!a || !b) return fn();
    (void)hipEventRecord(a, st);
    hipError_t e = fn();
    (void)hipEventRecord(b, st);
    p.pending.push_back({stage, {a, b}});
    return e;
}

// fp32: the table serves transforms of float data (they take other radices).
bool make_fft_table(psht_plan_s &p, psht::FftTable &t, int n, bool fp32, hipStream_t st) {
    if (!psht::fft_factor(n, fp32, t.f)) return false;
    t.n = n;
    std::vector<double> tw(2 * (size_t)n);
    const long double pi = 3.141592653589793238462643383279502884L;
    for (int k = 0; k < n; ++k) {
        long double a = 2 * pi * k / n;
        tw[2 * k] = (double)cosl(a);
        tw[2 * k + 1] = (double)(-sinl(a));
    }
    return upload(p, t.d_tw, tw, st);
}

void fill_info(const psht_plan_s &p, psht_plan_info *info) {
    const psht::Geometry &g = p.g;
    std::memset(info, 0, sizeof(*info));
    info->lmax = g.lmax;
    info->spin = g.spin;
    info->Lmax = g.Lmax;
    info->n2 = g.N2;
    info->mmax = g.mmax;
    info->nufft_w = g.W;
    info->ntheta_grid = g.Ntheta;
    info->nphi_grid = g.Nphi;
    info->row_lo = g.row_lo;
    info->rows_used = g.rows_used;
    info->map_is_fp32 = g.fp32 ? 1 : 0;
    info->full_sky = g.full_sky ? 1 : 0;
    info->epsilon = g.eps;
    info->theta_star = g.theta_star;
    info->theta_min = g.theta_min;
    info->theta_max = g.theta_max;
    info->eps_apo = g.eps_apo;
    info->alpha = g.alpha;
    info->nufft_beta = g.beta;
    info->nufft_sigma = g.sigma;
    info->predicted_speedup = g.predicted_speedup;
    info->legendre_triples = g.legendre_triples;
    info->npoints = p.npts;
    info->resident_bytes = p.resident + (p.leg ? p.leg->bytes : 0);
    info->shared_bytes = p.leg ? p.leg->bytes : 0;
    info->workspace_bytes_per_map = p.ws_per_map;
    info->kernel_poly_err = g.es_poly_err;
    info->adj_segment = p.adj_seg;
    info->adj_waves = p.adj_waves;
    info->adj_rings_per_lane = p.adj_rmax;
    info->adj_states = p.n_adj_states;
    info->Lmax_rule = g.Lmax_rule;
    info->predicted_error = g.predicted_error;
    info->window = g.window;
    info->syn_segment = p.syn_seg;
    info->syn_parts = p.syn_parts;
}

struct ScopedDevFree {
    void *p = nullptr;
    ~ScopedDevFree() {
        if (p) (void)hipFree(p);
    }
};

// Segment length of the synthesis.  The synthesis runs one wave per (order m,
// group of bands) over the degrees of m; a small cap at high lmax has few such
// items (a few hundred orders), each thousands of sequential steps long, and
// leaves most of the GPU idle.  Such a plan cuts the degrees of every order
// into segments; segment k >= 1 of an order writes its own partial copy of F,
// which a second kernel adds in.  The length is the largest power of two (at
// least 64) for which the longest item costs at most a third of the average
// work per wave slot (two waves per SIMD), lengthened where needed to at most
// 33 segments per order (32 partial copies).  Orders shorter than three segments
// of less than 256 degrees are not segmented (the partial-sum launch costs what
// they gain: lmax 128 cap 10.3 against 9.7 us); longer ones are, from two
// segments on (lmax 3000, 1000 deg^2: 0.45 -> 0.32 ms; lmax 4096, 1500 deg^2:
// 1.00 -> 0.97 ms), unless their copies would enlarge the workspace.  A length of
// 2048 and more that holds a whole order is halved to give two segments (us of the
// stage, segments of 1024 or 2048 / none, spin 2: lmax 2000, 45 degrees 300 / 317;
// lmax 3000, 40 degrees 647 / 672; lmax 4096, 34 degrees 1068 / 1093, but 60 degrees
// 2530 / 2467 and lmax 6000, 30 degrees 2341 / 2290); shorter ones are not, since
// orders of up to 1024 degrees lose by two segments (lmax 1000, 60 degrees, 512
// degrees each 104 / 97).  The work is counted over all degrees l >= m, in steps
// of 128 rings, so that the size of the workspace does not depend on where the
// bands start.  Returns 0 for no segments.
int synth_segment_length(const psht::Geometry &g, int ncu, const std::vector<int> &first,
                         const std::vector<int> &last) {
    const int lmax = g.lmax, s = g.spin, M = g.mmax;
    double total = 0.0;
    for (int m = 0; m <= M; ++m) {
        if (first[m] < 0 || std::max(m, s) > lmax) continue;
        const int steps = lmax + 1 - std::max(m, s), nr = last[m] - first[m] + 1;
        for (int r = nr; r > 0; r -= 128) total += r <= 64 ? 0.5 * steps : steps;
    }
    const double slots = (double)std::max(ncu, 1) * 4 * 2;
    int S = 64;
    while ((double)S * 2 <= total / slots / 3.0) S *= 2;
    while ((int64_t)33 * S < (int64_t)lmax + 1 - s) S *= 2;
    if (const char *e = getenv("PSHT_SYN_SEG")) {  // tests and tuning runs: a power of two, at least 64; 0 for none
        const int v = atoi(e);
        if (v == 0) return 0;
        if (v >= 64 && (v & (v - 1)) == 0) return v;
    }
    const int n = lmax + 1 - s;
    if (3 * S <= n) return S;
    while (S >= 2048 && S >= n) S /= 2;
    if (S < 256 || S >= n) return 0;
    // two or three segments, where the copies fit the V and U region
    const size_t cs = g.fp32 ? 8 : 16, ldv = 2 * (size_t)M + 1;
    const size_t copies = (size_t)((n + S - 1) / S - 1) * ldv * g.nring * 16;
    return copies <= (size_t)g.rows_used * (ldv + g.Nphi) * cs ? S : 0;
}

// Bands, stored states and work lists of the Legendre stages.
//
// Adjoint.  The plan takes the smallest G of 1, 2, 4 waves per workgroup with
// 512 G >= rings (at most 8 bands per wave).  An item covers every started band
// of its order over one segment of S degrees: S is the largest power of two (at
// least 64) for which the longest item costs at most a third of the average
// work per wave slot (two waves per SIMD): with longest-first placement the
// last items then finish close together.  An order with more bands than one
// item holds (32 at G = 4) is cut into band groups; their items add into the
// output, which is cleared first.
bool build_legendre(psht_plan_s &p, int ncu, hipStream_t st, psht::Error &err) {
    const psht::Geometry &g = p.g;
    const int lmax = g.lmax, s = g.spin, M = g.mmax;
    auto nomem = [&](const char *what) {
        err = {PSHT_ERR_NOMEM, what};
        return false;
    };
    auto device = [&](hipError_t e, const char *what) {
        err = {e == hipErrorOutOfMemory ? PSHT_ERR_NOMEM : PSHT_ERR_DEVICE,
               std::string(what) + ": " + hipGetErrorString(e)};
        return false;
    };
    std::vector<int> first(M + 1, -1), last(M + 1, -1);
    for (int j = 0; j < g.nring; ++j)
        for (int m = 0; m <= std::min(M, (int)g.ring_mmax[j]); ++m) {
            if (first[m] < 0) first[m] = j;
            last[m] = j;
        }
    // bands of each order from its last ring downwards
    std::vector<psht::LegBand> geo;
    std::vector<psht::LegOrder> orders(M + 2);
    int nrmax = 1;
    for (int m = 0; m <= M; ++m) {
        orders[m] = psht::LegOrder{last[m], (int32_t)geo.size()};
        if (first[m] < 0 || std::max(m, s) > lmax) continue;
        nrmax = std::max(nrmax, last[m] - first[m] + 1);
        for (int top = last[m]; top >= first[m]; top -= 64)
        {
            uint64_t mask = 0;
            for (int i = 0; i < 64; ++i) {
                const int j = top - 63 + i;
                if (j >= first[m] && g.ring_mmax[j] >= m) mask |= uint64_t(1) << i;
            }
            geo.push_back(psht::LegBand{top - 63, 0, 0, m, mask});
        }
    }
    orders[M + 1] = psht::LegOrder{-1, (int32_t)geo.size()};
    const int nbands = (int)geo.size();
    std::vector<int32_t> bs(nbands), live(nbands);
    ScopedDevFree d_init, d_live, d_lost;
    hipError_t e = hipMalloc(&d_init.p, sizeof(psht::LegBand) * (size_t)std::max(nbands, 1));
    if (e == hipSuccess) e = hipMalloc(&d_live.p, sizeof(int32_t) * (size_t)std::max(nbands, 1));
    if (e == hipSuccess) e = hipMalloc(&d_lost.p, 2 * sizeof(int32_t));
    if (e != hipSuccess) return device(e, "Legendre bands");
    auto *init = static_cast<psht::LegBand *>(d_init.p);
    auto *d_lv = static_cast<int32_t *>(d_live.p);
    if (!dalloc(p, p.d_band_bs, nbands) || !upload(p, p.d_orders, orders, st)) return nomem("Legendre bands");
    if (nbands > 0) {
        e = hipMemcpy(init, geo.data(), sizeof(geo[0]) * nbands, hipMemcpyHostToDevice);
        if (e == hipSuccess) e = psht::launch_leg_starts(p, init, nbands, p.d_band_bs, d_lv, st);
        if (e == hipSuccess)
            e = hipMemcpyAsync(bs.data(), p.d_band_bs, sizeof(int32_t) * nbands, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipMemcpyAsync(live.data(), d_lv, sizeof(int32_t) * nbands, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return device(e, "Legendre start degrees");
    }
    // by order: the first degree at which a ring is in the unscaled range
    std::vector<int32_t> olive(M + 1, lmax + 1);
    for (int i = 0; i < nbands; ++i) olive[geo[i].order] = std::min(olive[geo[i].order], live[i]);
    // by start degree within each order
    std::vector<int> by(nbands);
    for (int i = 0; i < nbands; ++i) by[i] = i;
    double total = 0.0;
    for (int m = 0; m <= M; ++m)
        std::stable_sort(by.begin() + orders[m].band0, by.begin() + orders[m + 1].band0,
                         [&](int u, int v) { return bs[u] < bs[v]; });
    for (int i = 0; i < nbands; ++i) total += lmax + 1 - bs[i];

    int G = 1;
    while (G < psht::kAdjMaxWaves && 64 * psht::kAdjMaxBands * G < nrmax) G *= 2;
    int group_max = psht::kAdjMaxBands * G;  // bands per item
    if (const char *v = getenv("PSHT_ADJ_GROUP"))  // tests and tuning runs: smaller groups (in rings)
        if (atoi(v) >= 1) group_max = std::min(group_max, std::max(1, atoi(v) / 64));
    const int rmax = (std::min((nrmax + 63) / 64, group_max) + G - 1) / G;
    const double slots = (double)std::max(ncu, 1) * 4 * 2;
    int S = 64;
    while (S * 2 <= lmax + 1 && (double)(S * 2) * rmax <= total / slots / 3.0) S *= 2;
    if (const char *v = getenv("PSHT_ADJ_SEG")) {  // tuning runs: a power of two, at least 64
        const int x = atoi(v);
        if (x >= 64 && x <= 1 << 15 && (x & (x - 1)) == 0) S = x;
    }
    p.syn_seg = synth_segment_length(g, ncu, first, last);
    if (p.syn_seg > 0) S = std::min(S, p.syn_seg);

    // stored states; one that leaves the double range although it matters before
    // the next (seen at spins in the hundreds only, in the weaker sign) shortens the
    // segments of the adjoint, whose items run from state to state, to 64 degrees,
    // in which no value grows from 2^-960 to 2^-64.  The items of the synthesis run
    // on over several states: where one that leaves the range matters at any later
    // degree, they reload at every state (syn_reload)
    std::vector<psht::LegBand> bands(nbands);
    if (!dalloc(p, p.d_bands, nbands)) return nomem("Legendre bands");
    for (;;) {
        int64_t blk = 0;
        for (int i = 0; i < nbands; ++i) {
            bands[i] = geo[by[i]];
            const int l0 = std::max(bands[i].order, s), at = bs[by[i]];
            bands[i].bs = at;
            bands[i].blk = (int32_t)blk;
            blk += 1 + (lmax - l0) / S - (at - l0) / S;
        }
        p.adj_seg = S;
        p.n_adj_states = blk * 64;
        const size_t held = p.allocations.size(), resident = p.resident;
        if (!dalloc(p, p.d_st_p, (size_t)blk * 128) || (s > 0 && !dalloc(p, p.d_st_m, (size_t)blk * 128)))
            return nomem("Legendre recurrence states");
        int32_t lost[2] = {0, 0};
        if (nbands > 0) {
            e = hipMemcpy(p.d_bands, bands.data(), sizeof(bands[0]) * nbands, hipMemcpyHostToDevice);
            if (e == hipSuccess) e = psht::launch_fill_zero(d_lost.p, sizeof(lost), st);
            if (e == hipSuccess)
                e = psht::launch_leg_states(p, nbands, static_cast<int32_t *>(d_lost.p), st);
            if (e == hipSuccess) e = hipMemcpyAsync(lost, d_lost.p, sizeof(lost), hipMemcpyDeviceToHost, st);
            if (e == hipSuccess) e = hipStreamSynchronize(st);
            if (e != hipSuccess) return device(e, "Legendre recurrence states");
        }
        p.syn_reload = lost[1] > 0;
        if (lost[0] == 0) break;
        if (S == 64) {
            err = {PSHT_ERR_UNSUPPORTED, "Legendre recurrence leaves the double range within 64 degrees"};
            return false;
        }
        while (p.allocations.size() > held) {
            (void)hipFree(p.allocations.back());
            p.allocations.pop_back();
        }
        p.resident = resident;
        S = 64;
    }

    // adjoint items
    std::vector<psht::AdjItem> items;
    std::vector<double> cost;
    bool accumulate = false;
    int rused = 1;
    for (int m = 0; m <= M; ++m) {
        const int l0 = std::max(m, s), b0 = orders[m].band0, nb = orders[m + 1].band0 - b0;
        if (nb == 0) {
            if (m <= lmax) items.push_back(psht::AdjItem{m, m, lmax + 1, 0, 0, 1, 0, 0, 0}), cost.push_back(0.0);
            continue;
        }
        accumulate |= nb > group_max;
        for (int k = 0; l0 + k * S <= lmax; ++k) {
            const int la = l0 + k * S, lb = std::min(lmax + 1, la + S);
            int on = 0;
            while (on < nb && bands[b0 + on].bs < lb) ++on;
            for (int q = 0; q < std::max(on, 1); q += group_max) {
                const int n = std::min(group_max, on - q);
                const int waves = n <= psht::kAdjMaxBands ? 1 : G;
                double c = 0.0;  // per wave: band steps, and the reduction's share of every step
                for (int i = 0; i < n; ++i) c += lb - std::max(la, bands[b0 + q + i].bs);
                c /= waves;
                if (n > 0) c += 1.6 * (lb - std::max(la, bands[b0 + q].bs));
                items.push_back(psht::AdjItem{m, k == 0 ? m : la, lb, b0 + q, n, waves, olive[m],
                                              q == 0 ? bands[b0].bs : 0, last[m]});
                cost.push_back(c);
                rused = std::max(rused, (n + waves - 1) / waves);
            }
        }
    }
    // orders above mmax have no ring: their outputs are zero
    std::vector<psht::AdjItem> zeros;
    if (!accumulate)
        for (int m = M + 1; m <= lmax; ++m) zeros.push_back(psht::AdjItem{m, m, lmax + 1, 0, 0, 1, 0, 0, 0});
    // longest first (blocks are issued in order and dealt round-robin to the XCDs)
    auto longest_first = [](auto &list, const std::vector<double> &c) {
        std::vector<int> at(list.size());
        for (size_t i = 0; i < at.size(); ++i) at[i] = (int)i;
        std::stable_sort(at.begin(), at.end(), [&](int u, int v) { return c[u] > c[v]; });
        auto out = list;
        for (size_t i = 0; i < at.size(); ++i) out[i] = list[at[i]];
        list.swap(out);
    };
    longest_first(items, cost);
    {
        // one entry per wave: single-wave items fill workgroups of G with their neighbours
        // in cost; the zeros are spread evenly among them, so that their stores run
        // beside the sums (as fills of their own they took 40 of 221 us at lmax
        // 4000 on a 7-degree disc)
        std::vector<psht::AdjItem> waves, group, zgroup;
        size_t iz = 0, n = 0;
        auto put = [&](std::vector<psht::AdjItem> &g, const psht::AdjItem &it) {
            g.push_back(it);
            if ((int)g.size() < G) return;
            waves.insert(waves.end(), g.begin(), g.end());
            g.clear();
        };
        for (const psht::AdjItem &it : items) {
            ++n;
            while (iz * items.size() < n * zeros.size()) put(zgroup, zeros[iz++]);
            for (int w = 0; w < (it.waves > 1 ? G : 0); ++w) waves.push_back(it);
            if (it.waves == 1) put(group, it);
        }
        for (auto *g : {&group, &zgroup})
            while (!g->empty()) put(*g, psht::AdjItem{0, 0, 0, 0, 0, 1, 0, 0, 0});
        items.swap(waves);
    }
    p.adj_waves = G;
    p.adj_rmax = rused;
    p.adj_accumulate = accumulate;
    p.n_adj_items = (int)items.size();
    if (!upload(p, p.d_adj_items, items, st)) return nomem("uploading the adjoint work list");

    // synthesis items: seg degrees per segment (0: one segment), R bands per wave
    auto synth_items = [&](int seg, int R, int x, std::vector<psht::SynthItem> &list, std::vector<double> &c) {
        for (int m = x < 0 ? 0 : x; m <= M; m += x < 0 ? 1 : 8) {
            const int l0 = std::max(m, s), b0 = orders[m].band0, nb = orders[m + 1].band0 - b0;
            const int len = seg > 0 ? seg : lmax + 1;
            const size_t at = list.size();
            for (int q = 0; q < nb; q += R)
                for (int k = 0; l0 + k * len <= lmax; ++k) {
                    const int la = l0 + k * len, lb = std::min(lmax + 1, la + len);
                    int n = 0;
                    double w = 0.0;
                    while (n < std::min(R, nb - q) && bands[b0 + q + n].bs < lb)
                        w += lb - std::max(la, bands[b0 + q + n++].bs);
                    if (n == 0) continue;
                    list.push_back(psht::SynthItem{m, la, lb, b0 + q, n, k, 0, 0});
                    c.push_back(w + 0.3 * (lb - std::max(la, bands[b0 + q].bs)));
                }
            if (list.size() == at) continue;
            const size_t least = std::min_element(c.begin() + at, c.end()) - c.begin();
            list[least].live = olive[m];
            list[least].start = bands[b0].bs;
            c[least] += 0.2 * (bands[b0].bs - olive[m]);
        }
    };
    const int rmax_synth = p.syn_reload ? psht::kSynthReloadBands : 4;
    const int fixed = std::min(rmax_synth, psht::leg_bands_per_wave());  // 0: not fixed
    // segmented lists: syn_seg degrees; and for calls of several maps, which fill
    // the GPU with fewer items, four times as many (fewer copies of F to add) with two
    // bands per wave.  us of the stage, spin 2, 8 maps, the list of single maps / 1, 2, 4,
    // 8 times its segments: 5-degree disc at lmax 2048 174 / 151, 121, 118, 139; 10 degrees
    // 298 / 279, 252, 248, 275; 3 degrees at lmax 4096 346 / 289, 262, 268, 289; 18 degrees
    // at lmax 3000 1193 / 1128, 1089, 1083, 1132.  Short transforms and few maps would
    // want fewer (5 degrees at lmax 1024, 8 maps 54 / 49, 48, 61, 94; 3 maps 33 / 30, 36, 49,
    // 81; 3 degrees at lmax 512, 3 maps 16 / 19, 22, 32, 51).
    p.syn_parts = 0;
    if (p.syn_seg > 0) {
        p.syn_r = fixed ? fixed : rmax_synth;
        // copies for every segment of the longest order
        p.syn_parts = (lmax + 1 - s + p.syn_seg - 1) / p.syn_seg - 1;
        p.multi_seg = 4 * p.syn_seg < lmax + 1 - s ? 4 * p.syn_seg : 0;
        p.multi_r = fixed ? fixed : 2;
        auto list = [&](int seg, int R, psht::SynthItem *&d, int &n) {
            std::vector<psht::SynthItem> syn;
            std::vector<double> c;
            synth_items(seg, R, -1, syn, c);
            longest_first(syn, c);
            n = (int)syn.size();
            return upload(p, d, syn, st);
        };
        if (!list(p.syn_seg, p.syn_r, p.d_syn_items, p.n_syn_items) ||
            (p.multi_seg > 0 && !list(p.multi_seg, p.multi_r, p.d_multi_items, p.n_multi_items)))
            return nomem("uploading the synthesis work list");
    }
    // plain list: the items of an order on one XCD (blocks are dealt round-robin
    // to the eight), so that they share its L2, each XCD's longest first
    p.leg_r = fixed ? fixed : (nbands >= 10 * slots ? rmax_synth : nbands >= slots ? 2 : 1);
    std::vector<psht::SynthItem> per[8], plain;
    size_t most = 0;
    for (int x = 0; x < 8; ++x) {
        std::vector<double> c;
        synth_items(0, p.leg_r, x, per[x], c);
        longest_first(per[x], c);
        most = std::max(most, per[x].size());
    }
    for (size_t i = 0; i < most; ++i)
        for (int x = 0; x < 8; ++x)
            plain.push_back(i < per[x].size() ? per[x][i] : psht::SynthItem{0, 0, 0, 0, 0, 0, 0, 0});
    p.n_leg_items = (int)plain.size();
    if (!upload(p, p.d_leg_items, plain, st)) return nomem("uploading the synthesis work list");
    return true;
}

psht_status plan_create_impl(psht_plan *out, int lmax, int spin, int64_t npoints, const double *theta,
                             const double *phi, double epsilon, int precision, const psht_plan_options *opts,
                             hipStream_t st) {
    if (!out) return fail(PSHT_ERR_ARG, "out is NULL");
    *out = nullptr;
    if (lmax < 0 || spin < 0 || spin > lmax) return fail(PSHT_ERR_ARG, "need lmax >= 0 and 0 <= spin <= lmax");
    if (lmax > 16384) return fail(PSHT_ERR_UNSUPPORTED, "lmax above 16384");
    if (!(epsilon >= 1e-14 && epsilon <= 1e-2)) return fail(PSHT_ERR_ARG, "epsilon must lie in [1e-14, 1e-2]");
    if (precision < PSHT_PREC_AUTO || precision > PSHT_PREC_FP64) return fail(PSHT_ERR_ARG, "unknown precision");
    // the slot layout of the sorted points (at most two entries per point) is indexed in int32
    if (npoints < 0 || npoints >= (int64_t(1) << 30)) return fail(PSHT_ERR_ARG, "npoints must lie in [0, 2^30)");
    if (npoints > 0 && (!theta || !phi)) return fail(PSHT_ERR_ARG, "theta/phi are NULL");

    // theta range and validity (one device-to-host synchronisation)
    double tmin = 0.0, tmax = 0.0;
    if (npoints > 0) {
        ScopedDevFree stats;
        hipError_t e = hipMalloc(&stats.p, sizeof(double) * 3 * 1024);
        if (e != hipSuccess) return device_fail(e, "allocating point statistics");
        e = psht::launch_point_stats(theta, phi, npoints, static_cast<double *>(stats.p), st);
        if (e != hipSuccess) return device_fail(e, "point statistics kernel");
        std::vector<double> h(3 * 1024);
        e = hipMemcpyAsync(h.data(), stats.p, h.size() * sizeof(double), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return device_fail(e, "reading point statistics");
        double mn = 1e300, mx = -1e300, bad = 0;
        for (int b = 0; b < 1024; ++b) {
            mn = std::min(mn, h[3 * b]);
            mx = std::max(mx, h[3 * b + 1]);
            bad += h[3 * b + 2];
        }
        if (bad > 0)
            return fail(PSHT_ERR_ARG, "some theta outside [0, pi] or phi not finite (" +
                                          std::to_string((long long)bad) + " points)");
        tmin = mn;
        tmax = mx;
    }

    std::unique_ptr<psht_plan_s, void (*)(psht_plan_s *)> plan(new psht_plan_s(), free_plan);
    psht_plan_s &p = *plan;
    p.npts = npoints;
    psht::Error err;
    if (!psht::geometry_compute(p.g, lmax, spin, tmax, tmin, epsilon, precision, true, err, true, opts))
        return fail(err);
    const psht::Geometry &g = p.g;
    const bool fp32 = g.fp32;
    const int fmax = fp32 ? psht::kFftMaxLds32 : psht::kFftMaxLds64;
    // The Theta grid (NT = 2 N2 points) above the LDS limit runs as two N2-point
    // transforms (even and odd rows); N2 itself must fit.
    if (g.N2 > fmax)
        return fail(PSHT_ERR_UNSUPPORTED, "Theta circle of " + std::to_string(g.N2) + " samples exceeds the LDS FFT limit");
    p.theta_split = g.Ntheta > fmax;
    if (const char *e = getenv("PSHT_THETA_SPLIT"))  // tests and tuning runs: 1 forces the split where possible
        if (atoi(e) == 1 && g.Ntheta == 2 * g.N2) p.theta_split = true;
    if (p.theta_split && g.Ntheta != 2 * g.N2)
        return fail(PSHT_ERR_UNSUPPORTED, "Theta grid above the LDS limit that is not twice the circle");
    // phi rows run as g.phi_parts transforms of Nphi / phi_parts points (see params.cpp)
    if (g.Nphi / g.phi_parts > fmax)
        return fail(PSHT_ERR_UNSUPPORTED, "phi grid of " + std::to_string(g.Nphi) + " exceeds the LDS FFT limit");

    p.leg = psht::leg_table_get(lmax, spin, err);
    if (!p.leg) return fail(err);

    // rings
    std::vector<double> ry(g.nring), rch(g.nring), rsh(g.nring);
    for (int j = 0; j < g.nring; ++j) {
        long double t = g.ring_theta[j], sh = sinl(t / 2);
        ry[j] = (double)(2 * sh * sh);
        rch[j] = (double)cosl(t / 2);
        rsh[j] = (double)sh;
    }
    if (!upload(p, p.d_ring_y, ry, st) || !upload(p, p.d_ring_ch, rch, st) || !upload(p, p.d_ring_sh, rsh, st) ||
        !upload(p, p.d_ring_w, g.ring_w, st) || !upload(p, p.d_ring_mmax, g.ring_mmax, st))
        return fail(PSHT_ERR_NOMEM, "uploading ring tables");

    // Legendre bands, states and work lists
    {
        int dev = 0, ncu = 0;
        (void)hipGetDevice(&dev);
        (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
        psht::Error e2;
        if (!build_legendre(p, ncu, st, e2)) return fail(e2);
    }

    // NUFFT tables (the kernel transforms as the factors the stages multiply by)
    std::vector<double> scale_t(g.psihat_theta), scale_p(g.psihat_phi);
    for (double &x : scale_t) x = 1.0 / (g.N2 * x);
    for (double &x : scale_p) x = 1.0 / x;
    if (!upload(p, p.d_scale_t, scale_t, st) || !upload(p, p.d_scale_p, scale_p, st) ||
        (!g.es_poly.empty() && !upload(p, p.d_es_poly, g.es_poly, st)) ||
        (!g.es_poly32.empty() && !upload(p, p.d_es_poly32, g.es_poly32, st)))
        return fail(PSHT_ERR_NOMEM, "uploading kernel tables");
    if (!make_fft_table(p, p.fft_n2, g.N2, g.fp32, st) || !make_fft_table(p, p.fft_nt, g.Ntheta, g.fp32, st) ||
        !make_fft_table(p, p.fft_np, g.Nphi, g.fp32, st))
        return fail(PSHT_ERR_NOMEM, "FFT tables");
    if (g.phi_parts > 1 && !make_fft_table(p, p.fft_np_part, g.Nphi / g.phi_parts, g.fp32, st))
        return fail(PSHT_ERR_NOMEM, "FFT tables");

    // points: bucket sort into tiles (PSHT_TILE="<rows>x<cols>" overrides the shape
    // for tuning runs).  A point on a cell near tile borders adds into it from more
    // tiles where they are smaller, in an FP32 plan's float grid: its adjoint's error
    // does not show it (against the FP64 plan of the same grid, mean of 8 runs, default /
    // 16 x 32 tiles: 2-degree disc at lmax 512 2.34e-7 / 2.37e-7, 5-degree disc at lmax
    // 1024 1.842e-7 / 1.838e-7, 20-degree cap at lmax 300 2.71e-7 / 2.69e-7).
    psht::tile_shape(g.rows_used, g.Nphi, g.W, npoints, p.tile_x, p.tile_y);
    if (const char *ts = getenv("PSHT_TILE")) {
        int tx = 0, ty = 0;
        if (sscanf(ts, "%dx%d", &tx, &ty) == 2 && tx >= 4 && ty >= 8 && tx <= 64 && ty <= 128 &&
            (size_t)(tx + g.W - 1) * ((ty + g.W - 1) | 1) * 16 <= 65536) {
            p.tile_x = tx;
            p.tile_y = ty;
        }
    }
    p.ntx = (g.rows_used + p.tile_x - 1) / p.tile_x;
    p.nty = (g.Nphi + p.tile_y - 1) / p.tile_y;
    p.ntiles = p.ntx * p.nty;
    if (!dalloc(p, p.d_tile_start, (size_t)p.ntiles + 1) || !dalloc(p, p.d_dropped, 2))
        return fail(PSHT_ERR_NOMEM, "allocating sorted points");
    if (psht::launch_fill_zero(p.d_dropped, 2 * sizeof(unsigned long long), st) != hipSuccess)
        return fail(PSHT_ERR_DEVICE, "clearing the point counters");
    {
        ScopedDevFree keys, cursor, pstart, tpx, tpy, tperm;
        const size_t nn = (size_t)std::max<int64_t>(npoints, 1);
        hipError_t e = hipMalloc(&keys.p, sizeof(int32_t) * nn);
        if (e == hipSuccess) e = hipMalloc(&cursor.p, sizeof(int32_t) * (size_t)p.ntiles);
        if (e == hipSuccess) e = hipMalloc(&pstart.p, sizeof(int32_t) * ((size_t)p.ntiles + 1));
        if (e == hipSuccess) e = hipMalloc(&tpx.p, sizeof(double) * nn);
        if (e == hipSuccess) e = hipMalloc(&tpy.p, sizeof(double) * nn);
        if (e == hipSuccess) e = hipMalloc(&tperm.p, sizeof(int32_t) * nn);
        if (e != hipSuccess) return device_fail(e, "sort scratch");
        e = psht::launch_point_sort_count(p, theta, phi, static_cast<int32_t *>(keys.p),
                                          static_cast<int32_t *>(cursor.p), static_cast<int32_t *>(pstart.p),
                                          static_cast<double *>(tpx.p), static_cast<double *>(tpy.p),
                                          static_cast<int32_t *>(tperm.p), st);
        int32_t total = 0;
        if (e == hipSuccess)
            e = hipMemcpyAsync(&total, p.d_tile_start + p.ntiles, sizeof(int32_t), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return device_fail(e, "point sort");
        p.n_entries = total;
        const size_t ne = (size_t)std::max<int64_t>(p.n_entries, 1);
        if (!dalloc(p, p.d_px, ne) || !dalloc(p, p.d_py, ne) || !dalloc(p, p.d_perm, ne))
            return fail(PSHT_ERR_NOMEM, "allocating sorted points");
        // p.d_dropped[1] counts sorted entries outside their tile
        e = psht::launch_point_sort_order(p, static_cast<int32_t *>(keys.p), static_cast<const int32_t *>(pstart.p),
                                          static_cast<const double *>(tpx.p), static_cast<const double *>(tpy.p),
                                          static_cast<const int32_t *>(tperm.p), p.d_dropped + 1, st);
        unsigned long long bad = 0;
        if (e == hipSuccess)
            e = hipMemcpyAsync(&bad, p.d_dropped + 1, sizeof(bad), hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return device_fail(e, "point sort");
        if (bad != 0)
            return fail(PSHT_ERR_DEVICE, "internal error: " + std::to_string(bad) +
                                             " sorted points have a stencil outside their NUFFT tile");
    }

    // workspace per map
    const size_t cs = fp32 ? 8 : 16;
    p.ws_F = align256((size_t)(2 * g.mmax + 1) * g.nring * 16);
    p.ws_V = align256((size_t)g.rows_used * (2 * g.mmax + 1) * cs);
    p.ws_U = align256((size_t)g.rows_used * g.Nphi * cs);
    // the synthesis' partial copies of F use the V and U region, which is
    // free until the Legendre stage has added them into F
    p.ws_per_map = p.ws_F + std::max(p.ws_V + p.ws_U, (size_t)p.syn_parts * p.ws_F);
    *out = plan.release();
    return PSHT_OK;
}

// Maps per launch of the stages after the Legendre step (before it, in the
// adjoint): as many as keep their V and U, which one stage writes and the next
// reads, within half of the 256 MB last-level cache.
int maps_per_launch(const psht_plan_s &p, int nmaps) {
    const size_t room = size_t(128) << 20, one = std::max<size_t>(p.ws_V + p.ws_U, 1);
    return (int)std::min<size_t>((size_t)nmaps, std::max<size_t>(1, std::min<size_t>(room / one, 1024)));
}

bool check_ws(const psht_plan_s &p, int nmaps, void *ws, size_t ws_bytes) {
    if (nmaps == 0) return true;
    return ws != nullptr && ws_bytes >= (size_t)nmaps * p.ws_per_map;
}

}  // namespace

psht_status psht::set_error(psht_status code, const char *msg) { return fail(code, msg); }

extern "C" {

psht_status psht_plan_create(psht_plan *out, int lmax, int spin, int64_t npoints, const double *theta,
                             const double *phi, double epsilon, int precision, void *hip_stream) {
    return psht_plan_create_ex(out, lmax, spin, npoints, theta, phi, epsilon, precision, nullptr, hip_stream);
}

psht_status psht_plan_create_ex(psht_plan *out, int lmax, int spin, int64_t npoints, const double *theta,
                                const double *phi, double epsilon, int precision, const psht_plan_options *opts,
                                void *hip_stream) {
    try {
        return plan_create_impl(out, lmax, spin, npoints, theta, phi, epsilon, precision, opts,
                                static_cast<hipStream_t>(hip_stream));
    } catch (const std::bad_alloc &) {
        return fail(PSHT_ERR_NOMEM, "host allocation failed");
    } catch (const std::exception &e) {
        return fail(PSHT_ERR_DEVICE, e.what());
    } catch (...) {
        return fail(PSHT_ERR_DEVICE, "unknown error");
    }
}

psht_status psht_plan_query(psht_plan plan, psht_plan_info *info) {
    if (!plan || !info) return fail(PSHT_ERR_ARG, "plan or info is NULL");
    fill_info(*plan, info);
    return PSHT_OK;
}

}  // extern "C"


// Synthesis of nmaps maps with the given workspace (shared by psht_synth,
// psht_synth_grad and the entry point without allocation).
psht_status psht::synth_run(psht_plan plan, int nmaps, const void *alm, void *map, void *workspace, size_t ws_bytes,
                            double mscale, void *hip_stream) {
    if (!plan) return fail(PSHT_ERR_ARG, "plan is NULL");
    if (nmaps < 0) return fail(PSHT_ERR_ARG, "nmaps < 0");
    if (nmaps > 0 && (!alm || (!map && plan->npts > 0))) return fail(PSHT_ERR_ARG, "alm or map is NULL");
    if (!check_ws(*plan, nmaps, workspace, ws_bytes))
        return fail(PSHT_ERR_WORKSPACE, "workspace smaller than nmaps * workspace_bytes_per_map");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const psht::Geometry &g = plan->g;
    const size_t alm_bytes = (size_t)(g.lmax + 1) * (g.lmax + 2) / 2 * 2 * 16;
    const size_t map_bytes = (size_t)plan->npts * (g.fp32 ? 8 : 16);
    psht_plan_s &P = *plan;
    const int64_t wss = (int64_t)P.ws_per_map;
    char *ws = static_cast<char *>(workspace);
    constexpr int kMost = 1024;  // maps per Legendre launch
    for (int i = 0; i < nmaps;) {
        const int nl = std::min(nmaps - i, kMost), group = maps_per_launch(P, nl);
        hipError_t e = timed(P, PSHT_T_LEG_SYNTH, st, [&] {
            return psht::launch_leg_synth(P, static_cast<const char *>(alm) + i * alm_bytes, ws + i * wss, true,
                                          psht::MapBatch{nl, wss}, mscale, st);
        });
        for (int k = i; k < i + nl && e == hipSuccess; k += group) {
            const psht::MapBatch mb{std::min(group, i + nl - k), wss};
            char *F = ws + k * wss, *V = F + P.ws_F, *U = V + P.ws_V;
            e = timed(P, PSHT_T_THETA_SYNTH, st, [&] { return psht::launch_theta_synth(P, F, V, mb, st); });
            if (e == hipSuccess)
                e = timed(P, PSHT_T_PHI_SYNTH, st, [&] { return psht::launch_phi_synth(P, V, U, mb, st); });
            if (e == hipSuccess)
                e = timed(P, PSHT_T_INTERP, st, [&] {
                    return psht::launch_interp(P, U, static_cast<char *>(map) + k * map_bytes, mb, st);
                });
        }
        if (e != hipSuccess) return device_fail(e, "synthesis launch");
        i += nl;
    }
    return PSHT_OK;
}

namespace {

psht_status adjoint_impl(psht_plan plan, int nmaps, const void *map, void *alm, void *workspace, size_t ws_bytes,
                         double mscale, void *hip_stream) {
    if (!plan) return fail(PSHT_ERR_ARG, "plan is NULL");
    if (nmaps < 0) return fail(PSHT_ERR_ARG, "nmaps < 0");
    if (nmaps > 0 && (!alm || (!map && plan->npts > 0))) return fail(PSHT_ERR_ARG, "alm or map is NULL");
    if (!check_ws(*plan, nmaps, workspace, ws_bytes))
        return fail(PSHT_ERR_WORKSPACE, "workspace smaller than nmaps * workspace_bytes_per_map");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const psht::Geometry &g = plan->g;
    const size_t alm_bytes = (size_t)(g.lmax + 1) * (g.lmax + 2) / 2 * 2 * 16;
    const size_t map_bytes = (size_t)plan->npts * (g.fp32 ? 8 : 16);
    psht_plan_s &P = *plan;
    const int64_t wss = (int64_t)P.ws_per_map;
    const int group = maps_per_launch(P, std::max(nmaps, 1));
    for (int i = 0; i < nmaps; i += group) {
        const psht::MapBatch mb{std::min(group, nmaps - i), wss};
        char *F = static_cast<char *>(workspace) + i * wss, *V = F + P.ws_F, *U = V + P.ws_V;
        const void *m = static_cast<const char *>(map) + i * map_bytes;
        void *a = static_cast<char *>(alm) + i * alm_bytes;
        hipError_t e = timed(P, PSHT_T_GRID_ZERO, st, [&] { return psht::launch_grid_zero(P, U, mb, st); });
        if (e == hipSuccess) e = timed(P, PSHT_T_SPREAD, st, [&] { return psht::launch_spread(P, m, U, mb, st); });
        if (e == hipSuccess)
            e = timed(P, PSHT_T_PHI_ADJ, st, [&] { return psht::launch_phi_adjoint(P, U, V, mb, st); });
        if (e == hipSuccess)
            e = timed(P, PSHT_T_THETA_ADJ, st, [&] { return psht::launch_theta_adjoint(P, V, F, mb, st); });
        if (e == hipSuccess)
            e = timed(P, PSHT_T_LEG_ADJ, st, [&] { return psht::launch_leg_adjoint(P, F, a, mb, mscale, st); });
        if (e != hipSuccess) return device_fail(e, "adjoint launch");
    }
    return PSHT_OK;
}

}  // namespace

extern "C" {

psht_status psht_synth(psht_plan plan, int nmaps, const void *alm, void *map, void *workspace, size_t ws_bytes,
                       void *hip_stream) {
    return psht::synth_run(plan, nmaps, alm, map, workspace, ws_bytes, 1.0, hip_stream);
}

psht_status psht_adjoint(psht_plan plan, int nmaps, const void *map, void *alm, void *workspace, size_t ws_bytes,
                         void *hip_stream) {
    return adjoint_impl(plan, nmaps, map, alm, workspace, ws_bytes, 1.0, hip_stream);
}

psht_status psht_adjoint_grad(psht_plan plan, int nmaps, const void *map_grad, void *alm_grad, void *workspace,
                              size_t ws_bytes, void *hip_stream) {
    return adjoint_impl(plan, nmaps, map_grad, alm_grad, workspace, ws_bytes, 2.0, hip_stream);
}

psht_status psht_synth_grad(psht_plan plan, int nmaps, const void *alm_grad, void *map_grad, void *workspace,
                            size_t ws_bytes, void *hip_stream) {
    return psht::synth_run(plan, nmaps, alm_grad, map_grad, workspace, ws_bytes, 0.5, hip_stream);
}

void psht_plan_destroy(psht_plan plan) { free_plan(plan); }

psht_status psht_plan_set_timing(psht_plan plan, int stages) {
    if (!plan) return fail(PSHT_ERR_ARG, "plan is NULL");
    for (auto &e : plan->pending) {
        (void)hipEventSynchronize(e.second.second);
        plan->event_pool.push_back(e.second.first);
        plan->event_pool.push_back(e.second.second);
    }
    plan->pending.clear();
    for (int i = 0; i < PSHT_T_COUNT; ++i) {
        plan->t_ms[i] = 0;
        plan->t_launches[i] = 0;
    }
    plan->timing = (unsigned)stages & (unsigned)PSHT_T_ALL;
    // events for 32 calls ahead: none is created while timed work is issued
    const int want = 64 * __builtin_popcount(plan->timing);
    while ((int)plan->event_pool.size() < want) {
        hipEvent_t e = nullptr;
        if (hipEventCreate(&e) != hipSuccess) return fail(PSHT_ERR_DEVICE, "creating timing events");
        plan->event_pool.push_back(e);
    }
    return PSHT_OK;
}

psht_status psht_plan_timing(psht_plan plan, double *ms, int64_t *launches) {
    if (!plan || !ms || !launches) return fail(PSHT_ERR_ARG, "NULL argument");
    for (auto &e : plan->pending) {
        hipError_t r = hipEventSynchronize(e.second.second);
        float t = 0.f;
        if (r == hipSuccess) r = hipEventElapsedTime(&t, e.second.first, e.second.second);
        if (r != hipSuccess) return device_fail(r, "timing events");
        plan->t_ms[e.first] += t;
        plan->t_launches[e.first] += 1;
        plan->event_pool.push_back(e.second.first);
        plan->event_pool.push_back(e.second.second);
    }
    plan->pending.clear();
    for (int i = 0; i < PSHT_T_COUNT; ++i) {
        ms[i] = plan->t_ms[i];
        launches[i] = plan->t_launches[i];
    }
    return PSHT_OK;
}

const char *psht_last_error(void) { return g_last_error.c_str(); }

psht_status psht_rotate_alm_workspace(int lmax, int ncomp, size_t *bytes) {
    if (lmax < 0 || lmax > 16383 || (ncomp != 1 && ncomp != 2) || !bytes)
        return fail(PSHT_ERR_ARG, "need 0 <= lmax <= 16383, ncomp 1 or 2, bytes not NULL");
    *bytes = (size_t)ncomp * (size_t)(lmax + 1) * (size_t)(2 * lmax + 1) * 16;
    return PSHT_OK;
}

psht_status psht_rotate_alm(int lmax, int ncomp, double alpha, double beta, double gamma, const void *alm_in,
                            void *alm_out, void *workspace, size_t ws_bytes, void *hip_stream) {
    size_t need = 0;
    if (psht_rotate_alm_workspace(lmax, ncomp, &need) != PSHT_OK) return PSHT_ERR_ARG;
    if (!std::isfinite(alpha) || !std::isfinite(beta) || !std::isfinite(gamma))
        return fail(PSHT_ERR_ARG, "rotation angles must be finite");
    if (!alm_in || !alm_out || !workspace) return fail(PSHT_ERR_ARG, "NULL array");
    const size_t bytes = (size_t)ncomp * (size_t)(lmax + 1) * (size_t)(lmax + 2) / 2 * 16;
    const char *a = (const char *)alm_in, *b = (const char *)alm_out;
    if (a < b + bytes && b < a + bytes) return fail(PSHT_ERR_ARG, "alm_in and alm_out overlap");
    if (ws_bytes < need) return fail(PSHT_ERR_WORKSPACE, "workspace smaller than psht_rotate_alm_workspace");
    // log2(n!) for n = 0..2 lmax, then W(n) for n = 0..lmax (rot_factor.h), per
    // (device, lmax), kept for the process lifetime
    static std::mutex mu;
    static std::map<std::pair<int, int>, double2 *> tables;
    double2 *lf = nullptr;
    {
        std::lock_guard<std::mutex> lock(mu);
        int dev = 0;
        (void)hipGetDevice(&dev);
        auto key = std::make_pair(dev, lmax);
        auto it = tables.find(key);
        if (it != tables.end()) {
            lf = it->second;
        } else try {
            std::vector<double2> h(2 * (size_t)lmax + 1);
            for (size_t n = 0; n < h.size(); ++n) {
                const long double v = lgammal((long double)n + 1) / logl(2.0L);
                h[n].x = (double)v;
                h[n].y = (double)(v - (long double)h[n].x);
            }
            std::vector<double2> w;
            psht::rot_w_table(lmax, w);
            h.insert(h.end(), w.begin(), w.end());
            void *d = nullptr;
            hipError_t e = hipMalloc(&d, h.size() * sizeof(double2));
            if (e != hipSuccess) return device_fail(e, "rotation tables");
            e = hipMemcpy(d, h.data(), h.size() * sizeof(double2), hipMemcpyHostToDevice);
            if (e != hipSuccess) {
                (void)hipFree(d);
                return device_fail(e, "rotation tables");
            }
            tables[key] = (double2 *)d;
            lf = (double2 *)d;
        } catch (const std::bad_alloc &) {
            return fail(PSHT_ERR_NOMEM, "host allocation failed");
        }
    }
    hipError_t e = psht::launch_rotate_alm(lmax, ncomp, alpha, beta, gamma, alm_in, alm_out, workspace, lf,
                                           lf + 2 * (size_t)lmax + 1, static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? PSHT_OK : device_fail(e, "rotation kernels");
}

psht_status psht_rotate_points(int64_t npoints, double alpha, double beta, double gamma, const double *theta,
                               const double *phi, double *theta_out, double *phi_out, double *psi_out,
                               void *hip_stream) {
    if (npoints < 0) return fail(PSHT_ERR_ARG, "npoints < 0");
    if (!std::isfinite(alpha) || !std::isfinite(beta) || !std::isfinite(gamma))
        return fail(PSHT_ERR_ARG, "rotation angles must be finite");
    if (npoints > 0 && (!theta || !phi || !theta_out || !phi_out || !psi_out))
        return fail(PSHT_ERR_ARG, "NULL array");
    psht::RotMatrix R;
    const double ca = std::cos(alpha), sa = std::sin(alpha), cb = std::cos(beta), sb = std::sin(beta),
                 cg = std::cos(gamma), sg = std::sin(gamma);
    // Rz(alpha) Ry(beta) Rz(gamma)
    const double Y[3][3] = {{cb * cg, -cb * sg, sb}, {sg, cg, 0.0}, {-sb * cg, sb * sg, cb}};
    for (int c = 0; c < 3; ++c) {
        R.r[0][c] = ca * Y[0][c] - sa * Y[1][c];
        R.r[1][c] = sa * Y[0][c] + ca * Y[1][c];
        R.r[2][c] = Y[2][c];
    }
    hipError_t e = psht::launch_rotate_points(npoints, R, theta, phi, theta_out, phi_out, psi_out,
                                              static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? PSHT_OK : device_fail(e, "point rotation kernel");
}

psht_status psht_spin_phase(int64_t npoints, int spin, int sign, int fp32, const double *psi, void *map,
                            void *hip_stream) {
    if (npoints < 0 || (sign != 1 && sign != -1) || (fp32 != 0 && fp32 != 1))
        return fail(PSHT_ERR_ARG, "need npoints >= 0, sign +-1, fp32 0 or 1");
    if (npoints > 0 && (!psi || !map)) return fail(PSHT_ERR_ARG, "NULL array");
    hipError_t e = psht::launch_spin_phase(npoints, (double)sign * spin, fp32, psi, map,
                                           static_cast<hipStream_t>(hip_stream));
    return e == hipSuccess ? PSHT_OK : device_fail(e, "spin phase kernel");
}

psht_status psht_great_circle_spectrum(int lmax, int spin, const double *cl, double *cm) {
    if (lmax < 0 || spin < 0 || spin > lmax || !cl || !cm) return fail(PSHT_ERR_ARG, "bad arguments");
    try {
        std::vector<double> v;
        psht::great_circle_spectrum(lmax, spin, cl, v);
        std::copy(v.begin(), v.end(), cm);
        return PSHT_OK;
    } catch (...) {
        return fail(PSHT_ERR_NOMEM, "host allocation failed");
    }
}

psht_status psht_plan_check(psht_plan plan, int64_t *dropped, void *hip_stream) {
    if (!plan || !dropped) return fail(PSHT_ERR_ARG, "plan or dropped is NULL");
    *dropped = 0;
    if (!plan->d_dropped) return PSHT_OK;
    unsigned long long v = 0;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    hipError_t e = hipMemcpyAsync(&v, plan->d_dropped, sizeof(v), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return device_fail(e, "reading the point counter");
    *dropped = (int64_t)v;
    return PSHT_OK;
}

psht_status psht_plan_geometry(int lmax, int spin, double theta_star, double epsilon, int precision,
                               psht_plan_info *info, double *ring_theta, double *ring_weight, int32_t *ring_mmax,
                               int capacity) {
    return psht_plan_geometry_ex(lmax, spin, theta_star, epsilon, precision, nullptr, info, ring_theta, ring_weight,
                                 ring_mmax, capacity);
}

psht_status psht_plan_geometry_ex(int lmax, int spin, double theta_star, double epsilon, int precision,
                                  const psht_plan_options *opts, psht_plan_info *info, double *ring_theta,
                                  double *ring_weight, int32_t *ring_mmax, int capacity) {
    try {
        if (!info) return fail(PSHT_ERR_ARG, "info is NULL");
        if (capacity < 0 || (capacity > 0 && (!ring_theta || !ring_weight || !ring_mmax)))
            return fail(PSHT_ERR_ARG, "ring arrays are NULL");
        psht_plan_s p;
        psht::Error err;
        if (!psht::geometry_compute(p.g, lmax, spin, theta_star, 0.0, epsilon, precision, false, err, capacity > 0,
                                    opts))
            return fail(err);
        fill_info(p, info);
        info->workspace_bytes_per_map = 0;
        info->resident_bytes = 0;
        int n = std::min(capacity, p.g.nring);
        for (int j = 0; j < n; ++j) {
            ring_theta[j] = p.g.ring_theta[j];
            ring_weight[j] = p.g.ring_w[j];
            ring_mmax[j] = p.g.ring_mmax[j];
        }
        return PSHT_OK;
    } catch (const std::bad_alloc &) {
        return fail(PSHT_ERR_NOMEM, "host allocation failed");
    } catch (...) {
        return fail(PSHT_ERR_DEVICE, "unknown error");
    }
}

psht_status psht_stage_ex(psht_plan plan, int stage, const void *in, void *out, void *workspace, size_t ws_bytes,
                          void *hip_stream) {
    if (stage == PSHT_STAGE_LEGENDRE_SYNTH && workspace != nullptr && plan != nullptr && plan->syn_seg > 0) {
        // with a workspace: the work list synth_run uses (degree segments with
        // partial copies of F in the workspace)
        if (!in || !out) return fail(PSHT_ERR_ARG, "in or out is NULL");
        if (!check_ws(*plan, 1, workspace, ws_bytes))
            return fail(PSHT_ERR_WORKSPACE, "workspace smaller than workspace_bytes_per_map");
        hipStream_t st = static_cast<hipStream_t>(hip_stream);
        const psht::Geometry &g = plan->g;
        hipError_t e = hipSuccess;
        // F and its partial copies lie in the workspace; F then goes to the output
        char *F = static_cast<char *>(workspace);
        if (e == hipSuccess) e = psht::launch_fill_zero(F, plan->ws_F, st);
        if (e == hipSuccess) e = psht::launch_leg_synth(*plan, in, F, true, psht::MapBatch(), 1.0, st);
        if (e == hipSuccess)
            e = hipMemcpyAsync(out, F, (size_t)(2 * g.mmax + 1) * g.nring * 16, hipMemcpyDeviceToDevice, st);
        if (e != hipSuccess) return device_fail(e, "stage launch");
        return PSHT_OK;
    }
    if (stage == PSHT_STAGE_LEGENDRE_SYNTH || stage == PSHT_STAGE_LEGENDRE_ADJOINT)
        return psht_stage(plan, stage, in, out, hip_stream);
    if (stage != PSHT_STAGE_FOURIER_SYNTH && stage != PSHT_STAGE_FOURIER_ADJOINT)
        return fail(PSHT_ERR_ARG, "unknown stage");
    if (!plan || !in || !out) return fail(PSHT_ERR_ARG, "plan, in or out is NULL");
    if (!check_ws(*plan, 1, workspace, ws_bytes))
        return fail(PSHT_ERR_WORKSPACE, "workspace smaller than workspace_bytes_per_map");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    psht_plan_s &P = *plan;
    char *ws = static_cast<char *>(workspace);
    void *V = ws + P.ws_F;
    void *U = ws + P.ws_F + P.ws_V;
    hipError_t e;
    if (stage == PSHT_STAGE_FOURIER_SYNTH) {
        e = psht::launch_theta_synth(P, in, V, psht::MapBatch(), st);
        if (e == hipSuccess) e = psht::launch_phi_synth(P, V, U, psht::MapBatch(), st);
        if (e == hipSuccess) e = psht::launch_interp(P, U, out, psht::MapBatch(), st);
    } else {
        e = psht::launch_grid_zero(P, U, psht::MapBatch(), st);
        if (e == hipSuccess) e = psht::launch_spread(P, in, U, psht::MapBatch(), st);
        if (e == hipSuccess) e = psht::launch_phi_adjoint(P, U, V, psht::MapBatch(), st);
        if (e == hipSuccess) e = psht::launch_theta_adjoint(P, V, out, psht::MapBatch(), st);
    }
    if (e != hipSuccess) return device_fail(e, "stage launch");
    return PSHT_OK;
}

psht_status psht_stage(psht_plan plan, int stage, const void *in, void *out, void *hip_stream) {
    if (!plan || !in || !out) return fail(PSHT_ERR_ARG, "plan, in or out is NULL");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const psht::Geometry &g = plan->g;
    hipError_t e;
    if (stage == PSHT_STAGE_LEGENDRE_SYNTH) {
        e = psht::launch_fill_zero(out, (size_t)(2 * g.mmax + 1) * g.nring * 16, st);
        if (e == hipSuccess) e = psht::launch_leg_synth(*plan, in, out, false, psht::MapBatch(), 1.0, st);
    } else if (stage == PSHT_STAGE_LEGENDRE_ADJOINT) {
        e = psht::launch_fill_zero(out, (size_t)(g.lmax + 1) * (g.lmax + 2) / 2 * 2 * 16, st);
        if (e == hipSuccess) e = psht::launch_leg_adjoint(*plan, in, out, psht::MapBatch(), 1.0, st);
    } else {
        return fail(PSHT_ERR_ARG, "unknown stage");
    }
    if (e != hipSuccess) return device_fail(e, "stage launch");
    return PSHT_OK;
}

psht_status psht_fft(int n, int batch, int sign, int fp32, const void *in, void *out, void *hip_stream) {
    static std::mutex mu;
    static std::map<std::tuple<int, int, bool>, psht_plan_s *> tables;  // kept for the process lifetime
    if (n < 1 || batch < 0 || (sign != 1 && sign != -1)) return fail(PSHT_ERR_ARG, "bad n, batch or sign");
    if (batch > 0 && (!in || !out)) return fail(PSHT_ERR_ARG, "in or out is NULL");
    if (n > (fp32 ? psht::kFftMaxLds32 : psht::kFftMaxLds64)) return fail(PSHT_ERR_UNSUPPORTED, "n above the LDS limit");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    psht_plan_s *holder;
    {
        std::lock_guard<std::mutex> lock(mu);
        int dev = 0;
        (void)hipGetDevice(&dev);
        auto key = std::make_tuple(n, dev, fp32 != 0);
        auto it = tables.find(key);
        if (it == tables.end()) {
            // only here: the search for few passes is host work (3.9 us at n = 9360, in calls of 0.5 us)
            psht::FftFactors f;
            if (!psht::fft_factor(n, fp32 != 0, f))
                return fail(PSHT_ERR_UNSUPPORTED, "n has a prime factor outside 2,3,5,7,11,13");
            holder = new psht_plan_s();
            if (!make_fft_table(*holder, holder->fft_np, n, fp32 != 0, st) || hipStreamSynchronize(st) != hipSuccess) {
                free_plan(holder);
                return fail(PSHT_ERR_NOMEM, "FFT table");
            }
            tables[key] = holder;
        } else {
            holder = it->second;
        }
    }
    hipError_t e = psht::launch_fft_rows(holder->fft_np, batch, sign, fp32 != 0, in, out, st);
    if (e != hipSuccess) return device_fail(e, "fft launch");
    return PSHT_OK;
}

// Host evaluation of lambda+-_lm(theta), l = 0..lmax, with the tables, seeds,
// recurrence and rescaling the GPU kernels use (values still scaled below the
// double range are reported as zero).
psht_status psht_legendre_column(int lmax, int spin, int m, double theta, double *lam_plus, double *lam_minus) {
    if (lmax < 0 || spin < 0 || spin > lmax || m < 0 || m > lmax || !lam_plus || !lam_minus)
        return fail(PSHT_ERR_ARG, "bad arguments");
    try {
        psht::LegTable t;
        psht::leg_table_host(t, lmax, spin);
        for (int l = 0; l <= lmax; ++l) lam_plus[l] = lam_minus[l] = 0.0;
        const int l0 = std::max(m, spin);
        double up, um, upp = 0.0, ump = 0.0;
        int kp, km;
        psht::leg_seed(t.h_kmant[m], t.h_kexp[m], m, spin, std::cos(theta / 2), std::sin(theta / 2), up, kp, um, km);
        const int64_t base = (int64_t)m * (2 * lmax + 1 - m) / 2;
        const double sh = std::sin(theta / 2), y = 2 * sh * sh;
        for (int l = l0; l <= lmax; ++l) {
            const double *c = &t.h_coef[4 * (base + l)];
            lam_plus[l] = kp == 0 ? c[3] * up : 0.0;
            lam_minus[l] = km == 0 ? c[3] * um : 0.0;
            if (l < lmax) {
                double np = std::fma(std::fma(c[0], y, c[1]), up, -upp);
                upp = up;
                up = np;
                psht::leg_rescale(up, upp, kp);
                double nm = std::fma(std::fma(c[0], y, c[2]), um, -ump);
                ump = um;
                um = nm;
                psht::leg_rescale(um, ump, km);
            }
        }
        return PSHT_OK;
    } catch (...) {
        return fail(PSHT_ERR_NOMEM, "host allocation failed");
    }
}

}  // extern "C"
