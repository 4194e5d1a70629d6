// fb_split.h -- Hermite steps with two or four lanes a body, for wavefronts
// that are alone on their SIMD.
#pragma once

#include "fb_bpl.h"

#include <type_traits>

namespace fb {
namespace {

// A lone wavefront is bound by its own instructions, an interaction after
// another: 33 each, one evaluation of N - 1 of them after the other.  Here G
// neighbouring lanes, 2 or 4, hold the same body.  Each works out the terms of
// its share of the partners (27 instructions each), and the sums run on in the
// order of bpl_eval: the first lane adds its terms, the next takes the sums
// over (a quad permute) and adds its own, and the last one's go to all.  So
// every bit is that of the other Hermite kernels, for three quarters (G = 2) or
// half to two thirds (4) of the instructions and as many fewer LDS reads.  A
// wavefront holds a G-th of the systems, so it pays while the device has SIMDs
// to spare.  Microseconds a step, one lane a body (fb_unrolled.hip), 2, 4, with
// 0.1 and 1 wavefronts of four lanes a body on a SIMD:
//   n = 5    0.75 0.62 0.60   0.77 0.68 0.72     n = 10   1.50 1.07 0.89   1.52 1.14 1.05
//       6    0.89 0.76 0.69   0.91 0.81 0.82         12   1.86 1.25 0.96   1.89 1.30 1.11
//       8    1.19 0.92 0.76   1.18 0.99 0.90         16   2.38 1.57 1.16   2.42 1.60 1.36
// and with 1 and 2 wavefronts of two lanes a body, one lane against two:
//   n = 5    0.83 0.77   1.08 1.26               n = 10   1.67 1.32   2.00 2.34
//       6    0.98 0.93   1.27 1.58                   12   1.98 1.50   2.21 2.70
//       8    1.30 1.16   1.65 1.93                   16   2.49 1.88   2.93 3.55
// and with adaptive steps and both stop rules, one lane against the kernel
// taken, with 0.1 and 1 wavefronts of two lanes a body (all without HillBound,
// which takes 5 to 15% off either):
//   n = 5    1.47 1.26   1.58 1.52               n = 10   2.61 1.76   2.82 2.29
//       6    1.65 1.41   1.75 1.71                   12   3.19 1.83   3.31 2.54
//       8    2.02 1.50   2.17 2.00                   16   4.22 2.11   4.48 3.25
// hence the lines of bpl_mapping and fused_split.  1000 steps of 1000 x 6 915
// -> 725 us; 24 requests to a server (3..10 bodies) 15.5 -> 10.4 ms.

// quad_perm controls: every lane of a body's G reads the lane before it (the
// first itself), or lane k of them.
template <int G>
constexpr int share_before()
{
    return G == 2 ? 0 | (0 << 2) | (2 << 4) | (2 << 6) : 0 | (0 << 2) | (1 << 4) | (2 << 6);
}
template <int G>
constexpr int share_of(int k)
{
    return G == 2 ? k | (k << 2) | ((2 + k) << 4) | ((2 + k) << 6) : k | (k << 2) | (k << 4) | (k << 6);
}

template <int CTRL>
__device__ __forceinline__ void share_read3(double (&a)[3])
{
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const unsigned long long u = __double_as_longlong(a[c]);
        const int lo = __builtin_amdgcn_mov_dpp((int)(u & 0xffffffffull), CTRL, 0xf, 0xf, true);
        const int hi = __builtin_amdgcn_mov_dpp((int)(u >> 32), CTRL, 0xf, 0xf, true);
        a[c] = __longlong_as_double(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
    }
}

// One partner's terms: a += mr3 r, j += mr3 w.
struct SplitTerm {
    double mr3, r[3], w[3];
};

// (the expressions of bpl_interact_p)
template <bool TS>
__device__ __forceinline__ SplitTerm split_term(const Partner &Pj, const double (&xi)[3],
                                                const double (&vi)[3], double &wmax, double &r2)
{
    SplitTerm t;
    const double2 p0 = Pj.p0, p1 = Pj.p1, p2 = Pj.p2;
    const double rx = p0.x - xi[0], ry = p0.y - xi[1], rz = p1.x - xi[2];
    const double ux = p1.y - vi[0], uy = p2.x - vi[1], uz = p2.y - vi[2];
    r2 = fma(rz, rz, fma(ry, ry, rx * rx));
    const double ru = fma(rz, uz, fma(ry, uy, rx * ux));
    const double ri = rsqrt_nr(r2);
    const double ri2 = ri * ri;
    t.mr3 = Pj.mj * (ri2 * ri);
    const double al = 3.0 * ru * ri2;
    t.r[0] = rx;
    t.r[1] = ry;
    t.r[2] = rz;
    t.w[0] = fma(-al, rx, ux);
    t.w[1] = fma(-al, ry, uy);
    t.w[2] = fma(-al, rz, uz);
    if (TS) {
        const double u2 = fma(uz, uz, fma(uy, uy, ux * ux));
        wmax = fmax(wmax, fma(al, ru, u2) * ri2);
    }
    return t;
}

__device__ __forceinline__ void split_add(const SplitTerm &t, double (&a)[3], double (&jk)[3])
{
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        a[c] = fma(t.mr3, t.r[c], a[c]);
        jk[c] = fma(t.mr3, t.w[c], jk[c]);
    }
}

// Place of a lane: its body's LDS entry, which of the body's lanes it is, and
// its partners' entries and masses.
template <int N, int G>
struct SplitSeat {
    static constexpr int kTerms = (N - 1 + G - 1) / G;            // of every lane but the last
    static constexpr int kLast = (N - 1 + kTerms - 1) / kTerms - 1;   // the lane of the last partner
    int entry, share, idx[kTerms];
    double m[kTerms];
};

// The sums of lanes K.. of a body, in turn (every lane goes through all turns;
// lane k's sums are right after turn k).
template <int N, int G, int K>
__device__ __forceinline__ void split_turns(const SplitTerm (&t)[SplitSeat<N, G>::kTerms],
                                            double (&a)[3], double (&jk)[3])
{
    using Seat = SplitSeat<N, G>;
    constexpr int kAdd = K < Seat::kLast ? Seat::kTerms : N - 1 - Seat::kLast * Seat::kTerms;
#pragma unroll
    for (int k = 0; k < kAdd; ++k)
        split_add(t[k], a, jk);
    if constexpr (K < Seat::kLast) {
        share_read3<share_before<G>()>(a);
        share_read3<share_before<G>()>(jk);
        split_turns<N, G, K + 1>(t, a, jk);
    }
}

// Maximum over the lanes of a body, to all of them.
template <int G>
__device__ __forceinline__ double share_max(double v)
{
    auto other = [&](auto ctrl) {
        double t[3] = {v, v, v};
        share_read3<decltype(ctrl)::value>(t);
        v = fmax(v, t[0]);
    };
    other(std::integral_constant<int, 1 | (0 << 2) | (3 << 4) | (2 << 6)>());
    if constexpr (G == 4)
        other(std::integral_constant<int, 2 | (3 << 2) | (0 << 4) | (1 << 6)>());
    return v;
}

// With TS, also the step rule's quantity w and the stop rules' bound hb over
// this lane's own partners, ic2 their 1 / c^2 (ri2 by the star's lane only).
template <int N, int G, bool TS>
__device__ __forceinline__ void split_eval(BplLds &L, const SplitSeat<N, G> &s,
                                           const double (&xi)[3], const double (&vi)[3],
                                           double (&a)[3], double (&jk)[3], double &w,
                                           const double (&ic2)[SplitSeat<N, G>::kTerms],
                                           HillBound &hb)
{
    using Seat = SplitSeat<N, G>;
    if (s.share == 0) {
        L.xy[s.entry] = make_double2(xi[0], xi[1]);
        L.zvx[s.entry] = make_double2(xi[2], vi[0]);
        L.vyvz[s.entry] = make_double2(vi[1], vi[2]);
    }
    wave_sync();
    Partner p[Seat::kTerms];
#pragma unroll
    for (int k = 0; k < Seat::kTerms; ++k)
        p[k] = Partner{L.xy[s.idx[k]], L.zvx[s.idx[k]], L.vyvz[s.idx[k]], s.m[k]};
    __builtin_amdgcn_sched_barrier(0);
    SplitTerm t[Seat::kTerms];
    hb.least = DBL_MAX;
#pragma unroll
    for (int k = 0; k < Seat::kTerms; ++k) {
        double r2;
        t[k] = split_term<TS>(p[k], xi, vi, w, r2);
        if (TS) {
            hb.least = fmin(hb.least, r2 * ic2[k]);   // (the star's 1 / c^2 here is DBL_MAX)
            if (k == N - 2 - Seat::kLast * Seat::kTerms)
                hb.ri2 = r2;   // the star on lane kLast
        }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        a[c] = 0.0;
        jk[c] = 0.0;
    }
    split_turns<N, G, 0>(t, a, jk);
    share_read3<share_of<G>(Seat::kLast)>(a);
    share_read3<share_of<G>(Seat::kLast)>(jk);
    wave_sync();
}

template <int N, int G, bool TS>
__device__ __forceinline__ void split_step(BplLds &L, const SplitSeat<N, G> &s, const Coef &k,
                                           const double (&x)[3], const double (&v)[3],
                                           const double (&a0)[3], const double (&j0)[3],
                                           double (&xc)[3], double (&vc)[3], double (&ak)[3],
                                           double (&jk)[3], double &w,
                                           const double (&ic2)[SplitSeat<N, G>::kTerms],
                                           HillBound &hb, double &moved2)
{
    double bx[3], bv[3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
        predict_comp(k, x[c], v[c], a0[c], j0[c], xc[c], vc[c], bx[c], bv[c]);
    split_eval<N, G, false>(L, s, xc, vc, ak, jk, w, ic2, hb);
#pragma unroll
    for (int c = 0; c < 3; ++c)
        correct_comp(k, bx[c], bv[c], ak[c], jk[c], xc[c], vc[c]);
    const double x1[3] = {xc[0], xc[1], xc[2]};
    split_eval<N, G, TS>(L, s, xc, vc, ak, jk, w, ic2, hb);
#pragma unroll
    for (int c = 0; c < 3; ++c)
        correct_comp(k, bx[c], bv[c], ak[c], jk[c], xc[c], vc[c]);
    if (TS) {
        const double d0 = xc[0] - x1[0], d1 = xc[1] - x1[1], d2 = xc[2] - x1[2];
        moved2 = fma(d2, d2, fma(d1, d1, d0 * d0));
    }
}

// nrun fixed steps of this lane's system (bpl_fixed_steps).
template <int N, int G>
__device__ __forceinline__ void split_fixed_steps(BplLds &L, const SplitSeat<N, G> &s, const Coef &k,
                                                  const bool live, const int nrun, double (&x)[3],
                                                  double (&v)[3], double (&a0)[3], double (&j0)[3])
{
    const unsigned long long who = __ballot(live && nrun > 0);
    if (who == 0ull)
        return;
    const int n0 = __builtin_amdgcn_readlane(nrun, __builtin_ctzll(who));
    double w = 0.0, moved2 = 0.0;
    HillBound hb;
    if (__all(!live || nrun == n0)) {
#pragma unroll 1
        for (int q = 0; q < n0; ++q) {
            double xc[3], vc[3], ak[3], jk[3];
            split_step<N, G, false>(L, s, k, x, v, a0, j0, xc, vc, ak, jk, w, s.m, hb, moved2);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                x[c] = xc[c];
                v[c] = vc[c];
                a0[c] = ak[c];
                j0[c] = jk[c];
            }
        }
        return;
    }
    int q = 0;
#pragma unroll 1
    do {
        const bool act = q < nrun;
        double xc[3], vc[3], ak[3], jk[3];
        split_step<N, G, false>(L, s, k, x, v, a0, j0, xc, vc, ak, jk, w, s.m, hb, moved2);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            x[c] = act ? xc[c] : x[c];
            v[c] = act ? vc[c] : v[c];
            a0[c] = act ? ak[c] : a0[c];
            j0[c] = act ? jk[c] : j0[c];
        }
        ++q;
    } while (__any(q < nrun));
}

// OR of the stop-flag bits (1, 2, 4) over the lanes of system sys.
template <int N, int G>
__device__ __forceinline__ int split_or_flags(const int sys, const int v)
{
    constexpr int S = split_systems(N, G);
    constexpr unsigned long long kBase = [] {
        unsigned long long m = 0;
        for (int k = 0; k < N; ++k)
            m |= ((1ull << G) - 1) << (G * k * S);
        return m;
    }();
    const unsigned long long sm = kBase << (G * sys);
    int r = 0;
#pragma unroll
    for (int bit = 1; bit <= 4; bit <<= 1)
        if (__ballot((v & bit) != 0) & sm)
            r |= bit;
    return r;
}

// Stop-rule flags and the system's maximum of w (bpl_stop_flags_regs): every
// lane tests its body with its own share of the partners.
template <int N, int G>
__device__ __forceinline__ int split_stop_flags(BplLds &L, const SplitSeat<N, G> &s, const int b,
                                                const int sys, const double mi,
                                                const double inv24m0, const double (&x)[3],
                                                const double (&v)[3], const double w,
                                                double &wsys, const HillBound &part,
                                                const double moved2, const double move2_most,
                                                const bool act, const StepParams &P)
{
    constexpr int kTerms = SplitSeat<N, G>::kTerms;
    int fl = (finite3(x) && finite3(v)) ? 0 : 1;
    wsys = share_max<G>(w);
    if (!P.stop_rules) {
        if (P.adaptive == 1) {
            if (s.share == 0)
                L.mr[s.entry].y = wsys;
            wave_sync();
            double r[kTerms];
#pragma unroll
            for (int k = 0; k < kTerms; ++k)
                r[k] = L.mr[s.idx[k]].y;
            wave_sync();
#pragma unroll
            for (int k = 0; k < kTerms; ++k)
                wsys = fmax(wsys, r[k]);
            wsys = share_max<G>(wsys);
        }
        return __any(fl) ? split_or_flags<N, G>(sys, fl) : 0;
    }
    // the system's maxima of w and of how far its bodies moved, and whether its
    // planets can trigger at all
    if (s.share == 0)
        L.xy[s.entry] = make_double2(wsys, moved2);
    wave_sync();
    double2 mx[kTerms];
#pragma unroll
    for (int k = 0; k < kTerms; ++k)
        mx[k] = L.xy[s.idx[k]];
    wave_sync();
    double d2 = moved2;
#pragma unroll
    for (int k = 0; k < kTerms; ++k) {
        wsys = fmax(wsys, mx[k].x);
        d2 = fmax(d2, mx[k].y);
    }
    wsys = share_max<G>(wsys);
    d2 = share_max<G>(d2);
    HillBound hb = part;
    {
        double t[3] = {hb.ri2, 0.0, 0.0};
        share_read3<share_of<G>(SplitSeat<N, G>::kLast)>(t);
        hb.ri2 = t[0];
    }
    if (!__any(act && b >= 1 && may_stop(hb, d2, move2_most, P)))
        return __any(fl) ? split_or_flags<N, G>(sys, fl) : 0;
    if (s.share == 0) {
        L.xy[s.entry] = make_double2(x[0], x[1]);
        L.zvx[s.entry] = make_double2(x[2], 0.0);
    }
    wave_sync();
    double2 q0[kTerms], q1[kTerms];
#pragma unroll
    for (int k = 0; k < kTerms; ++k) {
        q0[k] = L.xy[s.idx[k]];
        q1[k] = L.zvx[s.idx[k]];
    }
    const double2 s0 = L.xy[sys];
    const double2 s1 = L.zvx[sys];
    wave_sync();
    const double dx = x[0] - s0.x, dy = x[1] - s0.y, dz = x[2] - s1.x;
    const double rb = sqrt(fma(dz, dz, fma(dy, dy, dx * dx)));
    if (P.stop_rules & 1) {
        double rp[kTerms];
        if (s.share == 0)
            L.mr[s.entry].y = rb;
        wave_sync();
#pragma unroll
        for (int k = 0; k < kTerms; ++k)
            rp[k] = L.mr[s.idx[k]].y;
        wave_sync();
        if (b >= 1) {
#pragma unroll
            for (int k = 0; k < kTerms; ++k) {
                const double ex = x[0] - q0[k].x, ey = x[1] - q0[k].y, ez = x[2] - q1[k].x;
                const double sep2 = fma(ez, ez, fma(ey, ey, ex * ex));
                // (the last partner in evaluation order is the star)
                if (s.share * kTerms + k < N - 2 && hill_close(sep2, mi, s.m[k], inv24m0, rb, rp[k]))
                    fl |= 2;
            }
        }
    }
    if (b >= 1 && (P.stop_rules & 2) && rb > P.r_eject)
        fl |= 4;
    return split_or_flags<N, G>(sys, fl);
}

// Integrate one tile (at most split_systems(N, G) systems) for at most P.quantum
// steps; bpl_run's contract.  SOLO: of the batch io instead of the bucket,
// with the evaluation it starts from.
template <int N, int G, bool ADV, bool SOLO = false>
__device__ __forceinline__ bool split_run(BplLds &L, const Bucket &B, const int first,
                                          const int count, const int *list, const StepParams &P,
                                          int &slot_out, const SoloIO &io = SoloIO())
{
    constexpr int S = split_systems(N, G), kTerms = SplitSeat<N, G>::kTerms;
    const int lane = threadIdx.x & 63, j = lane / G;
    const int braw = j / S;
    const int b = braw < N ? braw : N - 1;
    const int sys = j - braw * S;
    const bool valid = braw < N && sys < count;
    int slot = 0;
    if (valid)
        slot = list ? list[first + sys] : first + sys;
    slot_out = slot;
    const size_t pitch = SOLO ? 0 : B.pitch;
    double mi = 0.0, x[3] = {0.0, 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0};
    double a0[3] = {0.0, 0.0, 0.0}, j0[3] = {0.0, 0.0, 0.0};
    Clock c{};
    c.status = ST_DONE;
    if (SOLO && valid) {
        solo_load(io, N, slot, b, mi, x, v);
        c = solo_clock(io);
    }
    if (!SOLO && valid) {
        mi = B.st[(R_M * N + b) * pitch + slot];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            x[k] = B.st[((R_X + k) * N + b) * pitch + slot];
            v[k] = B.st[((R_V + k) * N + b) * pitch + slot];
            a0[k] = B.st[((R_A + k) * N + b) * pitch + slot];
            j0[k] = B.st[((R_J + k) * N + b) * pitch + slot];
        }
        c = load_clock(B, slot);
    }
    const bool live = c.status == ST_ACTIVE;
    SplitSeat<N, G> s;
    s.entry = j;   // = braw S + sys
    s.share = lane & (G - 1);
    if (s.share == 0)
        L.mr[j].x = mi;
    wave_sync();
#pragma unroll
    for (int k = 0; k < kTerms; ++k) {
        // what is past the last partner is not added: any entry
        const int kk = min(s.share * kTerms + k, N - 2);
        const int skip = b == 0 ? 1 << 20 : b;
        const int p = kk < N - 2 ? kk + 1 + (kk + 1 >= skip ? 1 : 0) : (b == 0 ? N - 1 : 0);
        s.idx[k] = p * S + sys;
        s.m[k] = L.mr[s.idx[k]].x;
    }
    if constexpr (SOLO) {
        double w = 0.0;
        HillBound hb;
        split_eval<N, G, false>(L, s, x, v, a0, j0, w, s.m, hb);
    }
    if constexpr (!ADV) {
        int budget = P.quantum;
#pragma unroll 1
        for (int seg = 0; seg < 2; ++seg) {
            double h = c.dt;
            const int nrun = run_segment(c, P, seg, budget, h);
            split_fixed_steps<N, G>(L, s, make_coef(h), live, nrun, x, v, a0, j0);
            budget -= nrun;
            run_segment_end(c, P, seg, nrun);
        }
        const int fl = split_or_flags<N, G>(sys, (finite3(x) && finite3(v)) ? 0 : 1);
        if (live && fl)
            c.status = ST_NONFINITE;
    } else {
        const double inv24m0 = 1.0 / (24.0 * L.mr[sys].x);
        double ic2[kTerms], ic2_most = 0.0;
#pragma unroll
        for (int k = 0; k < kTerms; ++k) {
            const bool planet = s.share * kTerms + k < N - 2;
            ic2[k] = planet && P.stop_rules ? hill_scale(mi, s.m[k], inv24m0) : DBL_MAX;
            ic2_most = fmax(ic2_most, planet ? ic2[k] : 0.0);
        }
        const double move2_most = move_scale(share_max<G>(ic2_most));
        for (int q = 0; q < P.quantum; ++q) {
            double h = 0.0;
            bool last = false;
            const bool act = P.adaptive ? plan_step_adaptive(c, P, h, last)
                                        : valid && plan_step(c, P, h, last);
            if (!__any(act))
                break;
            double xc[3], vc[3], ak[3], jk[3], w = 0.0, moved2 = 0.0;
            HillBound hb;
            split_step<N, G, true>(L, s, make_coef(h), x, v, a0, j0, xc, vc, ak, jk, w, ic2, hb,
                                   moved2);
            double dtp = 0.0;
            if (P.adaptive == 2) {
                const double aa = fma(ak[2], ak[2], fma(ak[1], ak[1], ak[0] * ak[0]));
                const double jj = fma(jk[2], jk[2], fma(jk[1], jk[1], jk[0] * jk[0]));
                if (s.share == 0)
                    L.mr[s.entry].y = jj / aa;
                wave_sync();
                double r = L.mr[sys].y;   // body order
#pragma unroll
                for (int k = 1; k < N; ++k)
                    r += L.mr[k * S + sys].y;
                wave_sync();
                dtp = P.eta * rsqrt_nr(r);
            }
            if (act) {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    x[k] = xc[k];
                    v[k] = vc[k];
                    a0[k] = ak[k];
                    j0[k] = jk[k];
                }
            }
            double wsys = 0.0;
            const int fl = split_stop_flags<N, G>(L, s, b, sys, mi, inv24m0, x, v, w, wsys,
                                                  hb, moved2, move2_most, act, P);
            if (P.adaptive == 1)
                dtp = P.eta * rsqrt_nr(wsys);
            if (P.adaptive) {
                finish_step_adaptive(c, act, last, h, dtp, fl);
            } else if (act) {
                finish_step(c, P, last, h, dtp);
                if (fl)
                    c.status = status_of_flags(fl);
            }
        }
    }
    if (SOLO && live && s.share == 0)
        solo_store(io, N, slot, b, x, v, c.status);
    if (!SOLO && live && s.share == 0) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            B.st[((R_X + k) * N + b) * pitch + slot] = x[k];
            B.st[((R_V + k) * N + b) * pitch + slot] = v[k];
            B.st[((R_A + k) * N + b) * pitch + slot] = a0[k];
            B.st[((R_J + k) * N + b) * pitch + slot] = j0[k];
        }
        if (b == 0)
            store_clock(B, slot, c);
    }
    return valid && braw == 0 && s.share == 0 && c.status == ST_ACTIVE;
}

}  // namespace
}  // namespace fb
