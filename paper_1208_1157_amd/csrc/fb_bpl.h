// fb_bpl.h -- Hermite steps with one body per lane of a wavefront, shared by
// the kernels that run such tiles.
#pragma once

#include "fb_device.h"

#include <cfloat>

// Partner-loop unroll of the body-per-lane evaluation: full unrolling lets
// the scheduler hoist every partner's LDS loads and costs occupancy.
#ifndef FB_BPL_UNROLL
#define FB_BPL_UNROLL 1
#endif

namespace fb {
namespace {

// Stop-rule flags after a committed step: bit 0 non-finite, bit 1 two
// planets within one mutual Hill radius, bit 2 a planet beyond r_eject.
// The Hill test sep < ((m_i+m_j)/(3 m0))^(1/3) (r_i+r_j)/2 (r the astrocentric
// distance) is evaluated without roots as
// sep^6 < ((m_i+m_j)/(24 m0))^2 ((r_i+r_j)^2)^3.
__device__ __forceinline__ bool hill_close(double sep2, double mi, double mj, double inv24m0,
                                           double ri, double rj)
{
    const double mu = (mi + mj) * inv24m0;
    const double w = (ri + rj) * (ri + rj);
    return sep2 * sep2 * sep2 < mu * mu * (w * w * w);
}

// The Hill and ejection tests trigger in few steps of few systems, and cost two
// exchanges through LDS and 16 instructions a pair in each.  A bound from the
// step's last evaluation, whose pair separations s and distances r_i from the
// star are at hand, tells which wavefronts need them at all.  Two planets trigger at a separation S <
// q (R_i + R_j), q = ((m_i + m_j) / (24 m0))^(1/3), and R_j <= R_i + S, so only
// if S < c R_i with c = 2 q / (1 - q).  If no body has moved by more than
// d <= 0.02 c / (1 + c) r_i since that evaluation, S >= s - 2 d and R_i <=
// r_i + 2 d, and s^2 >= 1.1 c^2 r_i^2 (s >= 1.048 c r_i) rules it out; likewise
// 1.2 r_i^2 < r_eject^2 an ejection (r_i + 2 d <= 1.04 r_i).
// A step of 8 bodies with both rules, a wavefront a SIMD: 2.55 -> 2.22 us; 10
// orbits of 65536 systems of 4..8 bodies 71 -> 66 ms.

// 1 / c^2 of a pair, at most 1e8 (a smaller pair is treated as one of c = 1e-4);
// 0, so never ruled out, from q = 1 on and for NaN.
__device__ __forceinline__ double hill_scale(const double mi, const double mj, const double inv24m0)
{
    const double q = cbrt((mi + mj) * inv24m0);
    const double ic = (1.0 - q) / (q + q);
    return q < 1.0 ? fmin(ic * ic, 1e8) : 0.0;
}

// Largest (d / r_i)^2 for a body whose largest 1 / c^2 is ic2: (0.02 / (1 + 1/c))^2,
// or less.
__device__ __forceinline__ double move_scale(const double ic2)
{
    return 1e-4 / (1.0 + ic2);   // (1 + 1/c)^2 <= 2 (1 + 1/c^2); 0.02^2 / 2 = 2e-4
}

// What the tests' bound takes from an evaluation: the least s^2 / c^2 over the
// planet partners, and r_i^2.
struct HillBound {
    double least, ri2;
};

// Whether a lane's planet may trigger a stop rule; d2 is the largest square
// of a distance that a body of its system has moved by since the bound.
__device__ __forceinline__ bool may_stop(const HillBound &hb, const double d2,
                                         const double move2_most, const StepParams &P)
{
    return !(d2 <= move2_most * hb.ri2) || ((P.stop_rules & 1) && !(hb.least >= 1.1 * hb.ri2)) ||
           ((P.stop_rules & 2) && !(1.2 * hb.ri2 < P.r_eject * P.r_eject));
}

// ---------------------------------------------------------------------------
// body-per-lane (BPL)
// ---------------------------------------------------------------------------

// LDS slot of the k-th planet partner (0 <= k < N-2, the other planets in
// ascending order) of body b of system s, with own = b S (the star lane
// passes 64, past every body): (k + 1) S + s, moved one body up from b on.
// The body offset (k + 1) S is uniform, so the slot costs a compare, a select
// and an add per partner.
template <int N>
__device__ __forceinline__ int partner_slot(const int k, const int s, const int own)
{
    constexpr int S = 64 / N;
    const int ks = (k + 1) * S;
    return s + ks + (ks >= own ? S : 0);
}

// A partner's evaluation state as read from the wavefront's LDS slice.
struct Partner {
    double2 p0, p1, p2;   // (x, y), (z, vx), (vy, vz)
    double mj;
};

__device__ __forceinline__ Partner bpl_partner(const BplLds &L, const int idx)
{
    return Partner{L.xy[idx], L.zvx[idx], L.vyvz[idx], L.mr[idx].x};
}

// One interaction of body i (this lane) with partner P: adds m_j A and m_j J
// (Eq. 1 and its time derivative).
template <bool TS>
__device__ __forceinline__ void bpl_interact_p(const Partner &Pj, const double (&xi)[3],
                                               const double (&vi)[3], double (&a)[3],
                                               double (&jk)[3], double &wmax, double *r2_out = nullptr)
{
    const double2 p0 = Pj.p0, p1 = Pj.p1, p2 = Pj.p2;
    const double mj = Pj.mj;
    const double rx = p0.x - xi[0], ry = p0.y - xi[1], rz = p1.x - xi[2];
    const double ux = p1.y - vi[0], uy = p2.x - vi[1], uz = p2.y - vi[2];
    const double r2 = fma(rz, rz, fma(ry, ry, rx * rx));
    if (r2_out)
        *r2_out = r2;
    const double ru = fma(rz, uz, fma(ry, uy, rx * ux));
    const double ri = rsqrt_nr(r2);
    const double ri2 = ri * ri;
    const double mr3 = mj * (ri2 * ri);
    const double al = 3.0 * ru * ri2;
    a[0] = fma(mr3, rx, a[0]);
    a[1] = fma(mr3, ry, a[1]);
    a[2] = fma(mr3, rz, a[2]);
    jk[0] = fma(mr3, fma(-al, rx, ux), jk[0]);
    jk[1] = fma(mr3, fma(-al, ry, uy), jk[1]);
    jk[2] = fma(mr3, fma(-al, rz, uz), jk[2]);
    if (TS) {
        const double u2 = fma(uz, uz, fma(uy, uy, ux * ux));
        wmax = fmax(wmax, fma(al, ru, u2) * ri2);
    }
}

// One interaction of body i (this lane) with the partner stored at LDS index
// idx.
template <bool TS>
__device__ __forceinline__ void bpl_interact(const BplLds &L, const int idx,
                                             const double (&xi)[3], const double (&vi)[3],
                                             double (&a)[3], double (&jk)[3], double &wmax)
{
    bpl_interact_p<TS>(bpl_partner(L, idx), xi, vi, a, jk, wmax);
}

// Accelerations and jerks of this lane's body from all n-1 partners read
// from the wavefront's LDS slice.  Partner order: the other planets in
// ascending order, then the star (the star lane sums planets 1..n-1), so the
// star's contribution is added last.  Branch-free: the n-2 planet partners
// skip this lane's own index arithmetically and the last partner is peeled.
// ILP unrolls the partner loop fully (kernels with one or two waves a SIMD,
// which need independent interactions in flight); the accumulation order is
// the same either way.
template <int N, bool TS, bool ILP = false>
__device__ __forceinline__ void bpl_eval(BplLds &L, const int lane, const int b, const int s,
                                         const double (&xi)[3], const double (&vi)[3],
                                         double (&a)[3], double (&jk)[3], double &wmax)
{
    constexpr int S = 64 / N;
    L.xy[lane] = make_double2(xi[0], xi[1]);
    L.zvx[lane] = make_double2(xi[2], vi[0]);
    L.vyvz[lane] = make_double2(vi[1], vi[2]);
    wave_sync();
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        a[c] = 0.0;
        jk[c] = 0.0;
    }
    const int own = b == 0 ? 64 : b * S;
    if constexpr (ILP) {
#pragma unroll
        for (int k = 0; k < N - 2; ++k)
            bpl_interact<TS>(L, partner_slot<N>(k, s, own), xi, vi, a, jk, wmax);
    } else {
#pragma unroll FB_BPL_UNROLL
        for (int k = 0; k < N - 2; ++k)
            bpl_interact<TS>(L, partner_slot<N>(k, s, own), xi, vi, a, jk, wmax);
    }
    bpl_interact<TS>(L, (b == 0 ? N - 1 : 0) * S + s, xi, vi, a, jk, wmax);
    wave_sync();
}

template <int N, bool ILP = false>
__device__ __forceinline__ int bpl_stop_flags(BplLds &L, const int lane, const int b,
                                              const int s, const double mi, const double inv24m0,
                                              const double (&x)[3], const double (&v)[3],
                                              const StepParams &P)
{
    constexpr int S = 64 / N;
    int fl = (finite3(x) && finite3(v)) ? 0 : 1;
    if (!P.stop_rules)
        return __any(fl) ? sys_or_flags<N>(s, fl) : 0;
    L.xy[lane] = make_double2(x[0], x[1]);
    L.zvx[lane] = make_double2(x[2], 0.0);
    wave_sync();
    const double2 s0 = L.xy[s];
    const double2 s1 = L.zvx[s];
    const double dx = x[0] - s0.x, dy = x[1] - s0.y, dz = x[2] - s1.x;
    const double rb = sqrt(fma(dz, dz, fma(dy, dy, dx * dx)));
    L.mr[lane].y = rb;
    wave_sync();
    if (b >= 1) {
        if ((P.stop_rules & 2) && rb > P.r_eject)
            fl |= 4;
        if (P.stop_rules & 1) {
            const int own = b * S;
            auto hill = [&](const int k) {
                const int idx = partner_slot<N>(k, s, own);
                const double2 q0 = L.xy[idx];
                const double2 q1 = L.zvx[idx];
                const double ex = x[0] - q0.x, ey = x[1] - q0.y, ez = x[2] - q1.x;
                const double sep2 = fma(ez, ez, fma(ey, ey, ex * ex));
                if (hill_close(sep2, mi, L.mr[idx].x, inv24m0, rb, L.mr[idx].y))
                    fl |= 2;
            };
            if constexpr (ILP) {
#pragma unroll
                for (int k = 0; k < N - 2; ++k)
                    hill(k);
            } else {
#pragma unroll 1
                for (int k = 0; k < N - 2; ++k)
                    hill(k);
            }
        }
    }
    wave_sync();
    return sys_or_flags<N>(s, fl);
}

// Unrolled variants of the evaluation and of the stop-rule pass, for a wave
// that has its SIMD to itself or shares it with one other and so waits out most
// LDS round trips and dependent latencies: the partner slots (pidx) and masses
// (pm) of this lane's body, in evaluation order, are fixed over the run and held
// in registers, and partners are read before the first interaction: all of
// them, or (PARTS) a part of them at a time, where all would not leave room for
// a second wave (14 and more bodies in fixed steps, which that wave gains: 240
// VGPRs instead of 340).
template <int N>
__device__ __forceinline__ int eval_partner(const int k, const int b)
{
    const int skip = b == 0 ? (1 << 20) : b;
    return k < N - 2 ? k + 1 + (k + 1 >= skip ? 1 : 0) : (b == 0 ? N - 1 : 0);
}

// Interactions with the partners of part PART of PARTS, all read before the
// first of them, and of the parts after it.
template <int N, bool TS, int PART, int PARTS>
__device__ __forceinline__ void bpl_partners(const BplLds &L, const int (&pidx)[N - 1],
                                             const double (&pm)[N - 1], const double (&xi)[3],
                                             const double (&vi)[3], double (&a)[3],
                                             double (&jk)[3], double &wmax,
                                             const double (&ic2)[N - 1], HillBound &hb)
{
    constexpr int K0 = PART * (N - 1) / PARTS, K1 = (PART + 1) * (N - 1) / PARTS;
    Partner pj[K1 - K0];
#pragma unroll
    for (int k = K0; k < K1; ++k)
        pj[k - K0] = Partner{L.xy[pidx[k]], L.zvx[pidx[k]], L.vyvz[pidx[k]], pm[k]};
    if constexpr (N <= 9 || PARTS > 1)   // (more partners' state does not fit the VGPRs at once)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = K0; k < K1; ++k) {
        double r2;
        bpl_interact_p<TS>(pj[k - K0], xi, vi, a, jk, wmax, &r2);
        if (TS) {
            if (k < N - 2)
                hb.least = fmin(hb.least, r2 * ic2[k]);
            else
                hb.ri2 = r2;
        }
    }
    if constexpr (PART + 1 < PARTS) {
        __builtin_amdgcn_sched_barrier(0);
        bpl_partners<N, TS, PART + 1, PARTS>(L, pidx, pm, xi, vi, a, jk, wmax, ic2, hb);
    }
}

// With TS, also the bound hb of the stop rules, with the pairs' 1 / c^2 in ic2.
template <int N, bool TS, int PARTS>
__device__ __forceinline__ void bpl_eval_regs(BplLds &L, const int lane, const int (&pidx)[N - 1],
                                              const double (&pm)[N - 1], const double (&xi)[3],
                                              const double (&vi)[3], double (&a)[3],
                                              double (&jk)[3], double &wmax,
                                              const double (&ic2)[N - 1], HillBound &hb)
{
    L.xy[lane] = make_double2(xi[0], xi[1]);
    L.zvx[lane] = make_double2(xi[2], vi[0]);
    L.vyvz[lane] = make_double2(vi[1], vi[2]);
    wave_sync();
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        a[c] = 0.0;
        jk[c] = 0.0;
    }
    hb.least = DBL_MAX;
    bpl_partners<N, TS, 0, PARTS>(L, pidx, pm, xi, vi, a, jk, wmax, ic2, hb);
    wave_sync();
}

// Stop-rule flags (as bpl_stop_flags) and the system maximum of the step
// rule's w (as sys_max): one exchange of each lane's position and w gives
// the star's position, the partners' positions and every w; a second, of
// the astrocentric distances, the Hill test's partner radii.
template <int N>
__device__ __forceinline__ int bpl_stop_flags_regs(BplLds &L, const int lane, const int b,
                                                   const int s, const int (&pidx)[N - 1],
                                                   const double (&pm)[N - 1], const double mi,
                                                   const double inv24m0, const double (&x)[3],
                                                   const double (&v)[3], const double w,
                                                   double &wsys, const HillBound &hb,
                                                   const double moved2, const double move2_most,
                                                   const bool act, const StepParams &P)
{
    int fl = (finite3(x) && finite3(v)) ? 0 : 1;
    if (!P.stop_rules) {
        wsys = P.adaptive == 1 ? sys_max<N>(L, lane, s, w) : w;
        return __any(fl) ? sys_or_flags<N>(s, fl) : 0;
    }
    // the system's maxima of w and of how far its bodies moved: max is exact,
    // so the partners' order gives the body-order result
    L.xy[lane] = make_double2(w, moved2);
    wave_sync();
    double2 mx[N - 1];
#pragma unroll
    for (int k = 0; k < N - 1; ++k)
        mx[k] = L.xy[pidx[k]];
    wave_sync();
    wsys = w;
    double d2 = moved2;
#pragma unroll
    for (int k = 0; k < N - 1; ++k) {
        wsys = fmax(wsys, mx[k].x);
        d2 = fmax(d2, mx[k].y);
    }
    if (!__any(act && b >= 1 && may_stop(hb, d2, move2_most, P)))
        return __any(fl) ? sys_or_flags<N>(s, fl) : 0;
    L.xy[lane] = make_double2(x[0], x[1]);
    L.zvx[lane] = make_double2(x[2], 0.0);
    wave_sync();
    double2 q0[N - 1], q1[N - 1];
#pragma unroll
    for (int k = 0; k < N - 1; ++k) {
        q0[k] = L.xy[pidx[k]];
        q1[k] = L.zvx[pidx[k]];
    }
    const double2 s0 = L.xy[s];
    const double2 s1 = L.zvx[s];
    wave_sync();
    const double dx = x[0] - s0.x, dy = x[1] - s0.y, dz = x[2] - s1.x;
    const double rb = sqrt(fma(dz, dz, fma(dy, dy, dx * dx)));
    if (P.stop_rules & 1) {
        // the partners' astrocentric distances: a second exchange is
        // shorter than computing N - 2 more square roots per lane
        double rp[N - 1];
        L.mr[lane].y = rb;
        wave_sync();
#pragma unroll
        for (int k = 0; k < N - 2; ++k)
            rp[k] = L.mr[pidx[k]].y;
        wave_sync();
        if (b >= 1) {
#pragma unroll
            for (int k = 0; k < N - 2; ++k) {
                const double ex = x[0] - q0[k].x, ey = x[1] - q0[k].y, ez = x[2] - q1[k].x;
                const double sep2 = fma(ez, ez, fma(ey, ey, ex * ex));
                if (hill_close(sep2, mi, pm[k], inv24m0, rb, rp[k]))
                    fl |= 2;
            }
        }
    }
    if (b >= 1 && (P.stop_rules & 2) && rb > P.r_eject)
        fl |= 4;
    return sys_or_flags<N>(s, fl);
}

// One P(EC)^2 step with the coefficients k: (xc, vc) the corrected state, (ak,
// jk) the last evaluation; with TS the step rule's quantity w of it, and (REGS)
// the stop rules' bound hb and how far the body moved after it.
template <int N, bool TS, bool REGS, bool ILP>
__device__ __forceinline__ void bpl_step(BplLds &L, const int lane, const int b, const int s,
                                         const int (&pidx)[N - 1], const double (&pm)[N - 1],
                                         const Coef &k, const double (&x)[3], const double (&v)[3],
                                         const double (&a0)[3], const double (&j0)[3],
                                         double (&xc)[3], double (&vc)[3], double (&ak)[3],
                                         double (&jk)[3], double &w, const double (&ic2)[N - 1],
                                         HillBound &hb, double &moved2)
{
    constexpr int PARTS = !TS && N >= 14 ? 3 : 1;
    double bx[3], bv[3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
        predict_comp(k, x[c], v[c], a0[c], j0[c], xc[c], vc[c], bx[c], bv[c]);
    if constexpr (REGS)
        bpl_eval_regs<N, false, PARTS>(L, lane, pidx, pm, xc, vc, ak, jk, w, ic2, hb);
    else
        bpl_eval<N, false, ILP>(L, lane, b, s, xc, vc, ak, jk, w);
#pragma unroll
    for (int c = 0; c < 3; ++c)
        correct_comp(k, bx[c], bv[c], ak[c], jk[c], xc[c], vc[c]);
    const double x1[3] = {xc[0], xc[1], xc[2]};
    if constexpr (REGS)
        bpl_eval_regs<N, TS, PARTS>(L, lane, pidx, pm, xc, vc, ak, jk, w, ic2, hb);
    else
        bpl_eval<N, TS, ILP>(L, lane, b, s, xc, vc, ak, jk, w);
#pragma unroll
    for (int c = 0; c < 3; ++c)
        correct_comp(k, bx[c], bv[c], ak[c], jk[c], xc[c], vc[c]);
    if (TS && REGS) {
        const double d0 = xc[0] - x1[0], d1 = xc[1] - x1[1], d2 = xc[2] - x1[2];
        moved2 = fma(d2, d2, fma(d1, d1, d0 * d0));
    }
}

// nrun fixed steps of this lane's system.  Where every running lane has the
// same count (live lanes; the state of the others is never stored) the loop
// carries no per-lane bookkeeping and the state needs no selects; otherwise a
// lane past its count keeps its state.
template <int N, bool REGS, bool ILP>
__device__ __forceinline__ void bpl_fixed_steps(BplLds &L, const int lane, const int b,
                                                const int s, const int (&pidx)[N - 1],
                                                const double (&pm)[N - 1], const Coef &k,
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
            bpl_step<N, false, REGS, ILP>(L, lane, b, s, pidx, pm, k, x, v, a0, j0, xc, vc, ak,
                                          jk, w, pm, hb, moved2);
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
        bpl_step<N, false, REGS, ILP>(L, lane, b, s, pidx, pm, k, x, v, a0, j0, xc, vc, ak, jk, w,
                                      pm, hb, moved2);
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

// Integrate one tile (floor(64/N) systems) with one body per lane for at
// most P.quantum steps.  Every lane of the wavefront executes the same
// control flow (the LDS exchanges need it); lanes of finished, padding or
// absent systems compute but never commit.  REGS: partner tables
// in registers, for kernels with one or two waves a SIMD; WIDE: the LDS
// stride and register file of the system-per-lane fused class.  Returns, on the star lane of each present system, whether that
// system is still active.
template <int N, bool ADV, bool WIDE, bool REGS>
__device__ __forceinline__ bool bpl_run(const Bucket &B, const int first, const int count, const int *list,
                        const StepParams &P, int &slot_out)
{
    constexpr int S = 64 / N;
    constexpr bool ILP = WIDE || REGS;   // unrolled partner loops
    BplLds &L = *reinterpret_cast<BplLds *>(wave_lds_base<sizeof(BplLds), WIDE>());
    const int lane = threadIdx.x & 63;
    const int braw = lane / S;
    const int b = braw < N ? braw : N - 1;
    const int s = lane - braw * S;
    const bool valid = braw < N && s < count;
    int slot = 0;
    if (valid)
        slot = list ? list[first + s] : first + s;
    slot_out = slot;
    const size_t pitch = B.pitch;
    double mi = 0.0, x[3] = {0.0, 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0};
    double a0[3] = {0.0, 0.0, 0.0}, j0[3] = {0.0, 0.0, 0.0};
    Clock c{};
    c.status = ST_DONE;
    if (valid) {
        mi = B.st[(R_M * N + b) * pitch + slot];
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            x[cc] = B.st[((R_X + cc) * N + b) * pitch + slot];
            v[cc] = B.st[((R_V + cc) * N + b) * pitch + slot];
            a0[cc] = B.st[((R_A + cc) * N + b) * pitch + slot];
            j0[cc] = B.st[((R_J + cc) * N + b) * pitch + slot];
        }
        c = load_clock(B, slot);
    }
    const bool live = c.status == ST_ACTIVE;   // systems that may step: only they are stored
    L.mr[lane].x = mi;
    wave_sync();
    int pidx[N - 1];
    double pm[N - 1];
#pragma unroll
    for (int k = 0; k < N - 1; ++k) {
        pidx[k] = REGS ? eval_partner<N>(k, b) * S + s : 0;
        pm[k] = REGS ? L.mr[pidx[k]].x : 0.0;
    }
    if constexpr (!ADV) {
        int budget = P.quantum;
#pragma unroll 1
        for (int seg = 0; seg < 2; ++seg) {
            double h = c.dt;
            const int nrun = run_segment(c, P, seg, budget, h);
            bpl_fixed_steps<N, REGS, ILP>(L, lane, b, s, pidx, pm, make_coef(h), live, nrun, x, v,
                                          a0, j0);
            budget -= nrun;
            run_segment_end(c, P, seg, nrun);
        }
    } else {
        // Hill-test scale of the system's star, fixed over the run.
        const double inv24m0 = 1.0 / (24.0 * L.mr[s].x);
        double ic2[N - 1], ic2_most = 0.0;
#pragma unroll
        for (int k = 0; k < N - 1; ++k)
            ic2[k] = REGS && P.stop_rules ? hill_scale(mi, pm[k], inv24m0) : 0.0;
#pragma unroll
        for (int k = 0; k < N - 2; ++k)
            ic2_most = fmax(ic2_most, ic2[k]);
        const double move2_most = move_scale(ic2_most);
        for (int q = 0; q < P.quantum; ++q) {
            double h = 0.0;
            bool last = false;
            bool act;
            if constexpr (REGS)   // invalid lanes hold an inactive clock
                act = P.adaptive ? plan_step_adaptive(c, P, h, last) : valid && plan_step(c, P, h, last);
            else
                act = valid && plan_step(c, P, h, last);
            if (!__any(act))
                break;
            double xc[3], vc[3], ak[3], jk[3], w = 0.0, moved2 = 0.0;
            HillBound hb;
            bpl_step<N, true, REGS, ILP>(L, lane, b, s, pidx, pm, make_coef(h), x, v, a0, j0, xc,
                                         vc, ak, jk, w, ic2, hb, moved2);
            double dtp = 0.0;
            if (!REGS && P.adaptive == 1)
                dtp = P.eta * rsqrt_nr(sys_max<N>(L, lane, s, w));
            if (P.adaptive == 2) {
                const double aa = fma(ak[2], ak[2], fma(ak[1], ak[1], ak[0] * ak[0]));
                const double jj = fma(jk[2], jk[2], fma(jk[1], jk[1], jk[0] * jk[0]));
                dtp = P.eta * rsqrt_nr(sys_sum<N>(L, lane, s, jj / aa));
            }
            if (act) {
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) {
                    x[cc] = xc[cc];
                    v[cc] = vc[cc];
                    a0[cc] = ak[cc];
                    j0[cc] = jk[cc];
                }
            }
            if constexpr (REGS) {
                // one exchange for the step rule's maximum and the stop rules
                // (same values and order of decisions as below)
                double wsys = 0.0;
                const int fl = bpl_stop_flags_regs<N>(L, lane, b, s, pidx, pm, mi, inv24m0, x, v,
                                                      w, wsys, hb, moved2, move2_most, act, P);
                if (P.adaptive == 1)
                    dtp = P.eta * rsqrt_nr(wsys);
                if (P.adaptive) {
                    finish_step_adaptive(c, act, last, h, dtp, fl);
                } else if (act) {
                    finish_step(c, P, last, h, dtp);
                    if (fl)
                        c.status = status_of_flags(fl);
                }
            } else {
                if (act)
                    finish_step(c, P, last, h, dtp);
                const int fl = bpl_stop_flags<N, WIDE>(L, lane, b, s, mi, inv24m0, x, v, P);
                if (act && fl)
                    c.status = status_of_flags(fl);
            }
        }
    }
    if constexpr (!ADV) {
        const int fl = sys_or_flags<N>(s, (finite3(x) && finite3(v)) ? 0 : 1);
        if (live && fl)
            c.status = ST_NONFINITE;
    }
    if (live) {
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            B.st[((R_X + cc) * N + b) * pitch + slot] = x[cc];
            B.st[((R_V + cc) * N + b) * pitch + slot] = v[cc];
            B.st[((R_A + cc) * N + b) * pitch + slot] = a0[cc];
            B.st[((R_J + cc) * N + b) * pitch + slot] = j0[cc];
        }
        if (b == 0)
            store_clock(B, slot, c);
    }
    return valid && b == 0 && braw == 0 && c.status == ST_ACTIVE;
}

}  // namespace
}  // namespace fb
