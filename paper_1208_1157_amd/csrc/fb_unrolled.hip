// fb_unrolled.hip -- Hermite steps with one body per lane where the partner
// loops are unrolled and the whole register file is used: partner tables in
// registers, all partner reads of an evaluation issued before its first
// interaction and, up to four bodies, the bodies' state exchanged by lane
// permutes instead of through LDS.  The arithmetic and its order are those of
// the other Hermite kernels, so a result does not depend on which of them ran.
//
// Ensembles that fill the device system per lane do not come here.  One that
// gives a SIMD a single wavefront waits out the latencies of a step, of which
// the exchange of the bodies' state is the longest; with more wavefronts the
// rolled loops' address arithmetic and the dependent chain of one interaction
// after another still cost issue slots.  Microseconds per step against the
// rolled loops of k_plain_bpl (3 waves per SIMD), fixed steps:
//   waves per SIMD     n = 3        4           6           8          12
//   0.1             0.64 0.46  0.95 0.62  1.40 0.92  1.91 1.18  2.80 1.90
//   1               0.72 0.55  1.45 0.76  2.10 1.32  2.81 1.77  4.14 2.48
//   2               1.06 1.05  1.69 1.45  2.50 2.26  3.30 2.91  4.91 4.20
//   4                                     4.46 4.15  5.90 5.42  8.75 7.72
//   8                                                           15.8 14.6
// 13..16 bodies, of which (from 14 on) two wavefronts on a SIMD hold a third of
// the partners at a time: 60 steps of 16 bodies, 8192 systems (2 wavefronts a SIMD) 540 and 350
// us, 16000 730 and 645, 32000 1402 and 1240, 131072 4977 and 4574;
// and with adaptive steps and the stop rules, 1 and 4 waves per SIMD: n = 8
// 1.68x and 1.17x, n = 12 1.63x and 0.93x (its registers leave one wave per
// SIMD), n = 2 and 3 past one wave 0.94x and 0.88x.  bpl_mapping draws the line.
#include "fb_bpl.h"

namespace fb {
namespace {

// ---------------------------------------------------------------------------
// quads: systems of 2..4 bodies on the four lanes of a DPP quad
// ---------------------------------------------------------------------------
// Lane 4 s + b holds body b of system s (16 systems a wavefront; lanes past
// the system's bodies idle).  A quad permute moves a partner's value to every
// lane in one VALU instruction per 32 bits, with a pattern that gives each
// lane its own k-th partner in evaluation order; an exchange through LDS
// costs a wave that is alone on its SIMD about 450 clocks, twice a step.

// quad_perm control: lane b of every quad reads lane P(b).
constexpr int quad_ctrl(int p0, int p1, int p2, int p3)
{
    return p0 | (p1 << 2) | (p2 << 4) | (p3 << 6);
}

// The k-th partner of each body in evaluation order (the other planets in
// ascending order, then the star; the star: planets 1..N-1).  Idle lanes read
// the star.
template <int N>
constexpr int quad_partner(int k)
{
    int p[4] = {0, 0, 0, 0};
    for (int b = 0; b < N; ++b) {
        const int skip = b == 0 ? 1 << 20 : b;
        p[b] = k < N - 2 ? k + 1 + (k + 1 >= skip ? 1 : 0) : (b == 0 ? N - 1 : 0);
    }
    return quad_ctrl(p[0], p[1], p[2], p[3]);
}

template <int CTRL>
__device__ __forceinline__ double quad_read(const double v)
{
    const unsigned long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)(u & 0xffffffffull), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(u >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

template <int CTRL>
__device__ __forceinline__ int quad_read_i(const int v)
{
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}

// Interactions K..N-2 of this lane's body (by recursion: the permute pattern
// is an immediate of the instruction).
template <int N, bool TS, int K>
__device__ __forceinline__ void quad_interact(const double (&pm)[N - 1], const double (&xi)[3],
                                              const double (&vi)[3], double (&a)[3],
                                              double (&jk)[3], double &wmax)
{
    constexpr int C = quad_partner<N>(K);
    const Partner p{make_double2(quad_read<C>(xi[0]), quad_read<C>(xi[1])),
                    make_double2(quad_read<C>(xi[2]), quad_read<C>(vi[0])),
                    make_double2(quad_read<C>(vi[1]), quad_read<C>(vi[2])), pm[K]};
    bpl_interact_p<TS>(p, xi, vi, a, jk, wmax);
    if constexpr (K + 1 < N - 1)
        quad_interact<N, TS, K + 1>(pm, xi, vi, a, jk, wmax);
}

template <int N, bool TS>
__device__ __forceinline__ void quad_eval(const double (&pm)[N - 1], const double (&xi)[3],
                                          const double (&vi)[3], double (&a)[3], double (&jk)[3],
                                          double &wmax)
{
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        a[c] = 0.0;
        jk[c] = 0.0;
    }
    quad_interact<N, TS, 0>(pm, xi, vi, a, jk, wmax);
}

// The value of body b of this lane's system.
template <int B>
__device__ __forceinline__ double quad_body(const double v)
{
    return quad_read<quad_ctrl(B, B, B, B)>(v);
}

// Maximum, and sum in body order, over the system's bodies.
template <int N>
__device__ __forceinline__ double quad_max(const double v)
{
    double r = fmax(quad_body<0>(v), quad_body<1>(v));
    if constexpr (N > 2)
        r = fmax(r, quad_body<2>(v));
    if constexpr (N > 3)
        r = fmax(r, quad_body<3>(v));
    return r;
}

template <int N>
__device__ __forceinline__ double quad_sum(const double v)
{
    double r = quad_body<0>(v) + quad_body<1>(v);
    if constexpr (N > 2)
        r += quad_body<2>(v);
    if constexpr (N > 3)
        r += quad_body<3>(v);
    return r;
}

template <int N>
__device__ __forceinline__ int quad_or(const int v)
{
    int r = quad_read_i<quad_ctrl(0, 0, 0, 0)>(v) | quad_read_i<quad_ctrl(1, 1, 1, 1)>(v);
    if constexpr (N > 2)
        r |= quad_read_i<quad_ctrl(2, 2, 2, 2)>(v);
    if constexpr (N > 3)
        r |= quad_read_i<quad_ctrl(3, 3, 3, 3)>(v);
    return r;
}

// Hill tests of this lane's planet with its partners K..N-3 (flag bit 2).
template <int N, int K>
__device__ __forceinline__ int quad_hill(const double (&pm)[N - 1], const double mi,
                                         const double inv24m0, const double (&x)[3],
                                         const double rb)
{
    if constexpr (K >= N - 2) {
        return 0;
    } else {
        constexpr int C = quad_partner<N>(K);
        const double ex = x[0] - quad_read<C>(x[0]), ey = x[1] - quad_read<C>(x[1]),
                     ez = x[2] - quad_read<C>(x[2]);
        const double sep2 = fma(ez, ez, fma(ey, ey, ex * ex));
        const int fl = hill_close(sep2, mi, pm[K], inv24m0, rb, quad_read<C>(rb)) ? 2 : 0;
        return fl | quad_hill<N, K + 1>(pm, mi, inv24m0, x, rb);
    }
}

// Stop-rule flags of bpl_stop_flags.
template <int N>
__device__ __forceinline__ int quad_stop_flags(const int b, const double (&pm)[N - 1],
                                               const double mi, const double inv24m0,
                                               const double (&x)[3], const double (&v)[3],
                                               const StepParams &P)
{
    int fl = (b >= N || (finite3(x) && finite3(v))) ? 0 : 1;
    if (P.stop_rules) {
        const double dx = x[0] - quad_body<0>(x[0]), dy = x[1] - quad_body<0>(x[1]),
                     dz = x[2] - quad_body<0>(x[2]);
        const double rb = sqrt(fma(dz, dz, fma(dy, dy, dx * dx)));
        const bool planet = b >= 1 && b < N;
        if (P.stop_rules & 1) {
            const int hit = quad_hill<N, 0>(pm, mi, inv24m0, x, rb);
            fl |= planet ? hit : 0;
        }
        if ((P.stop_rules & 2) && planet && rb > P.r_eject)
            fl |= 4;
    }
    return quad_or<N>(fl);
}

template <int N, bool TS>
__device__ __forceinline__ void quad_step(const double (&pm)[N - 1], const Coef &k,
                                          const double (&x)[3], const double (&v)[3],
                                          const double (&a0)[3], const double (&j0)[3],
                                          double (&xc)[3], double (&vc)[3], double (&ak)[3],
                                          double (&jk)[3], double &w)
{
    double bx[3], bv[3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
        predict_comp(k, x[c], v[c], a0[c], j0[c], xc[c], vc[c], bx[c], bv[c]);
    quad_eval<N, false>(pm, xc, vc, ak, jk, w);
#pragma unroll
    for (int c = 0; c < 3; ++c)
        correct_comp(k, bx[c], bv[c], ak[c], jk[c], xc[c], vc[c]);
    quad_eval<N, TS>(pm, xc, vc, ak, jk, w);
#pragma unroll
    for (int c = 0; c < 3; ++c)
        correct_comp(k, bx[c], bv[c], ak[c], jk[c], xc[c], vc[c]);
}

__device__ __forceinline__ void select3(const bool p, const double (&a)[3], double (&b)[3])
{
#pragma unroll
    for (int c = 0; c < 3; ++c)
        b[c] = p ? a[c] : b[c];
}

// nrun fixed steps (bpl_fixed_steps in quads).
template <int N>
__device__ __forceinline__ void quad_fixed_steps(const double (&pm)[N - 1], const Coef &k,
                                                 const bool live, const int nrun, double (&x)[3],
                                                 double (&v)[3], double (&a0)[3], double (&j0)[3])
{
    const unsigned long long who = __ballot(live && nrun > 0);
    if (who == 0ull)
        return;
    const int n0 = __builtin_amdgcn_readlane(nrun, __builtin_ctzll(who));
    double w = 0.0;
    if (__all(!live || nrun == n0)) {
#pragma unroll 1
        for (int q = 0; q < n0; ++q) {
            double xc[3], vc[3], ak[3], jk[3];
            quad_step<N, false>(pm, k, x, v, a0, j0, xc, vc, ak, jk, w);
            select3(true, xc, x);
            select3(true, vc, v);
            select3(true, ak, a0);
            select3(true, jk, j0);
        }
        return;
    }
    int q = 0;
#pragma unroll 1
    do {
        const bool act = q < nrun;
        double xc[3], vc[3], ak[3], jk[3];
        quad_step<N, false>(pm, k, x, v, a0, j0, xc, vc, ak, jk, w);
        select3(act, xc, x);
        select3(act, vc, v);
        select3(act, ak, a0);
        select3(act, jk, j0);
        ++q;
    } while (__any(q < nrun));
}

template <int N, int K>
__device__ __forceinline__ void quad_masses(const double mi, double (&pm)[N - 1])
{
    pm[K] = quad_read<quad_partner<N>(K)>(mi);
    if constexpr (K + 1 < N - 1)
        quad_masses<N, K + 1>(mi, pm);
}

constexpr int kQuadSystems = 16;   // systems per wavefront

// SOLO: of the batch io instead of the bucket, with the evaluation it starts
// from.
template <int N, bool ADV, bool SOLO = false>
__device__ __forceinline__ void quad_run(const Bucket &B, const int first, const int count,
                                         const StepParams &P, const SoloIO &io = SoloIO())
{
    static_assert(N >= 2 && N <= 4, "a quad holds up to four bodies");
    const int lane = threadIdx.x & 63;
    const int s = lane >> 2, b = lane & 3;
    const bool valid = b < N && s < count;
    const int slot = valid ? first + s : first;
    const size_t pitch = SOLO ? 0 : B.pitch;
    // idle lanes: apart from the star, so that nothing they compute is special
    double mi = 0.0, x[3] = {(double)(2 + b), 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0};
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
    double pm[N - 1];
    quad_masses<N, 0>(mi, pm);
    if constexpr (SOLO) {
        double w = 0.0;
        quad_eval<N, false>(pm, x, v, a0, j0, w);
    }
    if constexpr (!ADV) {
        int budget = P.quantum;
#pragma unroll 1
        for (int seg = 0; seg < 2; ++seg) {
            double h = c.dt;
            const int nrun = run_segment(c, P, seg, budget, h);
            quad_fixed_steps<N>(pm, make_coef(h), live, nrun, x, v, a0, j0);
            budget -= nrun;
            run_segment_end(c, P, seg, nrun);
        }
        const int fl = quad_or<N>((b >= N || (finite3(x) && finite3(v))) ? 0 : 1);
        if (live && fl)
            c.status = ST_NONFINITE;
    } else {
        const double inv24m0 = 1.0 / (24.0 * quad_body<0>(mi));
#pragma unroll 1
        for (int q = 0; q < P.quantum; ++q) {
            double h = 0.0;
            bool last = false;
            const bool act = P.adaptive ? plan_step_adaptive(c, P, h, last)
                                        : valid && plan_step(c, P, h, last);
            if (!__any(act))
                break;
            double xc[3], vc[3], ak[3], jk[3], w = 0.0;
            quad_step<N, true>(pm, make_coef(h), x, v, a0, j0, xc, vc, ak, jk, w);
            double dtp = 0.0;
            if (P.adaptive == 1) {
                dtp = P.eta * rsqrt_nr(quad_max<N>(w));
            } else if (P.adaptive == 2) {
                const double aa = fma(ak[2], ak[2], fma(ak[1], ak[1], ak[0] * ak[0]));
                const double jj = fma(jk[2], jk[2], fma(jk[1], jk[1], jk[0] * jk[0]));
                dtp = P.eta * rsqrt_nr(quad_sum<N>(jj / aa));
            }
            select3(act, xc, x);
            select3(act, vc, v);
            select3(act, ak, a0);
            select3(act, jk, j0);
            const int fl = quad_stop_flags<N>(b, pm, mi, inv24m0, x, v, P);
            if (P.adaptive) {
                finish_step_adaptive(c, act, last, h, dtp, fl);
            } else if (act) {
                finish_step(c, P, last, h, dtp);
                if (fl)
                    c.status = status_of_flags(fl);
            }
        }
    }
    if (SOLO && live)
        solo_store(io, N, slot, b, x, v, c.status);
    if (!SOLO && live) {
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
}

// ---------------------------------------------------------------------------
// kernels: one wavefront per workgroup
// ---------------------------------------------------------------------------

template <int N, bool ADV>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(N >= 14 && !ADV ? 2 : 1)))
void k_bpl_unrolled(Bucket B, StepParams P)
{
    if constexpr (N <= 4) {
        const int first = blockIdx.x * kQuadSystems;
        quad_run<N, ADV>(B, first, min(kQuadSystems, B.count - first), P);
    } else {
        constexpr int S = 64 / N;
        const int first = blockIdx.x * S;
        int slot;
        bpl_run<N, ADV, false, true>(B, first, min(S, B.count - first), nullptr, P, slot);
    }
}

template <int N>
__global__ __launch_bounds__(64) void k_solo_quads(SoloIO io, StepParams P)
{
    const int first = blockIdx.x * kQuadSystems;
    quad_run<N, false, true>(Bucket(), first, min(kQuadSystems, io.n_sys - first), P, io);
}

}  // namespace

hipError_t launch_solo_quads(const SoloIO &io, int n, const StepParams &P, hipStream_t s)
{
    if (io.n_sys <= 0)
        return hipSuccess;
    if (P.adaptive || P.stop_rules)
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)((io.n_sys + kQuadSystems - 1) / kQuadSystems));
    switch (n) {
    case 2: hipLaunchKernelGGL(k_solo_quads<2>, grid, dim3(64), 0, s, io, P); break;
    case 3: hipLaunchKernelGGL(k_solo_quads<3>, grid, dim3(64), 0, s, io, P); break;
    case 4: hipLaunchKernelGGL(k_solo_quads<4>, grid, dim3(64), 0, s, io, P); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int unrolled_tiles(const Bucket &B)
{
    const int S = B.n <= 4 ? kQuadSystems : 64 / B.n;
    return (B.count + S - 1) / S;
}

hipError_t launch_unrolled(const Bucket &B, const StepParams &P, hipStream_t s)
{
    if (B.count == 0)
        return hipSuccess;
    const bool adv = P.adaptive || P.stop_rules;
    const dim3 grid((unsigned)unrolled_tiles(B));
#define FB_L(NN)                                                                           \
    case NN:                                                                               \
        if (adv) hipLaunchKernelGGL((k_bpl_unrolled<NN, true>), grid, dim3(64), sizeof(BplLds), s, B, P); \
        else hipLaunchKernelGGL((k_bpl_unrolled<NN, false>), grid, dim3(64), sizeof(BplLds), s, B, P);    \
        break
    switch (B.n) {
        FB_L(2); FB_L(3); FB_L(4); FB_L(5); FB_L(6); FB_L(7); FB_L(8); FB_L(9); FB_L(10);
        FB_L(11); FB_L(12); FB_L(13); FB_L(14); FB_L(15); FB_L(16);
    default: return hipErrorInvalidValue;
    }
#undef FB_L
    return hipGetLastError();
}

}  // namespace fb
