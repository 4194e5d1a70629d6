// fb_rkck.hip -- Runge-Kutta Cash-Karp 4(5), Sections 2.2.2 and 4.3.2.
#include "fb_bpl.h"

namespace fb {
namespace {

// The embedded pair of Cash & Karp (ACM TOMS 16, 1990) on y = (x, v),
// y' = (v, a(x)): six stages, each one acceleration evaluation (Eq. 1,
// planets in ascending order, the star last).  The step advances with the
// fifth-order weights; the error estimate is the difference from the
// fourth-order weights.  Adaptive control: with X and V
// the largest |x_i| and |v_i| of the system at the step's start,
// E = max_i max(|dx_i| / (eps X), |dv_i| / (eps V)); E <= 1 accepts and
// proposes h min(5, max(0.2, 0.9 E^(-1/5))) (a step shortened onto t_end
// leaves the proposal as it was); E > 1 rejects (state and time unchanged)
// and retries with h max(0.1, 0.9 E^(-1/4)).
struct RkTableau {
    // coupling coefficients a[stage][j], j < stage
    static constexpr double a[6][5] = {
        {0, 0, 0, 0, 0},
        {1.0 / 5.0, 0, 0, 0, 0},
        {3.0 / 40.0, 9.0 / 40.0, 0, 0, 0},
        {3.0 / 10.0, -9.0 / 10.0, 6.0 / 5.0, 0, 0},
        {-11.0 / 54.0, 5.0 / 2.0, -70.0 / 27.0, 35.0 / 27.0, 0},
        {1631.0 / 55296.0, 175.0 / 512.0, 575.0 / 13824.0, 44275.0 / 110592.0, 253.0 / 4096.0}};
    // fifth-order weights, and fifth- minus fourth-order weights
    static constexpr double b[6] = {37.0 / 378.0, 0.0, 250.0 / 621.0, 125.0 / 594.0, 0.0,
                                    512.0 / 1771.0};
    static constexpr double e[6] = {37.0 / 378.0 - 2825.0 / 27648.0, 0.0,
                                    250.0 / 621.0 - 18575.0 / 48384.0,
                                    125.0 / 594.0 - 13525.0 / 55296.0, -277.0 / 14336.0,
                                    512.0 / 1771.0 - 1.0 / 4.0};

    // The stages by accelerations alone.  The velocity derivative of stage j is
    // v + h sum_l a[j][l] A_l, so stage s's position and the step's end are
    //   x + h c[s] v + h^2 sum_l aa(s, l) A_l,   x + h v + h^2 sum_l ba(l) A_l
    // with c[s] = sum_j a[s][j] and the products below: no velocity
    // derivatives to keep, and half the sums.
    static constexpr double c[6] = {0.0, 1.0 / 5.0, 3.0 / 10.0, 3.0 / 5.0, 1.0, 7.0 / 8.0};
    static constexpr double aa(int s, int l)
    {
        double t = 0.0;
        for (int j = l + 1; j < s; ++j)
            t += a[s][j] * a[j][l];
        return t;
    }
    static constexpr double ba(int l)
    {
        double t = 0.0;
        for (int j = l + 1; j < 6; ++j)
            t += b[j] * a[j][l];
        return t;
    }
};

// Sum over l = L..S-1 of aa(S, l) A_l[c] (S < 6) or ba(l) A_l[c] (S = 6), the
// first term a product; stage 1 has no term.
template <int S, int L>
__device__ __forceinline__ double rk_sum(const double (&kv)[6][3], const int c, const double t)
{
    constexpr double k = S < 6 ? RkTableau::aa(S, L) : RkTableau::ba(L);
    const double u = L == 0 ? k * kv[L][c] : fma(k, kv[L][c], t);
    if constexpr (L + 2 < (S < 6 ? S : 6))
        return rk_sum<S, L + 1>(kv, c, u);
    else
        return u;
}

// Component c of stage S's position of one body.
template <int S>
__device__ __forceinline__ double rk_stage(const double (&kv)[6][3], const int c, const double x,
                                           const double v, const double h)
{
    const double y = fma(h * RkTableau::c[S], v, x);
    if constexpr (S == 1)
        return y;
    else
        return fma(h * h, rk_sum<S, 0>(kv, c, 0.0), y);
}

// One body's state at the end of the step (fifth-order weights; those of
// stages 1 and 4 are zero).
__device__ __forceinline__ void rk_finish(const double (&kv)[6][3], const double h, double (&x)[3],
                                          double (&v)[3])
{
    using T = RkTableau;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        x[c] = fma(h, fma(h, rk_sum<6, 0>(kv, c, 0.0), v[c]), x[c]);
        const double sv = fma(T::b[5], kv[5][c], fma(T::b[3], kv[3][c],
                                                     fma(T::b[2], kv[2][c], T::b[0] * kv[0][c])));
        v[c] = fma(h, sv, v[c]);
    }
}

// ---------------------------------------------------------------------------
// system per lane, fixed steps
// ---------------------------------------------------------------------------

// Accelerations (Eq. 1) of every body at positions x, each pair once.
template <int N>
__device__ __forceinline__ void rk_spl_accel(const double (&m)[N], const double (&x)[N][3],
                                             double (&kv)[N][6][3], const int st)
{
    double a[N][3];
#pragma unroll
    for (int b = 0; b < N; ++b)
        a[b][0] = a[b][1] = a[b][2] = 0.0;
    auto pair = [&](const int i, const int j) {
        const double rx = x[j][0] - x[i][0], ry = x[j][1] - x[i][1], rz = x[j][2] - x[i][2];
        const double ri = rsqrt_nr(fma(rz, rz, fma(ry, ry, rx * rx)));
        const double ri3 = ri * ri * ri;
        const double mj3 = m[j] * ri3, mi3 = m[i] * ri3;
        a[i][0] = fma(mj3, rx, a[i][0]);
        a[i][1] = fma(mj3, ry, a[i][1]);
        a[i][2] = fma(mj3, rz, a[i][2]);
        a[j][0] = fma(-mi3, rx, a[j][0]);
        a[j][1] = fma(-mi3, ry, a[j][1]);
        a[j][2] = fma(-mi3, rz, a[j][2]);
    };
#pragma unroll
    for (int i = 1; i < N; ++i)
#pragma unroll
        for (int j = i + 1; j < N; ++j)
            pair(i, j);
#pragma unroll
    for (int j = 1; j < N; ++j)
        pair(0, j);
#pragma unroll
    for (int b = 0; b < N; ++b)
#pragma unroll
        for (int c = 0; c < 3; ++c)
            kv[b][st][c] = a[b][c];
}

// Accelerations of stage S (0: kv[.][0] must be filled) from those before it.
template <int N, int S>
__device__ __forceinline__ void rk_spl_stage(const double (&m)[N], const double (&x)[N][3],
                                             const double (&v)[N][3], double (&kv)[N][6][3],
                                             const double h)
{
    double xs[N][3];
#pragma unroll
    for (int b = 0; b < N; ++b)
#pragma unroll
        for (int c = 0; c < 3; ++c)
            xs[b][c] = rk_stage<S>(kv[b], c, x[b][c], v[b][c], h);
    rk_spl_accel<N>(m, xs, kv, S);
}

template <int N>
__device__ __forceinline__ void rk_spl_step(const double (&m)[N], double (&x)[N][3],
                                            double (&v)[N][3], const double h)
{
    double kv[N][6][3];
    rk_spl_accel<N>(m, x, kv, 0);
    rk_spl_stage<N, 1>(m, x, v, kv, h);
    rk_spl_stage<N, 2>(m, x, v, kv, h);
    rk_spl_stage<N, 3>(m, x, v, kv, h);
    rk_spl_stage<N, 4>(m, x, v, kv, h);
    rk_spl_stage<N, 5>(m, x, v, kv, h);
#pragma unroll
    for (int b = 0; b < N; ++b)
        rk_finish(kv[b], h, x[b], v[b]);
}

template <int N>
__device__ __forceinline__ void rk_spl_run(const Bucket &B, const int slot, const StepParams &P)
{
    Clock c = load_clock(B, slot);
    if (c.status != ST_ACTIVE)
        return;
    const size_t pitch = B.pitch;
    double m[N], x[N][3], v[N][3];
#pragma unroll
    for (int b = 0; b < N; ++b) {
        m[b] = B.st[(R_M * N + b) * pitch + slot];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            x[b][k] = B.st[((R_X + k) * N + b) * pitch + slot];
            v[b][k] = B.st[((R_V + k) * N + b) * pitch + slot];
        }
    }
    int budget = P.quantum;
#pragma unroll 1
    for (int seg = 0; seg < 2; ++seg) {
        double h = c.dt;
        const int nrun = run_segment(c, P, seg, budget, h);
#pragma unroll 1
        for (int q = 0; q < nrun; ++q)
            rk_spl_step<N>(m, x, v, h);
        budget -= nrun;
        run_segment_end(c, P, seg, nrun);
    }
    bool fin = true;
#pragma unroll
    for (int b = 0; b < N; ++b)
        fin = fin && finite3(x[b]) && finite3(v[b]);
    if (!fin)
        c.status = ST_NONFINITE;
#pragma unroll
    for (int b = 0; b < N; ++b)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            B.st[((R_X + k) * N + b) * pitch + slot] = x[b][k];
            B.st[((R_V + k) * N + b) * pitch + slot] = v[b][k];
        }
    store_clock(B, slot, c);
}

// Fixed steps, one system per lane, each pair once and nothing exchanged.
// Bound by FP64 issue (675 instructions a step of three bodies; unspilled to
// n = 4, with AGPR moves to 6; at 7 and 8 the stages' accelerations spill to
// memory, 1.6 times slower than body per lane).  131072 x 3 bodies, 1000
// steps: 3.19 ms (4.1e10 system-steps/s), body per lane 6.1 ms, and 8.43 ms
// body per lane with the stages' velocity derivatives kept.
template <int N>
__global__ __launch_bounds__(64) void k_rkck_spl(Bucket B, StepParams P)
{
    const int slot = blockIdx.x * blockDim.x + threadIdx.x;
    if (slot < B.count)
        rk_spl_run<N>(B, slot, P);
}

// ---------------------------------------------------------------------------
// body per lane of a wavefront
// ---------------------------------------------------------------------------

// Acceleration of this lane's body (Eq. 1) from its partners' positions, read
// from the wavefront's LDS slice with the mass beside z.
template <int N>
__device__ __forceinline__ void rk_accel(BplLds &L, const int lane, const int (&pidx)[N - 1],
                                         const double mi, const double (&xi)[3], double (&acc)[3])
{
    L.xy[lane] = make_double2(xi[0], xi[1]);
    L.zvx[lane] = make_double2(xi[2], mi);
    wave_sync();
    acc[0] = acc[1] = acc[2] = 0.0;
#pragma unroll
    for (int k = 0; k < N - 1; ++k) {
        const double2 p0 = L.xy[pidx[k]], p1 = L.zvx[pidx[k]];
        const double rx = p0.x - xi[0], ry = p0.y - xi[1], rz = p1.x - xi[2];
        const double ri = rsqrt_nr(fma(rz, rz, fma(ry, ry, rx * rx)));
        const double mr3 = p1.y * (ri * ri * ri);
        acc[0] = fma(mr3, rx, acc[0]);
        acc[1] = fma(mr3, ry, acc[1]);
        acc[2] = fma(mr3, rz, acc[2]);
    }
    wave_sync();
}

template <int N, int S>
__device__ __forceinline__ void rk_bpl_stage(BplLds &L, const int lane, const int (&pidx)[N - 1],
                                             const double mi, const double (&x)[3],
                                             const double (&v)[3], double (&kv)[6][3],
                                             const double h)
{
    double xs[3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
        xs[c] = rk_stage<S>(kv, c, x[c], v[c], h);
    rk_accel<N>(L, lane, pidx, mi, xs, kv[S]);
}

// One fixed step of this lane's body (the arithmetic of rk_spl_step).
template <int N>
__device__ __forceinline__ void rk_bpl_step(BplLds &L, const int lane, const int (&pidx)[N - 1],
                                            const double mi, double (&x)[3], double (&v)[3],
                                            const double h)
{
    double kv[6][3];
    rk_accel<N>(L, lane, pidx, mi, x, kv[0]);
    rk_bpl_stage<N, 1>(L, lane, pidx, mi, x, v, kv, h);
    rk_bpl_stage<N, 2>(L, lane, pidx, mi, x, v, kv, h);
    rk_bpl_stage<N, 3>(L, lane, pidx, mi, x, v, kv, h);
    rk_bpl_stage<N, 4>(L, lane, pidx, mi, x, v, kv, h);
    rk_bpl_stage<N, 5>(L, lane, pidx, mi, x, v, kv, h);
    rk_finish(kv, h, x, v);
}

__device__ __forceinline__ double norm2(const double (&p)[3])
{
    return fma(p[2], p[2], fma(p[1], p[1], p[0] * p[0]));
}

// E^(-1/5) to rounding, for E in [1e-5, 1e5] (elsewhere the step factor is at
// its limits): an estimate from the FP32 logarithm and exponential and one
// third-order step of the binomial series of (1 - e)^(-1/5), e = 1 - E y^5.
__device__ __forceinline__ double inv_fifth_root(const double E)
{
    const double y = (double)__builtin_amdgcn_exp2f(-0.2f * __builtin_amdgcn_logf((float)E));
    const double y2 = y * y;
    const double e = fma(-E * y, y2 * y2, 1.0);
    return fma(y * e, fma(3.0 / 25.0, e, 1.0 / 5.0), y);
}

// One trial step of this lane's body: the fifth-order result and the error
// estimate.
template <int N>
__device__ __forceinline__ void rk_bpl_trial(BplLds &L, const int lane, const int (&pidx)[N - 1],
                                             const double mi, const double (&x)[3],
                                             const double (&v)[3], const double h,
                                             double (&x5)[3], double (&v5)[3], double (&ex)[3],
                                             double (&ev)[3])
{
    using T = RkTableau;
    double kx[6][3], kv[6][3];
#pragma unroll
    for (int st = 0; st < 6; ++st) {
        double xs[3];
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            double dx = 0.0, dv = 0.0;
#pragma unroll
            for (int j = 0; j < st; ++j) {
                dx = fma(T::a[st][j], kx[j][cc], dx);
                dv = fma(T::a[st][j], kv[j][cc], dv);
            }
            xs[cc] = fma(h, dx, x[cc]);
            kx[st][cc] = fma(h, dv, v[cc]);
        }
        rk_accel<N>(L, lane, pidx, mi, xs, kv[st]);
    }
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) {
        double sx = 0.0, sv = 0.0, ux = 0.0, uv = 0.0;
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            if (j != 1 && j != 4) {   // the weights of stages 1 and 4 are zero
                sx = fma(T::b[j], kx[j][cc], sx);
                sv = fma(T::b[j], kv[j][cc], sv);
            }
            if (j != 1) {
                ux = fma(T::e[j], kx[j][cc], ux);
                uv = fma(T::e[j], kv[j][cc], uv);
            }
        }
        x5[cc] = fma(h, sx, x[cc]);
        v5[cc] = fma(h, sv, v[cc]);
        ex[cc] = h * ux;
        ev[cc] = h * uv;
    }
}

// The error norm E of the lane's system.  Square root and division round
// monotonically, so the maxima are taken of the squares, in one exchange.
template <int N>
__device__ __forceinline__ double rk_error(BplLds &L, const int lane, const int s,
                                           const double (&x)[3], const double (&v)[3],
                                           const double (&ex)[3], const double (&ev)[3],
                                           const double eps)
{
    constexpr int S = 64 / N;
    L.xy[lane] = make_double2(norm2(x), norm2(v));
    L.zvx[lane] = make_double2(norm2(ex), norm2(ev));
    wave_sync();
    double2 p = L.xy[s], q = L.zvx[s];
#pragma unroll
    for (int k = 1; k < N; ++k) {
        const double2 a = L.xy[k * S + s], b = L.zvx[k * S + s];
        p.x = fmax(p.x, a.x);
        p.y = fmax(p.y, a.y);
        q.x = fmax(q.x, b.x);
        q.y = fmax(q.y, b.y);
    }
    wave_sync();
    return fmax(sqrt(q.x) / (eps * sqrt(p.x)), sqrt(q.y) / (eps * sqrt(p.y)));
}

template <int N, bool ADV>
__device__ __forceinline__ void rk_bpl_run(const Bucket &B, const int first, const int count,
                                           const StepParams &P, const double eps)
{
    constexpr int S = 64 / N;
    BplLds &L = *reinterpret_cast<BplLds *>(wave_lds_base<sizeof(BplLds), false>());
    const int lane = threadIdx.x & 63;
    const int braw = lane / S;
    const int b = braw < N ? braw : N - 1;
    const int s = lane - braw * S;
    const bool valid = braw < N && s < count;
    const int slot = first + (valid ? s : 0);
    const size_t pitch = B.pitch;
    double mi = 0.0, x[3] = {0.0, 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0};
    Clock c{};
    c.status = ST_DONE;
    if (valid) {
        mi = B.st[(R_M * N + b) * pitch + slot];
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            x[cc] = B.st[((R_X + cc) * N + b) * pitch + slot];
            v[cc] = B.st[((R_V + cc) * N + b) * pitch + slot];
        }
        c = load_clock(B, slot);
    }
    const bool live = c.status == ST_ACTIVE;
    int pidx[N - 1];
#pragma unroll
    for (int k = 0; k < N - 1; ++k)
        pidx[k] = eval_partner<N>(k, b) * S + s;
    if constexpr (!ADV) {
        int budget = P.quantum;
#pragma unroll 1
        for (int seg = 0; seg < 2; ++seg) {
            double h = c.dt;
            const int nrun = run_segment(c, P, seg, budget, h);
            int q = 0;
            if (__any(nrun > 0))
#pragma unroll 1
                do {
                    double xn[3] = {x[0], x[1], x[2]}, vn[3] = {v[0], v[1], v[2]};
                    rk_bpl_step<N>(L, lane, pidx, mi, xn, vn, h);
                    const bool act = q < nrun;
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        x[k] = act ? xn[k] : x[k];
                        v[k] = act ? vn[k] : v[k];
                    }
                    ++q;
                } while (__any(q < nrun));
            budget -= nrun;
            run_segment_end(c, P, seg, nrun);
        }
        const int fl = sys_or_flags<N>(s, (finite3(x) && finite3(v)) ? 0 : 1);
        if (fl)
            c.status = ST_NONFINITE;
    } else {
#pragma unroll 1
        for (int q = 0; q < P.quantum; ++q) {
            double h = 0.0;
            bool last = false;
            const bool act = valid && plan_step(c, P, h, last);
            if (!__any(act))
                break;
            if (!act)
                h = 0.0;
            double x5[3], v5[3], ex[3], ev[3];
            rk_bpl_trial<N>(L, lane, pidx, mi, x, v, h, x5, v5, ex, ev);
            const double E = rk_error<N>(L, lane, s, x, v, ex, ev, eps);
            const bool accept = E <= 1.0;
            if (act && !accept) {
                if (!__builtin_isfinite(E))
                    c.status = ST_NONFINITE;
                else
                    c.dtn = h * fmax(0.1, 0.9 * pow(E, -0.25));
            }
            const double Ec = fmin(1e5, fmax(1e-5, E));
            const double f = 0.9 * inv_fifth_root(Ec);
            const double dtp = last ? c.dtn : h * (E > 0.0 ? fmin(5.0, fmax(0.2, f)) : 5.0);
            if (act && accept) {
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) {
                    x[cc] = x5[cc];
                    v[cc] = v5[cc];
                }
                finish_step(c, P, last, h, dtp);
            }
        }
    }
    if (live) {
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            B.st[((R_X + cc) * N + b) * pitch + slot] = x[cc];
            B.st[((R_V + cc) * N + b) * pitch + slot] = v[cc];
        }
        if (b == 0)
            store_clock(B, slot, c);
    }
}

// Every body-per-lane bucket of an ensemble in one launch, largest n first;
// a wavefront takes one tile.  Partner slots in registers, unrolled partner
// loops, masses beside z, the adaptive error norm's four maxima in one
// exchange (three, one after another, before) and no pow for the step factor.
// 9999 x 5 bodies, adaptive to one orbit: 976 -> 545 us; 100 x 5 bodies, 200
// fixed steps: 633 -> 371 us.
template <bool ADV>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2)))
void k_rkck_bpl(BucketSet set, StepParams P, double eps)
{
    const int tile = blockIdx.x;
    int k = 0;
    while (k < set.count && tile >= set.first[k + 1])
        ++k;
    if (k >= set.count)
        return;
    const Bucket B = set.b[k];
    const int S = 64 / B.n;
    const int first = (tile - set.first[k]) * S;
    const int count = min(S, B.count - first);
    switch (B.n) {
#define FB_C(NN) case NN: rk_bpl_run<NN, ADV>(B, first, count, P, eps); break;
        FB_C(2) FB_C(3) FB_C(4) FB_C(5) FB_C(6) FB_C(7) FB_C(8) FB_C(9) FB_C(10) FB_C(11)
        FB_C(12) FB_C(13) FB_C(14) FB_C(15) FB_C(16)
#undef FB_C
    default: break;
    }
}

// ---------------------------------------------------------------------------
// Runge-Kutta Cash-Karp for large systems (n > 16): one body per lane across
// a workgroup
// ---------------------------------------------------------------------------
// The stages, weights and error control of k_rkck_bpl in the large-n
// layout.  Each stage's positions go to one of two LDS copies in turn, so a
// stage costs one workgroup barrier; a body's own term is an exact zero
// through the r^2 floor, so every lane runs the same partner loop (planets in
// ascending order, the star last).

// Acceleration of this lane's body (Eq. 1) at the stage positions xs,
// published in copy cp.
__device__ __forceinline__ void large_rk_accel(const LargeView &V, const int T, const int cp,
                                               const LargeLane &l, const int n,
                                               const double (&xs)[3], double (&acc)[3])
{
    double2 *xy = V.xy + cp * T, *zvx = V.zvx + cp * T;
    xy[l.tid] = make_double2(xs[0], xs[1]);
    zvx[l.tid] = make_double2(xs[2], 0.0);
    __syncthreads();
    acc[0] = acc[1] = acc[2] = 0.0;
    if (!l.valid)
        return;
    for (int k = 1; k <= n; ++k) {
        const int j = k < n ? k : 0;   // planets 1..n-1, then the star
        const double2 p0 = xy[l.base + j], p1 = zvx[l.base + j];
        const double rx = p0.x - xs[0], ry = p0.y - xs[1], rz = p1.x - xs[2];
        const double ri = rsqrt_nr(fmax(fma(rz, rz, fma(ry, ry, rx * rx)), kLargeMinR2));
        const double mr3 = V.m[l.base + j] * (ri * ri * ri);
        acc[0] = fma(mr3, rx, acc[0]);
        acc[1] = fma(mr3, ry, acc[1]);
        acc[2] = fma(mr3, rz, acc[2]);
    }
}

// Maximum of one value per lane over the lane's system, to every valid lane.
__device__ __forceinline__ double large_sys_max(const LargeView &V, const LargeLane &l,
                                                const int n, const double v)
{
    V.red[l.tid] = v;
    __syncthreads();
    double r = 0.0;
    if (l.valid) {
        r = V.red[l.base];
        for (int b = 1; b < n; ++b)
            r = fmax(r, V.red[l.base + b]);
    }
    __syncthreads();
    return r;
}

template <bool ADV>
__global__ __launch_bounds__(kLargeMaxLanes) void k_plain_rkck_large(Bucket B, StepParams P,
                                                                     double eps, int S)
{
    using Tb = RkTableau;
    const int T = blockDim.x, n = B.n;
    const LargeView V = large_view(T);
    const LargeLane l = large_lane(B, S);
    const size_t pitch = B.pitch;
    double mi = 0.0, x[3] = {0.0, 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0};
    Clock c;
    c.status = ST_DONE;
    if (l.valid) {
        mi = B.st[(R_M * n + l.b) * pitch + l.slot];
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            x[cc] = B.st[((R_X + cc) * n + l.b) * pitch + l.slot];
            v[cc] = B.st[((R_V + cc) * n + l.b) * pitch + l.slot];
        }
        c = load_clock(B, l.slot);
    }
    V.m[l.tid] = mi;   // ordered before any read by the loop's first barrier
    int cp = 0;
    for (int q = 0; q < P.quantum; ++q) {
        double h = 0.0;
        bool last = false;
        const bool act = l.valid && plan_step(c, P, h, last);
        if (!__syncthreads_or(act))
            break;
        if (!act)
            h = 0.0;
        double kx[6][3], kv[6][3];
#pragma unroll
        for (int st = 0; st < 6; ++st) {
            double xs[3];
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                double dx = 0.0, dv = 0.0;
#pragma unroll
                for (int j = 0; j < st; ++j) {
                    dx = fma(Tb::a[st][j], kx[j][cc], dx);
                    dv = fma(Tb::a[st][j], kv[j][cc], dv);
                }
                xs[cc] = fma(h, dx, x[cc]);
                kx[st][cc] = fma(h, dv, v[cc]);
            }
            large_rk_accel(V, T, cp, l, n, xs, kv[st]);
            cp ^= 1;
        }
        double x5[3], v5[3], ex[3], ev[3];
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            double sx = 0.0, sv = 0.0, ux = 0.0, uv = 0.0;
#pragma unroll
            for (int j = 0; j < 6; ++j) {
                sx = fma(Tb::b[j], kx[j][cc], sx);
                sv = fma(Tb::b[j], kv[j][cc], sv);
                ux = fma(Tb::e[j], kx[j][cc], ux);
                uv = fma(Tb::e[j], kv[j][cc], uv);
            }
            x5[cc] = fma(h, sx, x[cc]);
            v5[cc] = fma(h, sv, v[cc]);
            ex[cc] = h * ux;
            ev[cc] = h * uv;
        }
        bool accept = true;
        double dtp = 0.0;
        if (ADV) {
            const double X = large_sys_max(V, l, n, sqrt(norm2(x)));
            const double Vm = large_sys_max(V, l, n, sqrt(norm2(v)));
            const double E = large_sys_max(V, l, n, fmax(sqrt(norm2(ex)) / (eps * X), sqrt(norm2(ev)) / (eps * Vm)));
            accept = E <= 1.0;
            if (act && !accept) {
                if (!__builtin_isfinite(E))
                    c.status = ST_NONFINITE;
                else
                    c.dtn = h * fmax(0.1, 0.9 * pow(E, -0.25));
            }
            dtp = last ? c.dtn : h * (E > 0.0 ? fmin(5.0, fmax(0.2, 0.9 * pow(E, -0.2))) : 5.0);
        }
        if (act && accept) {
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                x[cc] = x5[cc];
                v[cc] = v5[cc];
            }
            finish_step(c, P, last, h, dtp);
        }
    }
    const int bad = ADV ? 0 : large_sys_or(V, l, n, (l.valid && !(finite3(x) && finite3(v))) ? 1 : 0);
    if (!l.valid)
        return;
    if (bad)
        c.status = ST_NONFINITE;
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) {
        B.st[((R_X + cc) * n + l.b) * pitch + l.slot] = x[cc];
        B.st[((R_V + cc) * n + l.b) * pitch + l.slot] = v[cc];
    }
    if (l.b == 0)
        store_clock(B, l.slot, c);
}

}  // namespace

hipError_t launch_rkck_spl(const Bucket &B, const StepParams &P, hipStream_t s)
{
    if (B.count == 0)
        return hipSuccess;
    const dim3 grid = grid_for(B.count, 64);
#define FB_L(NN) case NN: hipLaunchKernelGGL(k_rkck_spl<NN>, grid, dim3(64), 0, s, B, P); break
    static_assert(kMaxRkckSpl == 6, "the switch covers n = 2..kMaxRkckSpl");
    switch (B.n) {
        FB_L(2); FB_L(3); FB_L(4); FB_L(5); FB_L(6);
    default: return hipErrorInvalidValue;
    }
#undef FB_L
    return hipGetLastError();
}

hipError_t launch_rkck_bpl(const BucketSet &set, const StepParams &P, double eps, hipStream_t s)
{
    const int tiles = set.count > 0 ? set.first[set.count] : 0;
    if (tiles == 0)
        return hipSuccess;
    if (eps > 0.0)
        hipLaunchKernelGGL(k_rkck_bpl<true>, dim3(tiles), dim3(64), sizeof(BplLds), s, set, P, eps);
    else
        hipLaunchKernelGGL(k_rkck_bpl<false>, dim3(tiles), dim3(64), sizeof(BplLds), s, set, P, eps);
    return hipGetLastError();
}

hipError_t launch_rkck_large(const Bucket &B, const StepParams &P, double eps, hipStream_t s)
{
    if (B.count == 0)
        return hipSuccess;
    dim3 grid;
    int T, S;
    if (!large_launch(B, grid, T, S))
        return hipErrorInvalidValue;
    if (P.adaptive)
        hipLaunchKernelGGL(k_plain_rkck_large<true>, grid, dim3(T), large_lds_bytes(T), s, B, P, eps, S);
    else
        hipLaunchKernelGGL(k_plain_rkck_large<false>, grid, dim3(T), large_lds_bytes(T), s, B, P, eps, S);
    return hipGetLastError();
}

}  // namespace fb
