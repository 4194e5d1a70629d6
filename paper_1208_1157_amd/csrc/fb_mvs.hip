// fb_mvs.hip -- the step kernels of the mixed-variable symplectic integrator
// (Sections 2.2.3 and 4.3.3): democratic heliocentric drifts and kicks around
// one Kepler drift per planet.  The conversions to and from a bucket's MVS
// form and its read-back are in fb_kernels.hip.
#include "fb_device.h"

#include <climits>

namespace fb {
namespace {

// (r, v) advanced by dt on its Kepler orbit about mu.  The change x of the
// eccentric anomaly solves Kepler's equation in difference form,
//   n dt = x - (1 - r0/a) sin x + (r.v / sqrt(mu a)) (1 - cos x),
// by Newton iteration from x = n dt; Lagrange's f and g functions give the
// new state.  The caller has checked 1/a > 0.  Returns false if the
// iteration does not converge in kMvsNewtonMax steps.
constexpr int kMvsNewtonMax = 50;

__device__ __forceinline__ bool kepler_drift(const double mu, double (&r)[3], double (&v)[3],
                                             const double dt)
{
    const double r2 = fma(r[2], r[2], fma(r[1], r[1], r[0] * r[0]));
    const double v2 = fma(v[2], v[2], fma(v[1], v[1], v[0] * v[0]));
    const double rv = fma(r[2], v[2], fma(r[1], v[1], r[0] * v[0]));
    const double r0 = sqrt(r2);
    const double alpha = 2.0 / r0 - v2 / mu;
    const double a = 1.0 / alpha;
    const double sqmua = sqrt(mu * a);
    const double nmot = sqmua * alpha * alpha;   // sqrt(mu / a^3)
    const double ec = 1.0 - r0 * alpha;
    const double es = rv / sqmua;
    const double M = nmot * dt;
    double x = M, s = 0.0, c = 1.0;
    bool ok = false;
    for (int it = 0; it < kMvsNewtonMax; ++it) {
        sincos(x, &s, &c);
        const double F = fma(-ec, s, x) + fma(es, 1.0 - c, -M);
        const double dF = fma(es, s, fma(-ec, c, 1.0));
        const double dx = F / dF;
        x -= dx;
        if (fabs(dx) <= 1e-15 * (1.0 + fabs(x))) {
            ok = true;
            break;
        }
    }
    if (!ok)
        return false;
    sincos(x, &s, &c);
    const double omc = 1.0 - c;
    const double f = fma(-a / r0, omc, 1.0);
    const double g = dt - (x - s) / nmot;
    const double rn = a * fma(es, s, fma(-ec, c, 1.0));
    const double fd = -sqmua * s / (rn * r0);
    const double gd = fma(-a / rn, omc, 1.0);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double rk = r[k], vk = v[k];
        r[k] = fma(f, rk, g * vk);
        v[k] = fma(fd, rk, gd * vk);
    }
    return true;
}

// Drift of every Q_i by h sum_j m_j V_j / m0 and of X by h Vc (body 0's rows).
template <int N>
__device__ __forceinline__ void mvs_drift(const double (&m)[N], double (&Q)[N][3],
                                          const double (&V)[N][3], const double inv_m0,
                                          const double h)
{
    double P[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 1; i < N; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c)
            P[c] = fma(m[i], V[i][c], P[c]);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double dq = h * P[c] * inv_m0;
#pragma unroll
        for (int i = 1; i < N; ++i)
            Q[i][c] += dq;
        Q[0][c] = fma(h, V[0][c], Q[0][c]);
    }
}

template <int N>
__device__ __forceinline__ void mvs_kick(double (&V)[N][3], const double (&acc)[N][3], const double h)
{
#pragma unroll
    for (int i = 1; i < N; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c)
            V[i][c] = fma(h, acc[i][c], V[i][c]);
}

// One MVS step of h.  Returns ST_ACTIVE, or ST_UNBOUND when a planet's
// heliocentric orbit is not bound (the half drift and kick are undone, so
// the state is the step's start up to rounding) or Kepler's equation does not
// converge (state of the planets drifted so far).
template <int N>
__device__ __forceinline__ int mvs_step(const double (&m)[N], double (&Q)[N][3], double (&V)[N][3],
                                        double (&acc)[N][3], const double inv_m0, const double h)
{
    const double hh = 0.5 * h;
    mvs_drift<N>(m, Q, V, inv_m0, hh);
    mvs_kick<N>(V, acc, hh);
    bool bound = true;
#pragma unroll
    for (int i = 1; i < N; ++i) {
        const double r2 = fma(Q[i][2], Q[i][2], fma(Q[i][1], Q[i][1], Q[i][0] * Q[i][0]));
        const double v2 = fma(V[i][2], V[i][2], fma(V[i][1], V[i][1], V[i][0] * V[i][0]));
        bound = bound && (2.0 / sqrt(r2) - v2 / m[0] > 0.0);
    }
    if (!bound) {
        mvs_kick<N>(V, acc, -hh);
        mvs_drift<N>(m, Q, V, inv_m0, -hh);
        return ST_UNBOUND;
    }
#pragma unroll
    for (int i = 1; i < N; ++i)
        if (!kepler_drift(m[0], Q[i], V[i], h))
            return ST_UNBOUND;
    mvs_acc<N>(m, Q, acc);
    mvs_kick<N>(V, acc, hh);
    mvs_drift<N>(m, Q, V, inv_m0, hh);
    return ST_ACTIVE;
}

// Fixed-step MVS integration of one system per lane for at most P.quantum
// steps: the run's whole steps, then the shortened final step if one is due
// (the clock logic of the Hermite kernels).
template <int N>
__global__ __launch_bounds__(256) void k_plain_mvs(Bucket B, StepParams P)
{
    const int slot = blockIdx.x * blockDim.x + threadIdx.x;
    if (slot >= B.count)
        return;
    Clock c = load_clock(B, slot);
    if (c.status != ST_ACTIVE)
        return;
    double m[N], Q[N][3], V[N][3], acc[N][3];
    load_rows<N>(B, slot, m, Q, V, acc, true);
    const double inv_m0 = 1.0 / m[0];
    int budget = P.quantum;
#pragma unroll 1
    for (int seg = 0; seg < 2 && c.status == ST_ACTIVE && budget > 0; ++seg) {
        long long cnt = 0;
        double h = c.dt;
        if (seg == 0) {
            cnt = c.nfull - c.k;
            cnt = cnt < 0 ? 0 : cnt;
        } else {
            const double rem = c.t_end - c.t;
            if (rem * c.dt > 1e-9 * c.dt * c.dt) {
                cnt = 1;
                h = rem;
            } else {
                c.t = c.t_end;
                c.status = ST_DONE;
            }
        }
        cnt = min(cnt, (long long)budget);
        cnt = min(cnt, P.max_steps - c.steps);
        const int nrun = cnt > 0 ? (int)cnt : 0;
        int done = 0;
#pragma unroll 1
        for (; done < nrun; ++done) {
            const int st = mvs_step<N>(m, Q, V, acc, inv_m0, h);
            if (st != ST_ACTIVE) {
                c.status = st;
                break;
            }
        }
        budget -= done;
        c.steps += done;
        if (seg == 0) {
            c.k += done;
            if (done > 0)
                c.t = fma((double)c.k, c.dt, c.t0);
            if (c.status == ST_ACTIVE && c.k >= c.nfull) {
                const double rem = c.t_end - c.t;
                if (!(rem * c.dt > 1e-9 * c.dt * c.dt)) {
                    c.t = c.t_end;
                    c.status = ST_DONE;
                }
            }
        } else if (done > 0 && c.status == ST_ACTIVE) {
            c.t = c.t_end;
            c.status = ST_DONE;
        }
        if (c.status == ST_ACTIVE && c.steps >= P.max_steps)
            c.status = ST_MAXSTEPS;
    }
    bool fin = true;
#pragma unroll
    for (int b = 0; b < N; ++b)
        fin = fin && finite3(Q[b]) && finite3(V[b]);
    if (!fin)
        c.status = ST_NONFINITE;
    store_rows<N>(B, slot, Q, V, acc, true);
    store_clock(B, slot, c);
}

// Fixed-step MVS integration, one body per lane, for at most P.quantum steps
// (the clock of the Hermite kernels; the steps of mvs_step, with the
// outcomes of a system predicating its updates).  WAVES is the waves per
// SIMD the register allocator targets: 2 (unspilled) for systems of up to 16
// bodies, 4 (a few VGPRs spilled, twice the waves to hide the Kepler
// solver's latency) for larger ones, where it measured 16-23% faster.
template <int WAVES>
__global__ __launch_bounds__(kLargeMaxLanes) __attribute__((amdgpu_waves_per_eu(WAVES)))
void k_plain_mvs_large(Bucket B, StepParams P, int S)
{
    const int T = blockDim.x, n = B.n;
    const LargeView V = large_view(T);
    const LargeLane l = large_lane(B, S);
    const bool planet = l.b > 0;
    double mi, Q[3], W[3], acc[3];
    large_load_rows(B, l, mi, Q, W, acc);
    V.m[l.tid] = mi;
    Clock c;
    c.status = ST_DONE;
    if (l.valid)
        c = load_clock(B, l.slot);
    __syncthreads();
    const double m0 = l.valid ? V.m[l.base] : 1.0;
    const double inv_m0 = 1.0 / m0;
    // drift of Q (planets) by h sum_j m_j V_j / m0 and of X (star) by h Vc
    auto drift = [&](const bool on, const double h) {
        double Pm[3], unused[3];
        large_sys_wsum3(V, T, l, n, 1, mi, W, Pm, unused);
        if (!on)
            return;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (planet)
                Q[k] += h * Pm[k] * inv_m0;
            else
                Q[k] = fma(h, W[k], Q[k]);
        }
    };
    for (int q = 0; q < P.quantum; ++q) {
        double h = 0.0;
        bool last = false;
        const bool act = l.valid && plan_step(c, P, h, last);
        if (!__syncthreads_or(act))
            break;
        const double hh = 0.5 * h;
        drift(act, hh);
        if (act && planet)
#pragma unroll
            for (int k = 0; k < 3; ++k)
                W[k] = fma(hh, acc[k], W[k]);
        int unbound = 0;
        if (act && planet) {
            const double r2 = fma(Q[2], Q[2], fma(Q[1], Q[1], Q[0] * Q[0]));
            const double v2 = fma(W[2], W[2], fma(W[1], W[1], W[0] * W[0]));
            unbound = (2.0 / sqrt(r2) - v2 / m0 > 0.0) ? 0 : 1;
        }
        const int unbound_sys = large_sys_or(V, l, n, unbound);   // every lane: barriers inside
        const bool undo = act && unbound_sys;
        if (undo && planet)
#pragma unroll
            for (int k = 0; k < 3; ++k)
                W[k] = fma(-hh, acc[k], W[k]);
        drift(undo, -hh);
        const bool go = act && !undo;
        const int kfail = (go && planet && !kepler_drift(m0, Q, W, h)) ? 1 : 0;
        const int kfail_sys = large_sys_or(V, l, n, kfail);       // every lane: barriers inside
        const bool failed = go && kfail_sys;
        const bool ok = go && !failed;
        double an[3];
        large_mvs_acc(V, l, n, Q, an);
        if (ok && planet)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                acc[k] = an[k];
                W[k] = fma(hh, acc[k], W[k]);
            }
        drift(ok, hh);
        if (ok)
            finish_step(c, P, last, h, 0.0);
        if (undo || failed)
            c.status = ST_UNBOUND;
    }
    const int bad = large_sys_or(V, l, n, (l.valid && !(finite3(Q) && finite3(W))) ? 1 : 0);
    if (!l.valid)
        return;
    if (bad)
        c.status = ST_NONFINITE;
    large_store_rows(B, l, Q, W, acc, true);
    if (l.b == 0)
        store_clock(B, l.slot, c);
}

}  // namespace

#define FB_SWITCH_MVS(n, MACRO)                                                         \
    switch (n) {                                                                        \
    case 2: MACRO(2); break;  case 3: MACRO(3); break;  case 4: MACRO(4); break;        \
    case 5: MACRO(5); break;  case 6: MACRO(6); break;  case 7: MACRO(7); break;        \
    case 8: MACRO(8); break;                                                            \
    default: return hipErrorInvalidValue;                                               \
    }

hipError_t launch_plain_mvs(const Bucket &B, int mapping, int waves_per_group, const StepParams &P,
                            hipStream_t s)
{
    if (B.count == 0)
        return hipSuccess;
    if (B.n > kMaxMvsBodies || mapping != MAP_SPL) {
        dim3 lgrid;
        int T, S;
        if (!large_launch(B, 1, lgrid, T, S))
            return hipErrorInvalidValue;
        if (B.n > kMaxBodies)
            hipLaunchKernelGGL(k_plain_mvs_large<4>, lgrid, dim3(T), large_lds_bytes(T), s, B, P, S);
        else
            hipLaunchKernelGGL(k_plain_mvs_large<2>, lgrid, dim3(T), large_lds_bytes(T), s, B, P, S);
        return hipGetLastError();
    }
    const int W = waves_per_group < 1 ? 1 : (waves_per_group > 4 ? 4 : waves_per_group);
    const dim3 grid = grid_for(B.count, 64 * W);
#define FB_L(NN) hipLaunchKernelGGL(k_plain_mvs<NN>, grid, dim3(64 * W), 0, s, B, P)
    FB_SWITCH_MVS(B.n, FB_L)
#undef FB_L
    return hipGetLastError();
}

}  // namespace fb
