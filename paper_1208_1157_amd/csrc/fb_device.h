// fb_device.h -- device code shared by the kernels of libfewbody: the
// inverse square root, Eq. 3/4's coefficients, the per-system clock, and the
// lane layouts (a system per lane, a body per lane of a wavefront, a body per
// lane of a workgroup).
#pragma once

#include "fb_internal.h"

namespace fb {
namespace {

// ---------------------------------------------------------------------------
// small device helpers
// ---------------------------------------------------------------------------

// LDS exchange among the lanes of one wavefront: order this wave's LDS
// writes before its subsequent reads (no workgroup barrier needed: every
// exchange stays inside one wavefront's slice).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 1/sqrt(x): hardware estimate y (v_rsq_f64, relative error ~6e-8 on
// gfx950) refined by one third-order step of the series
// 1/sqrt(x) = y (1 - e)^(-1/2) = y (1 + e/2 + 3e^2/8 + ...), e = 1 - x y^2,
// whose truncation (~e^3) is far below FP64 rounding.
__device__ __forceinline__ double rsqrt_nr(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    const double p = fma(0.375, e, 0.5);
    return fma(y * e, p, y);
}

__device__ __forceinline__ bool finite3(const double (&p)[3])
{
    return __builtin_isfinite(p[0]) && __builtin_isfinite(p[1]) && __builtin_isfinite(p[2]);
}

// Wave-uniform copies (scalar registers) of values every lane holds alike:
// tests on them are scalar branches rather than exec-mask changes.
__device__ __forceinline__ int uniform_i(const int v)
{
    return __builtin_amdgcn_readfirstlane(v);
}

__device__ __forceinline__ long long uniform_ll(const long long v)
{
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(v & 0xffffffffll));
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(v >> 32));
    return (long long)(((unsigned long long)hi << 32) | lo);
}

__device__ __forceinline__ double uniform_d(const double v)
{
    return __longlong_as_double(uniform_ll(__double_as_longlong(v)));
}

__device__ __forceinline__ StepParams uniform_params(const StepParams &P)
{
    StepParams u;
    u.adaptive = uniform_i(P.adaptive);
    u.stop_rules = uniform_i(P.stop_rules);
    u.eta = uniform_d(P.eta);
    u.r_eject = uniform_d(P.r_eject);
    u.max_steps = uniform_ll(P.max_steps);
    u.quantum = uniform_i(P.quantum);
    u.simds = P.simds;
    return u;
}

// Step coefficients of the predictor (Eq. 3) and corrector (Eq. 4).
struct Coef {
    double h, hh2, hhh6;       // predictor: h, h^2/2, h^3/6
    double bxa, bxj, bva, bvj; // bases: -3/20 h^2, -7/60 h^3, -h/2, -5/12 h^2
    double cxa, cxj, cva, cvj; // corrections: 3/20 h^2, -h^3/30, h/2, -h^2/12
};

__device__ __forceinline__ Coef make_coef(double h)
{
    Coef k;
    const double h2 = h * h, h3 = h2 * h;
    k.h = h;
    k.hh2 = 0.5 * h2;
    k.hhh6 = h3 * (1.0 / 6.0);
    k.cxa = 0.15 * h2;
    k.cxj = h3 * (-1.0 / 30.0);
    k.cva = 0.5 * h;
    k.cvj = h2 * (-1.0 / 12.0);
    k.bxa = -k.cxa;
    k.bxj = h3 * (-7.0 / 60.0);
    k.bva = -k.cva;
    k.bvj = h2 * (-5.0 / 12.0);
    return k;
}

// Predicted state and the per-step bases of the corrector for one component.
__device__ __forceinline__ void predict_comp(const Coef &k, double x, double v, double a,
                                             double j, double &xp, double &vp, double &bx,
                                             double &bv)
{
    xp = fma(k.hhh6, j, fma(k.hh2, a, fma(k.h, v, x)));
    vp = fma(k.hh2, j, fma(k.h, a, v));
    bx = fma(k.bxj, j, fma(k.bxa, a, xp));
    bv = fma(k.bvj, j, fma(k.bva, a, vp));
}

// One correction of one component from the latest evaluation (ak, jk).
__device__ __forceinline__ void correct_comp(const Coef &k, double bx, double bv, double ak,
                                             double jk, double &xc, double &vc)
{
    xc = fma(k.cxj, jk, fma(k.cxa, ak, bx));
    vc = fma(k.cvj, jk, fma(k.cva, ak, bv));
}

// One wavefront's LDS slice: the current evaluation state of its 64 lanes
// (as 16-byte pairs so a partner costs three ds_read_b128 and one b64), and
// per lane its mass beside a reduction scratch value, so every row of a
// partner sits at the same 16-byte slot offset.
struct BplLds {
    double2 xy[64];
    double2 zvx[64];
    double2 vyvz[64];
    double2 mr[64];   // (mass, reduction scratch)
};

// System-per-lane steps of at least this many bodies park the corrector
// bases (6 doubles per body, idle during each evaluation) in the wavefront's
// LDS slice, so the evaluation's working set (12 doubles per body) stays in
// VGPRs.
#ifndef FB_SPL_LDS_MIN
#define FB_SPL_LDS_MIN 6
#endif

// Rows parked after the bases by the adaptive step loop (n <= kMaxSplAdv):
// the step size and the system's clock (t, t_end, carried step, run steps,
// steps, status, last step).
constexpr int kSplParkClock = 8;

// LDS bytes per wavefront a system-per-lane step of n bodies uses.
__host__ __device__ constexpr size_t spl_lds_bytes(int n)
{
    return n >= FB_SPL_LDS_MIN
               ? (size_t)(6 * n + (n <= kMaxSplAdv ? kSplParkClock : 0)) * 64 * sizeof(double)
               : 0;
}

// Per-wavefront LDS stride of the system-per-lane fused class, whose waves
// may run either kind of tile side by side in one workgroup: large enough
// for the body-per-lane slice and for the largest parked bases.
constexpr size_t kWideLdsStride = 6 * kMaxSplBodies * 64 * sizeof(double);
static_assert(kWideLdsStride >= sizeof(BplLds), "wide LDS stride too small");
static_assert(kWideLdsStride >= spl_lds_bytes(kMaxSplAdv) &&
                  kWideLdsStride >= spl_lds_bytes(kMaxSplBodies), "wide LDS stride too small");

// This wavefront's slice of its workgroup's dynamic LDS, reached through
// the module-level symbol (not a pointer argument) so separately compiled
// tile functions still address LDS directly.  PACKED is the slice size when
// every wave of the launch runs the same kind of tile; WIDE selects the
// common stride of the system-per-lane fused class.
template <size_t PACKED, bool WIDE>
__device__ __forceinline__ char *wave_lds_base()
{
    extern __shared__ char fb_dyn_lds[];
    return fb_dyn_lds + (size_t)(threadIdx.x >> 6) * (WIDE ? kWideLdsStride : PACKED);
}

// ---------------------------------------------------------------------------
// per-system clock (Algorithm 1's loop control)
// ---------------------------------------------------------------------------
struct Clock {
    double t, t_end, dt, dtn, t0;
    long long k, nfull, steps;
    int status;
};

__device__ __forceinline__ Clock load_clock(const Bucket &B, int s)
{
    Clock c;
    c.t = B.t[s];
    c.t_end = B.t_end[s];
    c.dt = B.dt[s];
    c.dtn = B.dtn[s];
    c.t0 = B.t0run[s];
    c.k = B.krun[s];
    c.nfull = B.nfull[s];
    c.steps = B.steps[s];
    c.status = B.status[s];
    return c;
}

// The clock of a system of a SoloIO batch at its start.
__device__ __forceinline__ Clock solo_clock(const SoloIO &io)
{
    Clock c{};
    c.dt = io.dt;
    c.nfull = io.n_steps;
    c.t_end = fma((double)io.n_steps, io.dt, 0.0);
    c.status = io.n_steps > 0 ? ST_ACTIVE : ST_DONE;
    return c;
}

// Body b of system s of a SoloIO batch.
__device__ __forceinline__ void solo_load(const SoloIO &io, const int n, const int s, const int b,
                                          double &m, double (&x)[3], double (&v)[3])
{
    const size_t row = (size_t)s * n + b;
    m = io.mass[row];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        x[k] = io.pos[3 * row + k];
        v[k] = io.vel[3 * row + k];
    }
}

__device__ __forceinline__ void solo_store(const SoloIO &io, const int n, const int s, const int b,
                                           const double (&x)[3], const double (&v)[3],
                                           const int status)
{
    const size_t row = (size_t)s * n + b;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        io.pos[3 * row + k] = x[k];
        io.vel[3 * row + k] = v[k];
    }
    if (b == 0 && io.status)
        io.status[s] = status;
}

__device__ __forceinline__ void store_clock(const Bucket &B, int s, const Clock &c)
{
    B.t[s] = c.t;
    B.dtn[s] = c.dtn;
    B.krun[s] = c.k;
    B.steps[s] = c.steps;
    B.status[s] = c.status;
}

// Size of the next step, or false (with the status updated) if the system
// takes no further step.
__device__ __forceinline__ bool plan_step(Clock &c, const StepParams &P, double &h, bool &last)
{
    if (c.status != ST_ACTIVE)
        return false;
    if (P.adaptive) {
        if (!(c.t < c.t_end)) {
            c.status = ST_DONE;
            return false;
        }
        if (c.steps >= P.max_steps) {
            c.status = ST_MAXSTEPS;
            return false;
        }
        if (__builtin_isnan(c.dtn)) {
            c.status = ST_NONFINITE;
            return false;
        }
        if (!(c.dtn >= 1e-12 * fabs(c.t_end))) {
            c.status = ST_STALLED;
            return false;
        }
        last = c.t + c.dtn >= c.t_end;
        h = last ? c.t_end - c.t : c.dtn;
        return true;
    }
    if (c.steps >= P.max_steps) {
        c.status = ST_MAXSTEPS;
        return false;
    }
    if (c.k < c.nfull) {
        h = c.dt;
        last = false;
        return true;
    }
    const double rem = c.t_end - c.t;
    if (rem * c.dt > 1e-9 * c.dt * c.dt) {   // remainder in the direction of dt
        h = rem;
        last = true;
        return true;
    }
    c.t = c.t_end;
    c.status = ST_DONE;
    return false;
}

__device__ __forceinline__ void finish_step(Clock &c, const StepParams &P, bool last, double h,
                                            double dt_prop)
{
    c.steps += 1;
    if (P.adaptive) {
        c.t = last ? c.t_end : c.t + h;
        c.dtn = dt_prop;
        if (last)
            c.status = ST_DONE;
        return;
    }
    if (last) {
        c.t = c.t_end;
        c.status = ST_DONE;
        return;
    }
    c.k += 1;
    c.t = fma((double)c.k, c.dt, c.t0);
    if (c.k >= c.nfull) {
        const double rem = c.t_end - c.t;
        if (!(rem * c.dt > 1e-9 * c.dt * c.dt)) {
            c.t = c.t_end;
            c.status = ST_DONE;
        }
    }
}

__device__ __forceinline__ int status_of_flags(int fl)
{
    return (fl & 1) ? ST_NONFINITE : (fl & 2) ? ST_ENCOUNTER : (fl & 4) ? ST_EJECTED : ST_ACTIVE;
}

// Adaptive-step forms of plan_step and finish_step (the same tests in the
// same order) as selects rather than branches, for a wave that runs alone on
// its SIMD, where every branch and exec-mask change is latency on the step's
// critical path.  A lane whose system is not active keeps its clock.
__device__ __forceinline__ bool plan_step_adaptive(Clock &c, const StepParams &P, double &h,
                                                   bool &last)
{
    const bool running = c.status == ST_ACTIVE;
    // every test evaluated, then the first that holds wins
    const bool done = !(c.t < c.t_end);
    const bool maxed = c.steps >= P.max_steps;
    const bool nonfinite = __builtin_isnan(c.dtn);
    const bool stalled = !(c.dtn >= 1e-12 * fabs(c.t_end));
    int ns = stalled ? ST_STALLED : ST_ACTIVE;
    ns = nonfinite ? ST_NONFINITE : ns;
    ns = maxed ? ST_MAXSTEPS : ns;
    ns = done ? ST_DONE : ns;
    c.status = running ? ns : c.status;
    last = c.t + c.dtn >= c.t_end;
    h = last ? c.t_end - c.t : c.dtn;
    return running && ns == ST_ACTIVE;
}

__device__ __forceinline__ void finish_step_adaptive(Clock &c, const bool act, const bool last,
                                                     const double h, const double dt_prop,
                                                     const int fl)
{
    c.steps += act ? 1 : 0;
    c.t = act ? (last ? c.t_end : c.t + h) : c.t;
    c.dtn = act ? dt_prop : c.dtn;
    const int st = fl ? status_of_flags(fl) : (last ? ST_DONE : c.status);
    c.status = act ? st : c.status;
}

// Run control of fixed steps without a per-step clock.  Segment 0 is the
// run's whole steps, segment 1 the shortened final step if one is due; the
// number of steps of size h the system takes in the segment, at most
// `budget` and P.max_steps allowing.
__device__ __forceinline__ int run_segment(Clock &c, const StepParams &P, const int seg,
                                           const int budget, double &h)
{
    if (c.status != ST_ACTIVE || budget <= 0)
        return 0;
    long long cnt = 0;
    h = c.dt;
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
    return cnt > 0 ? (int)cnt : 0;
}

// The clock after `done` steps of segment seg; `was_active`: the system
// entered the segment active (its steps may have stopped it since).
__device__ __forceinline__ void run_segment_end(Clock &c, const StepParams &P, const int seg,
                                                const int done)
{
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

template <int N>
__device__ __forceinline__ double sys_max(BplLds &L, int lane, int s, double v)
{
    constexpr int S = 64 / N;
    L.mr[lane].y = v;
    wave_sync();
    double r = L.mr[s].y;
#pragma unroll
    for (int k = 1; k < N; ++k)
        r = fmax(r, L.mr[k * S + s].y);
    wave_sync();
    return r;
}

// Sum over the system's lanes in body order (deterministic).
template <int N>
__device__ __forceinline__ double sys_sum(BplLds &L, int lane, int s, double v)
{
    constexpr int S = 64 / N;
    L.mr[lane].y = v;
    wave_sync();
    double r = L.mr[s].y;
#pragma unroll
    for (int k = 1; k < N; ++k)
        r += L.mr[k * S + s].y;
    wave_sync();
    return r;
}

// OR of the stop-flag bits (1, 2, 4) over the system's lanes (s, s + S, ...)
// from three wave ballots: no LDS round trip.
template <int N>
__device__ __forceinline__ int sys_or_flags(int s, int v)
{
    constexpr int S = 64 / N;
    constexpr unsigned long long kBase = [] {
        unsigned long long m = 0;
        for (int k = 0; k < N; ++k)
            m |= 1ull << (k * S);
        return m;
    }();
    const unsigned long long sm = kBase << s;
    int r = 0;
#pragma unroll
    for (int bit = 1; bit <= 4; bit <<= 1)
        if (__ballot((v & bit) != 0) & sm)
            r |= bit;
    return r;
}

// The clock part of a run's start for slot s, at time t with status st (systems
// stopped by a rule keep theirs); true when an adaptive step
// (rule 1 or 2) must still be proposed from the system's state.
__device__ __forceinline__ bool begin_run_clock(const Bucket &B, const int s, const int st,
                                                const double t, const RunStart &run)
{
    if (st != ST_ACTIVE && st != ST_DONE && st != ST_MAXSTEPS)
        return false;
    const double dt = run.dt, t_end = run.t_end;
    B.t0run[s] = t;
    B.krun[s] = 0;
    if (run.fixed_steps) {
        B.dt[s] = dt;
        B.nfull[s] = run.n_steps;
        B.t_end[s] = fma((double)run.n_steps, dt, t);
        B.status[s] = run.n_steps > 0 ? ST_ACTIVE : ST_DONE;
        return false;
    }
    B.t_end[s] = t_end;
    if (run.adaptive == 3) {   // Runge-Kutta Cash-Karp: dt is the first trial step
        B.nfull[s] = 0;
        B.dt[s] = 0.0;
        B.dtn[s] = dt;
        B.status[s] = t < t_end ? ST_ACTIVE : ST_DONE;
        return false;
    }
    if (run.adaptive) {
        B.nfull[s] = 0;
        B.dt[s] = 0.0;
        B.status[s] = t < t_end ? ST_ACTIVE : ST_DONE;
        // Eq. 5's step depends only on the stored (a0, j0), so it is always
        // recomputed (identical to the carried value); the pairwise rule's
        // carried step comes from the last evaluation's state and is kept.
        return run.adaptive == 2 || !(B.dtn[s] > 0.0);
    }
    B.dt[s] = dt;
    const double span = (t_end - t) / dt;
    long long nf = span > 0.0 ? (long long)floor(span) : 0;
    while (nf > 0 && (fma((double)nf, dt, t) - t_end) * dt > 0.0)
        --nf;
    B.nfull[s] = nf;
    B.status[s] = (t_end - t) * dt > 0.0 ? ST_ACTIVE : ST_DONE;
    return false;
}

template <int N>
__device__ __forceinline__ void load_rows(const Bucket &B, int s, double (&m)[N], double (&x)[N][3],
                                          double (&v)[N][3], double (&a)[N][3], bool with_a)
{
    const size_t pitch = B.pitch;
#pragma unroll
    for (int b = 0; b < N; ++b) {
        m[b] = B.st[(R_M * N + b) * pitch + s];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            x[b][c] = B.st[((R_X + c) * N + b) * pitch + s];
            v[b][c] = B.st[((R_V + c) * N + b) * pitch + s];
            a[b][c] = with_a ? B.st[((R_A + c) * N + b) * pitch + s] : 0.0;
        }
    }
}

template <int N>
__device__ __forceinline__ void store_rows(const Bucket &B, int s, const double (&x)[N][3],
                                           const double (&v)[N][3], const double (&a)[N][3],
                                           bool with_a)
{
    const size_t pitch = B.pitch;
#pragma unroll
    for (int b = 0; b < N; ++b)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            B.st[((R_X + c) * N + b) * pitch + s] = x[b][c];
            B.st[((R_V + c) * N + b) * pitch + s] = v[b][c];
            if (with_a)
                B.st[((R_A + c) * N + b) * pitch + s] = a[b][c];
        }
}

// Planet-planet accelerations at heliocentric positions Q[1..N-1].
template <int N>
__device__ __forceinline__ void mvs_acc(const double (&m)[N], const double (&Q)[N][3],
                                        double (&acc)[N][3])
{
#pragma unroll
    for (int i = 1; i < N; ++i)
        acc[i][0] = acc[i][1] = acc[i][2] = 0.0;
#pragma unroll
    for (int i = 1; i < N; ++i)
#pragma unroll
        for (int j = i + 1; j < N; ++j) {
            const double d0 = Q[j][0] - Q[i][0], d1 = Q[j][1] - Q[i][1], d2 = Q[j][2] - Q[i][2];
            const double s = rsqrt_nr(fma(d2, d2, fma(d1, d1, d0 * d0)));
            const double s3 = s * s * s;
            const double mj = m[j] * s3, mi = m[i] * s3;
            acc[i][0] = fma(mj, d0, acc[i][0]);
            acc[i][1] = fma(mj, d1, acc[i][1]);
            acc[i][2] = fma(mj, d2, acc[i][2]);
            acc[j][0] = fma(-mi, d0, acc[j][0]);
            acc[j][1] = fma(-mi, d1, acc[j][1]);
            acc[j][2] = fma(-mi, d2, acc[j][2]);
        }
}

// Lanes of the largest large-n workgroup (its LDS stays below 64 KiB).
constexpr int kLargeMaxLanes = 512;

// Dynamic LDS of a large-n workgroup holding T bodies: two copies of the
// evaluation state (three 16-byte pairs per body each), the masses, one
// reduction double and one int per body.
__host__ __device__ constexpr size_t large_lds_bytes(int T)
{
    return (size_t)T * (6 * sizeof(double2) + 2 * sizeof(double) + sizeof(int));
}

struct LargeView {
    double2 *xy, *zvx, *vyvz;   // copy c of lane l at [c * T + l]
    double *m;
    double *red;
    int *flag;
};

__device__ __forceinline__ LargeView large_view(const int T)
{
    extern __shared__ char fb_dyn_lds[];
    double2 *p = reinterpret_cast<double2 *>(fb_dyn_lds);
    LargeView V;
    V.xy = p;
    V.zvx = p + 2 * T;
    V.vyvz = p + 4 * T;
    V.m = reinterpret_cast<double *>(p + 6 * T);
    V.red = V.m + T;
    V.flag = reinterpret_cast<int *>(V.red + T);
    return V;
}

// Lane geometry of a large-n workgroup.
struct LargeLane {
    int tid, sys, b, base, slot;
    bool valid;
};

__device__ __forceinline__ LargeLane large_lane(const Bucket &B, const int S)
{
    LargeLane l;
    l.tid = threadIdx.x;
    l.sys = l.tid / B.n;
    l.b = l.tid - l.sys * B.n;
    l.base = l.sys * B.n;
    const int slot = blockIdx.x * S + l.sys;
    l.valid = l.sys < S && slot < B.count;
    l.slot = l.valid ? slot : 0;
    return l;
}

// Squared separations are floored here before the inverse distance is taken:
// a body's interaction with itself (r = u = 0) then contributes exact zeros
// with every intermediate finite, and no real pair comes this close.
constexpr double kLargeMinR2 = 1e-100;

// Over bodies b >= b0 of the lane's system: sum of w_b u_b (an fma chain in
// body order) and the star's own u, to every valid lane.  Three barriers.
__device__ __forceinline__ void large_sys_wsum3(const LargeView &V, const int T,
                                                const LargeLane &l, const int n, const int b0,
                                                const double w, const double (&u)[3],
                                                double (&sum)[3], double (&star_u)[3])
{
    double2 *in0 = V.xy + T, *in1 = V.zvx + T, *res = V.vyvz + T;
    in0[l.tid] = make_double2(u[0], u[1]);
    in1[l.tid] = make_double2(u[2], w);
    __syncthreads();
    if (l.valid && l.b == 0) {
        double s0 = 0.0, s1 = 0.0, s2 = 0.0;
        for (int b = b0; b < n; ++b) {
            const double2 p = in0[l.base + b], q = in1[l.base + b];
            s0 = fma(q.y, p.x, s0);
            s1 = fma(q.y, p.y, s1);
            s2 = fma(q.y, q.x, s2);
        }
        res[l.base] = make_double2(s0, s1);
        V.red[l.base] = s2;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 3; ++c)
        sum[c] = star_u[c] = 0.0;
    if (l.valid) {
        const double2 r = res[l.base], p = in0[l.base], q = in1[l.base];
        sum[0] = r.x;
        sum[1] = r.y;
        sum[2] = V.red[l.base];
        star_u[0] = p.x;
        star_u[1] = p.y;
        star_u[2] = q.x;
    }
    __syncthreads();
}

// OR of a per-lane flag over the lane's system, to every valid lane.
__device__ __forceinline__ int large_sys_or(const LargeView &V, const LargeLane &l, const int n,
                                            const int f)
{
    V.flag[l.tid] = f;
    __syncthreads();
    int r = 0;
    if (l.valid)
        for (int b = 0; b < n; ++b)
            r |= V.flag[l.base + b];
    __syncthreads();
    return r;
}

// Planet-planet acceleration of this lane's planet at heliocentric positions
// Q (each lane's own, published here); zero on the star's lane.
__device__ __forceinline__ void large_mvs_acc(const LargeView &V, const LargeLane &l, const int n,
                                              const double (&Q)[3], double (&acc)[3])
{
    V.xy[l.tid] = make_double2(Q[0], Q[1]);
    V.zvx[l.tid] = make_double2(Q[2], 0.0);
    __syncthreads();
    acc[0] = acc[1] = acc[2] = 0.0;
    if (l.valid && l.b > 0)
        for (int j = 1; j < n; ++j) {
            if (j == l.b)
                continue;
            const double2 p0 = V.xy[l.base + j], p1 = V.zvx[l.base + j];
            const double d0 = p0.x - Q[0], d1 = p0.y - Q[1], d2 = p1.x - Q[2];
            const double sr = rsqrt_nr(fma(d2, d2, fma(d1, d1, d0 * d0)));
            const double mj = V.m[l.base + j] * (sr * sr * sr);
            acc[0] = fma(mj, d0, acc[0]);
            acc[1] = fma(mj, d1, acc[1]);
            acc[2] = fma(mj, d2, acc[2]);
        }
    __syncthreads();
}

__device__ __forceinline__ void large_load_rows(const Bucket &B, const LargeLane &l, double &mi,
                                                double (&x)[3], double (&v)[3], double (&a)[3])
{
    mi = 0.0;
    const size_t pitch = B.pitch;
    const int n = B.n;
#pragma unroll
    for (int c = 0; c < 3; ++c)
        x[c] = v[c] = a[c] = 0.0;
    if (!l.valid)
        return;
    mi = B.st[(R_M * n + l.b) * pitch + l.slot];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        x[c] = B.st[((R_X + c) * n + l.b) * pitch + l.slot];
        v[c] = B.st[((R_V + c) * n + l.b) * pitch + l.slot];
        a[c] = B.st[((R_A + c) * n + l.b) * pitch + l.slot];
    }
}

__device__ __forceinline__ void large_store_rows(const Bucket &B, const LargeLane &l,
                                                 const double (&x)[3], const double (&v)[3],
                                                 const double (&a)[3], bool with_a)
{
    if (!l.valid)
        return;
    const size_t pitch = B.pitch;
    const int n = B.n;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        B.st[((R_X + c) * n + l.b) * pitch + l.slot] = x[c];
        B.st[((R_V + c) * n + l.b) * pitch + l.slot] = v[c];
        if (with_a)
            B.st[((R_A + c) * n + l.b) * pitch + l.slot] = a[c];
    }
}

inline dim3 grid_for(int n, int block) { return dim3((unsigned)((n + block - 1) / block)); }

// Launch geometry of a large-n bucket, one body per lane: grid, lanes,
// systems per workgroup.
inline bool large_launch(const Bucket &B, dim3 &grid, int &T, int &S)
{
    large_shape(B.n, T, S);
    if (S < 1)
        return false;
    grid = dim3((unsigned)((B.count + S - 1) / S));
    return true;
}

}  // namespace
}  // namespace fb
