// fb_mvs.hip -- the step kernels of the mixed-variable symplectic integrator
// (Sections 2.2.3 and 4.3.3): democratic heliocentric drifts and kicks around
// one Kepler drift per planet.  The conversion to a bucket's MVS form and
// its read-back are in fb_setup.hip (fb_kernels.hip above 16 bodies), that from
// it in fb_kernels.hip.
#include "fb_device.h"

#include <climits>

namespace fb {
namespace {

// ---------------------------------------------------------------------------
// Kepler drift
// ---------------------------------------------------------------------------
// A planet's state advances by dt on its Kepler orbit about mu as
//   r' = r + f r + g v,  v' = v + fd r + gd v
// (Lagrange's functions, with 1 taken out of f and of gd), in universal form:
// with beta = mu / a, x the change of the eccentric anomaly and
//   G1 = sin x / sqrt(beta), G2 = (1 - cos x) / beta, G3 = (x - sin x) / beta^(3/2),
//   f = -mu G2 / r0, g = dt - mu G3, fd = -mu G1 / (r0 r'), gd = -mu G2 / r'.

// What a drift needs of the orbit at its start: 1/r, r, r.v, and
// beta = 2 mu / r - v^2 (bound: beta > 0).
struct Orbit {
    double ir, r0, eta, beta;
};

__device__ __forceinline__ Orbit orbit_of(const double mu, const double (&r)[3],
                                          const double (&v)[3])
{
    Orbit o;
    const double r2 = fma(r[2], r[2], fma(r[1], r[1], r[0] * r[0]));
    const double v2 = fma(v[2], v[2], fma(v[1], v[1], v[0] * v[0]));
    o.eta = fma(r[2], v[2], fma(r[1], v[1], r[0] * v[0]));
    o.ir = rsqrt_nr(r2);
    o.r0 = r2 * o.ir;
    o.beta = fma(mu + mu, o.ir, -v2);
    return o;
}

// Kepler's equation by eccentric anomalies: x solves its difference form
//   n dt = x - (1 - r0/a) sin x + (r.v / sqrt(mu a)) (1 - cos x)
// by Halley's iteration from x = n dt (Newton's where the second derivative
// takes most of the first away); a correction below 1e-6 of the derivative is
// the last, and turns sin x and cos x by its second-order expansion.  ok is 0 if
// the iteration does not settle in kKeplerMost steps.  Serves what kepler_solve
// leaves to it; a separate function, so that its code stays out of the step
// loops.  Two or three sincos a drift for e < 0.6; Newton's iteration with one
// more sincos of the result took 4.5 to 6 of them, and failed 5 to 20 times as
// often for e > 0.9 (CPU, 20000 orbits each at steps of 0.1 to 40 periods; mean
// error against 80-bit arithmetic up to 7% smaller for e < 0.6, up to 7% larger
// for e > 0.9).  65536 systems of 2, 4, 8 bodies, 60 steps of a quarter of a
// period: 145, 406, 695 us; with Newton's iteration 190, 556, 855, and with that
// in the step loops, without the series before it, 171, 503, 990.
constexpr int kKeplerMost = 50;

struct KeplerG {
    double G1, G2, G3;
    int ok;
};

__device__ __noinline__ KeplerG kepler_general(const double mu, const double dt, const double r0,
                                               const double eta, const double beta)
{
    KeplerG k{0.0, 0.0, 0.0, 0};
    const double alpha = beta / mu;   // 1 / a
    const double sb = sqrt(beta);
    const double ec = fma(-r0, alpha, 1.0);
    const double es = eta * sb / mu;
    const double M = sb * alpha * dt;   // n dt, n = sqrt(mu / a^3)
    double x = M, s = 0.0, c = 1.0, dx = 0.0;
    for (int it = 0; it < kKeplerMost; ++it) {
        sincos(x, &s, &c);
        const double F = fma(-ec, s, x) + fma(es, 1.0 - c, -M);
        const double F1 = fma(es, s, fma(-ec, c, 1.0));
        const double F2 = fma(es, c, ec * s);
        const double newton = F / F1, h = fma(-0.5 * newton, F2, F1);
        dx = h > 0.5 * F1 ? F / h : newton;
        x -= dx;
        if (fabs(dx) <= 1e-6 * F1) {
            k.ok = 1;
            break;
        }
    }
    const double hd = 0.5 * dx;
    const double sn = fma(-dx, fma(hd, s, c), s), cn = fma(dx, fma(-hd, c, s), c);
    const double isb = 1.0 / sb;
    k.G1 = sn * isb;
    k.G2 = (1.0 - cn) * (isb * isb);
    k.G3 = (x - sn) / (beta * sb);
    return k;
}

// 1/x: hardware estimate (relative error below 1e-7) and one third-order step.
__device__ __forceinline__ double rcp_nr(double x)
{
    const double y = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
}

// f, g, fd and gd of a step of dt on the bound orbit o; false if Kepler's
// equation did not converge.  The universal anomaly s, x = sqrt(beta) s,
// solves r0 s + (r.v) G2 + (mu - beta r0) G3 = dt; G1..G3 are powers of s
// times Stumpff's functions of z = beta s^2 = x^2.  Up to z = 1 (a radian of
// eccentric anomaly) their series of 9 terms are exact to rounding and free
// of the cancellations in 1 - cos x and x - sin x.  s starts from its
// expansion to third order in dt/r0 and is corrected by Halley's iteration; a
// correction below 1e-6 s is the last, applied to G1..G3 by their own
// second-order expansion.  A step of a hundredth of a period takes one
// evaluation of the series: about 115 FP64 instructions a drift in all, where
// the eccentric-anomaly form took about 650 (3 Newton iterations of a sincos
// and a division, and 4 more divisions and square roots).
// Error of a drift against 80-bit arithmetic, in units of 2^-53 of |r| and
// |v|, worst of 40000 orbits of e < 0.6: 1.1 at dt/P = 0.01 and 6.5 at 0.13,
// where the eccentric-anomaly form has 2.9 and 10.
// Larger anomalies, and orbits that 8 corrections do not settle, go to
// kepler_general.
__device__ __forceinline__ bool kepler_solve(const double mu, const Orbit &o, const double dt,
                                             double &f, double &g, double &fd, double &gd)
{
    const double zeta = fma(-o.beta, o.r0, mu);
    const double u = dt * o.ir, a1 = o.eta * o.ir, b1 = zeta * o.ir;
    const double c1 = fma(0.5 * a1, a1, b1 * (-1.0 / 6.0));
    double s = u * fma(u, fma(u, c1, -0.5 * a1), 1.0);
    double G0, G1, G2, G3, ds;
    bool more = true, small = true, ok = true;
    int it = 0;
#pragma unroll 1
    do {
        const double s2 = s * s, z = o.beta * s2;
        double c3 = fma(-z, 1.0 / 121645100408832000.0, 1.0 / 355687428096000.0);
        c3 = fma(-z, c3, 1.0 / 1307674368000.0);
        c3 = fma(-z, c3, 1.0 / 6227020800.0);
        c3 = fma(-z, c3, 1.0 / 39916800.0);
        c3 = fma(-z, c3, 1.0 / 362880.0);
        c3 = fma(-z, c3, 1.0 / 5040.0);
        c3 = fma(-z, c3, 1.0 / 120.0);
        c3 = fma(-z, c3, 1.0 / 6.0);
        double c2 = fma(-z, 1.0 / 6402373705728000.0, 1.0 / 20922789888000.0);
        c2 = fma(-z, c2, 1.0 / 87178291200.0);
        c2 = fma(-z, c2, 1.0 / 479001600.0);
        c2 = fma(-z, c2, 1.0 / 3628800.0);
        c2 = fma(-z, c2, 1.0 / 40320.0);
        c2 = fma(-z, c2, 1.0 / 720.0);
        c2 = fma(-z, c2, 1.0 / 24.0);
        c2 = fma(-z, c2, 0.5);
        G2 = s2 * c2;
        G3 = (s * s2) * c3;
        G1 = fma(-o.beta, G3, s);
        G0 = fma(-o.beta, G2, 1.0);
        const double F = fma(zeta, G3, fma(o.eta, G2, fma(o.r0, s, -dt)));
        const double F1 = fma(zeta, G2, fma(o.eta, G1, o.r0));
        const double F2 = fma(o.eta, G0, zeta * G1);
        const double T1 = F1 + F1;
        ds = -(F * T1) * rcp_nr(fma(T1, F1, -(F * F2)));
        more = !(fabs(ds) <= 1e-6 * fabs(s));
        small = small && z <= 1.0;
        s += ds;
        ++it;
    } while (more && small && it < 8);
    // (a last correction of at most 1e-6 of s moves z by as little)
    const double hd = 0.5 * ds;
    const double n1 = fma(ds, fma(-(o.beta * hd), G1, G0), G1);
    const double n2 = fma(ds, fma(hd, G0, G1), G2);
    G3 = fma(ds, fma(hd, G1, G2), G3);
    G1 = n1;
    G2 = n2;
    if (more || !small) {
        const KeplerG k = kepler_general(mu, dt, o.r0, o.eta, o.beta);
        G1 = k.G1;
        G2 = k.G2;
        G3 = k.G3;
        ok = k.ok != 0;
    }
    const double irn = rcp_nr(fma(zeta, G2, fma(o.eta, G1, o.r0)));
    const double m2 = mu * G2;
    f = -(m2 * o.ir);
    gd = -(m2 * irn);
    g = fma(-mu, G3, dt);
    fd = -((mu * G1) * (o.ir * irn));
    return ok;
}

__device__ __forceinline__ void kepler_move(double (&r)[3], double (&v)[3], const double f,
                                            const double g, const double fd, const double gd)
{
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double rk = r[k], vk = v[k];
        r[k] = rk + fma(f, rk, g * vk);
        v[k] = vk + fma(fd, rk, gd * vk);
    }
}

// ---------------------------------------------------------------------------
// system per lane (n <= kMaxMvsBodies)
// ---------------------------------------------------------------------------
// Planets' momentum sum_j m_j V_j (in ascending order).
template <int N>
__device__ __forceinline__ void mvs_momentum(const double (&m)[N], const double (&V)[N][3],
                                             double (&P)[3])
{
    P[0] = P[1] = P[2] = 0.0;
#pragma unroll
    for (int i = 1; i < N; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c)
            P[c] = fma(m[i], V[i][c], P[c]);
}

// Drift by h: every Q_i by (h / m0) P, X by h Vc (body 0's rows).
template <int N>
__device__ __forceinline__ void mvs_drift(double (&Q)[N][3], const double (&V)[N][3],
                                          const double (&P)[3], const double inv_m0,
                                          const double h)
{
    const double k = h * inv_m0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
#pragma unroll
        for (int i = 1; i < N; ++i)
            Q[i][c] = fma(P[c], k, Q[i][c]);
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

// (The loops over bodies stand in functions of their own: the compiler unrolls
// a function's loops before it inlines the function, but those of a kernel
// only after its arrays have become indexed registers, which cost two moves
// per FP64 instruction.)

// The planets' orbits; true if all are bound.
template <int N>
__device__ __forceinline__ bool mvs_orbits(const double mu, const double (&Q)[N][3],
                                           const double (&V)[N][3], Orbit (&o)[N])
{
    bool bound = true;
#pragma unroll
    for (int i = 1; i < N; ++i) {
        o[i] = orbit_of(mu, Q[i], V[i]);
        bound = bound && o[i].beta > 0.0;
    }
    return bound;
}

template <int N>
__device__ __forceinline__ bool mvs_finite(const double (&Q)[N][3], const double (&V)[N][3])
{
    bool fin = true;
#pragma unroll
    for (int b = 0; b < N; ++b)
        fin = fin && finite3(Q[b]) && finite3(V[b]);
    return fin;
}

// Kepler drifts by h of planets I..N-1; a planet whose system has stopped (h
// = 0) or whose solution failed (solved becomes false) stays in place.
template <int N, int I>
__device__ __forceinline__ void mvs_kepler(const double mu, const Orbit (&o)[N], const double h,
                                           double (&Q)[N][3], double (&V)[N][3], bool &solved)
{
    double f, g, fd, gd;
    const bool ok = kepler_solve(mu, o[I], h, f, g, fd, gd);
    solved = solved && ok;
    if (!__all(ok && h != 0.0)) {
        const bool go = ok && h != 0.0;
        f = go ? f : 0.0;
        g = go ? g : 0.0;
        fd = go ? fd : 0.0;
        gd = go ? gd : 0.0;
    }
    kepler_move(Q[I], V[I], f, g, fd, gd);
    if constexpr (I + 1 < N)
        mvs_kepler<N, I + 1>(mu, o, h, Q, V, solved);
}

// Fixed-step MVS integration of one system per lane for at most P.quantum
// steps (the clock logic of the Hermite kernels; a run is whole steps, so it
// has no shortened last one).  Pm holds the planets' momentum at a step's start
// and end: the closing drift of a step and the opening one of the next use the
// same velocities.  Every lane takes every step of its wavefront, so the state
// is updated in place: a branch around the step, or a break out of it, cost a
// copy of the state each step (about as many moves as the step has FP64
// instructions).  A lane that stops before the others is stored before its next
// Kepler drift and goes on with h = 0 on registers that nothing reads any more:
// the accelerations they come to hold are those after the closing drift, not
// the carried ones to the last bit.
// Bound by FP64 issue.  131072 x 3 bodies, 4000 steps: 6.53 ms (8.0e10
// system-steps/s); 22.3 ms with the eccentric-anomaly drift and the branches.
template <int N>
__device__ __forceinline__ void mvs_spl_run(const Bucket &B, const int slot, const StepParams &P)
{
    Clock c = load_clock(B, slot);
    if (c.status != ST_ACTIVE)
        return;
    double m[N], Q[N][3], V[N][3], acc[N][3], Pm[3];
    load_rows<N>(B, slot, m, Q, V, acc, true);
    const double inv_m0 = 1.0 / m[0];
    mvs_momentum<N>(m, V, Pm);
    double hs = c.dt;
    const int nrun = run_segment(c, P, 0, P.quantum, hs);
    int done = 0;
    double h = nrun > 0 ? hs : 0.0;   // 0: stopped
    bool live = nrun > 0;             // its registers are its state
    bool finite = mvs_finite<N>(Q, V);
    auto keep = [&]() {
        finite = mvs_finite<N>(Q, V);
        store_rows<N>(B, slot, Q, V, acc, true);
        live = false;
    };
    // lanes that step, and lanes whose registers are their state
    unsigned long long going = __ballot(h != 0.0), owed = going;
    if (going != 0ull)
#pragma unroll 1
    do {
        double hh = 0.5 * h;
        mvs_drift<N>(Q, V, Pm, inv_m0, hh);
        mvs_kick<N>(V, acc, hh);
        bool solved = true;
        Orbit o[N];
        const bool bound = mvs_orbits<N>(m[0], Q, V, o);
        if ((__ballot(!bound) & going) | (owed & ~going)) {   // rare
            // undo the half step and stop
            const double back = bound ? 0.0 : -hh;
            mvs_kick<N>(V, acc, back);
            mvs_momentum<N>(m, V, Pm);
            mvs_drift<N>(Q, V, Pm, inv_m0, back);
            if (!bound && h != 0.0) {
                c.status = ST_UNBOUND;
                h = hh = 0.0;
            }
            if (live && h == 0.0)   // stopped here, or in the step before
                keep();
            owed = __ballot(live);
            (void)mvs_orbits<N>(m[0], Q, V, o);
        }
        mvs_kepler<N, 1>(m[0], o, h, Q, V, solved);
        if (__any(!solved && h != 0.0)) {
            if (!solved && h != 0.0) {
                c.status = ST_UNBOUND;
                h = hh = 0.0;
            }
        }
        mvs_acc<N>(m, Q, acc);
        mvs_kick<N>(V, acc, hh);
        mvs_momentum<N>(m, V, Pm);
        mvs_drift<N>(Q, V, Pm, inv_m0, hh);
        done += h != 0.0 ? 1 : 0;
        h = done < nrun ? h : 0.0;
        going = __ballot(h != 0.0);
    } while (going != 0ull);
    if (live)
        keep();
    run_segment_end(c, P, 0, done);
    if (!finite)
        c.status = ST_NONFINITE;
    store_clock(B, slot, c);
}

template <int N>
__global__ __launch_bounds__(256) void k_plain_mvs(Bucket B, StepParams P)
{
    const int slot = blockIdx.x * blockDim.x + threadIdx.x;
    if (slot < B.count)
        mvs_spl_run<N>(B, slot, P);
}

// ---------------------------------------------------------------------------
// body per lane of a wavefront (n <= kMaxBodies)
// ---------------------------------------------------------------------------

// Momentum of the system's planets in ascending order, to every lane (each
// sums for itself).  The caller orders the next write to the slice after it.
template <int N>
__device__ __forceinline__ void mvs_bpl_momentum(BplLds &L, const int lane, const int s,
                                                 const double mi, const double (&W)[3],
                                                 double (&Pm)[3])
{
    constexpr int S = 64 / N;
    L.xy[lane] = make_double2(W[0], W[1]);
    L.zvx[lane] = make_double2(W[2], mi);
    wave_sync();
    Pm[0] = Pm[1] = Pm[2] = 0.0;
#pragma unroll
    for (int j = 1; j < N; ++j) {
        const double2 p = L.xy[j * S + s], q = L.zvx[j * S + s];
        Pm[0] = fma(q.y, p.x, Pm[0]);
        Pm[1] = fma(q.y, p.y, Pm[1]);
        Pm[2] = fma(q.y, q.x, Pm[2]);
    }
}

// Integrate one tile (floor(64/N) systems), one body per lane, for at most
// P.quantum steps: the arithmetic of mvs_spl_run in the same order.  Each
// planet's lane drifts its own orbit, so the Kepler solver's latency is paid
// once a step; positions (with masses) and velocities are exchanged through
// the wavefront's LDS slice, one exchange for the accelerations and one for
// the momentum, with no workgroup barrier.  Every lane follows the same
// control flow; a system's outcome predicates its updates.
template <int N>
__device__ __forceinline__ void mvs_bpl_run(const Bucket &B, const int first, const int count,
                                            const StepParams &P)
{
    constexpr int S = 64 / N;
    BplLds &L = *reinterpret_cast<BplLds *>(wave_lds_base<sizeof(BplLds), false>());
    const int lane = threadIdx.x & 63;
    const int braw = lane / S;
    const int b = braw < N ? braw : N - 1;
    const int s = lane - braw * S;
    const bool valid = braw < N && s < count;
    const bool planet = b > 0;
    const int slot = first + (valid ? s : 0);
    const size_t pitch = B.pitch;
    double mi = 1.0, Q[3] = {1.0, 0.0, 0.0}, W[3] = {0.0, 0.0, 0.0}, acc[3] = {0.0, 0.0, 0.0};
    Clock c{};
    c.status = ST_DONE;
    if (valid) {
        mi = B.st[(R_M * N + b) * pitch + slot];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            Q[k] = B.st[((R_X + k) * N + b) * pitch + slot];
            W[k] = B.st[((R_V + k) * N + b) * pitch + slot];
            acc[k] = B.st[((R_A + k) * N + b) * pitch + slot];
        }
        c = load_clock(B, slot);
    }
    const bool entered = c.status == ST_ACTIVE;
    double Pm[3];
    mvs_bpl_momentum<N>(L, lane, s, mi, W, Pm);
    L.mr[lane].x = mi;
    wave_sync();
    const double m0 = L.mr[s].x;
    wave_sync();
    const double inv_m0 = 1.0 / m0;
    int budget = P.quantum;
#pragma unroll 1
    for (int seg = 0; seg < 2; ++seg) {
        double h = c.dt;
        const int nrun = run_segment(c, P, seg, budget, h);
        const double hh = 0.5 * h, kd = planet ? hh * inv_m0 : hh;
        int done = 0;
        bool run = nrun > 0;
        if (__any(run))
#pragma unroll 1
        do {
            double Qn[3], Wn[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                Qn[k] = fma(planet ? Pm[k] : W[k], kd, Q[k]);
                Wn[k] = planet ? fma(hh, acc[k], W[k]) : W[k];
            }
            const Orbit o = orbit_of(m0, Qn, Wn);
            const bool unbound = run && planet && !(o.beta > 0.0);
            bool go = run;
            if (__any(unbound)) {   // rare: undo the half step of the systems concerned
                const bool undo = sys_or_flags<N>(s, unbound ? 1 : 0) != 0 && run;
                go = run && !undo;
                double W0[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    W0[k] = W[k];
                    if (undo && planet)
                        W[k] = fma(-hh, acc[k], Wn[k]);
                }
                double Pu[3];
                mvs_bpl_momentum<N>(L, lane, s, mi, W, Pu);
                wave_sync();
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    if (undo)
                        Q[k] = fma(planet ? Pu[k] : W[k], -kd, Qn[k]);
                    else
                        W[k] = W0[k];
                }
                if (undo) {
                    c.status = ST_UNBOUND;
                    run = false;
                }
            }
            bool kfail = false, ok = go;
            if (go && planet) {
                double f, g, fd, gd;
                kfail = !kepler_solve(m0, o, h, f, g, fd, gd);
                if (!kfail)
                    kepler_move(Qn, Wn, f, g, fd, gd);
            }
            if (__any(kfail)) {     // rare: its other planets keep their drift
                const bool failed = sys_or_flags<N>(s, kfail ? 1 : 0) != 0 && go;
                ok = go && !failed;
                if (failed) {
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        Q[k] = Qn[k];
                        W[k] = Wn[k];
                    }
                    c.status = ST_UNBOUND;
                    run = false;
                }
            }
            // planet-planet accelerations at the drifted positions
            L.xy[lane] = make_double2(Qn[0], Qn[1]);
            L.zvx[lane] = make_double2(Qn[2], mi);
            wave_sync();
            double an[3] = {0.0, 0.0, 0.0};
            if constexpr (N > 2) {
                const int own = b == 0 ? S : b * S;   // the star's lane: as planet 1, unused
#pragma unroll
                for (int k = 0; k < N - 2; ++k) {
                    const int ks = (k + 1) * S;
                    const int idx = s + ks + (ks >= own ? S : 0);
                    const double2 p0 = L.xy[idx], p1 = L.zvx[idx];
                    const double d0 = p0.x - Qn[0], d1 = p0.y - Qn[1], d2 = p1.x - Qn[2];
                    const double sr = rsqrt_nr(fma(d2, d2, fma(d1, d1, d0 * d0)));
                    const double mj = p1.y * (sr * sr * sr);
                    an[0] = fma(mj, d0, an[0]);
                    an[1] = fma(mj, d1, an[1]);
                    an[2] = fma(mj, d2, an[2]);
                }
            }
            wave_sync();
            if (ok) {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    if (planet) {
                        acc[k] = an[k];
                        W[k] = fma(hh, an[k], Wn[k]);
                    }
                    Q[k] = Qn[k];
                }
            }
            mvs_bpl_momentum<N>(L, lane, s, mi, W, Pm);
            wave_sync();
            if (ok) {
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    Q[k] = fma(planet ? Pm[k] : W[k], kd, Q[k]);
                ++done;
                run = done < nrun;
            }
        } while (__any(run));
        budget -= done;
        run_segment_end(c, P, seg, done);
    }
    const int bad = sys_or_flags<N>(s, (valid && !(finite3(Q) && finite3(W))) ? 1 : 0);
    if (!valid || !entered)
        return;
    if (bad)
        c.status = ST_NONFINITE;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        B.st[((R_X + k) * N + b) * pitch + slot] = Q[k];
        B.st[((R_V + k) * N + b) * pitch + slot] = W[k];
        B.st[((R_A + k) * N + b) * pitch + slot] = acc[k];
    }
    if (b == 0)
        store_clock(B, slot, c);
}

// Every body-per-lane bucket of an ensemble in one launch, largest n first:
// a bucket of a few hundred systems fills a small part of the device, and one
// launch per bucket ran them one after another.  A wavefront takes one tile.
// Bound by the latency of a lone wave's step where the tiles are fewer than
// the SIMDs.  4099 systems of 5..12 bodies, 500 steps: 0.66 ms; 22.9 ms with
// the workgroup kernel below, a launch per body count.
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2)))
void k_mvs_bpl(BucketSet set, StepParams P)
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
#define FB_C(NN) case NN: mvs_bpl_run<NN>(B, first, count, P); break;
        FB_C(2) FB_C(3) FB_C(4) FB_C(5) FB_C(6) FB_C(7) FB_C(8) FB_C(9) FB_C(10) FB_C(11)
        FB_C(12) FB_C(13) FB_C(14) FB_C(15) FB_C(16)
#undef FB_C
    default: break;
    }
}

// ---------------------------------------------------------------------------
// body per lane of a workgroup (larger systems)
// ---------------------------------------------------------------------------

// sum_j m_j W_j over the planets of the lane's system in ascending order, to
// every lane (each sums for itself from LDS broadcasts).  One barrier; the
// arrays are copy 1 of the view, which nothing else here uses.
__device__ __forceinline__ void large_mvs_momentum(const LargeView &V, const int T,
                                                   const LargeLane &l, const int n,
                                                   const double mi, const double (&W)[3],
                                                   double (&Pm)[3])
{
    double2 *in0 = V.xy + T, *in1 = V.zvx + T;
    in0[l.tid] = make_double2(W[0], W[1]);
    in1[l.tid] = make_double2(W[2], mi);
    __syncthreads();
    Pm[0] = Pm[1] = Pm[2] = 0.0;
    if (l.valid)
#pragma unroll 4
        for (int j = 1; j < n; ++j) {
            const double2 p = in0[l.base + j], q = in1[l.base + j];
            Pm[0] = fma(q.y, p.x, Pm[0]);
            Pm[1] = fma(q.y, p.y, Pm[1]);
            Pm[2] = fma(q.y, q.x, Pm[2]);
        }
}

// Fixed-step MVS integration, one body per lane, for at most P.quantum steps
// (the clock of the Hermite kernels; the steps of mvs_spl_run, with the
// outcomes of a system predicating its updates).  A step has five barriers:
// one each for the momentum, whether any orbit is unbound and whether any
// Kepler solution failed (the systems concerned are found only then), and
// two for the accelerations; the momentum is carried to the next step.
// 128 VGPRs, 4 waves per SIMD, to hide the Kepler solver's latency.
__global__ __launch_bounds__(kLargeMaxLanes) __attribute__((amdgpu_waves_per_eu(4)))
void k_plain_mvs_large(Bucket B, StepParams P, int S)
{
    const int T = blockDim.x, n = B.n;
    const LargeView V = large_view(T);
    const LargeLane l = large_lane(B, S);
    const bool planet = l.b > 0;
    double mi, Q[3], W[3], acc[3], Pm[3];
    large_load_rows(B, l, mi, Q, W, acc);
    V.m[l.tid] = mi;
    Clock c;
    c.status = ST_DONE;
    if (l.valid)
        c = load_clock(B, l.slot);
    large_mvs_momentum(V, T, l, n, mi, W, Pm);   // its barrier orders V.m too
    __syncthreads();
    const double m0 = l.valid ? V.m[l.base] : 1.0;
    const double inv_m0 = 1.0 / m0;
    for (int q = 0; q < P.quantum; ++q) {
        double h = 0.0;
        bool last = false;
        const bool act = l.valid && plan_step(c, P, h, last);
        if (!__syncthreads_or(act))
            break;
        const double hh = 0.5 * h, kd = planet ? hh * inv_m0 : hh;
        if (act)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                Q[k] = fma(planet ? Pm[k] : W[k], kd, Q[k]);
                if (planet)
                    W[k] = fma(hh, acc[k], W[k]);
            }
        const Orbit o = orbit_of(m0, Q, W);
        const bool unbound = act && planet && !(o.beta > 0.0);
        bool go = act;
        if (__syncthreads_or(unbound)) {   // rare: undo the half step of the systems concerned
            const bool undo = large_sys_or(V, l, n, unbound) != 0 && act;
            if (undo && planet)
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    W[k] = fma(-hh, acc[k], W[k]);
            double Pu[3];
            large_mvs_momentum(V, T, l, n, mi, W, Pu);
            __syncthreads();
            if (undo) {
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    Q[k] = fma(planet ? Pu[k] : W[k], -kd, Q[k]);
                c.status = ST_UNBOUND;
            }
            go = act && !undo;
        }
        bool kfail = false, ok = go;
        if (go && planet) {
            double f, g, fd, gd;
            kfail = !kepler_solve(m0, o, h, f, g, fd, gd);
            if (!kfail)
                kepler_move(Q, W, f, g, fd, gd);
        }
        if (__syncthreads_or(kfail)) {     // rare
            const bool failed = large_sys_or(V, l, n, kfail) != 0 && go;
            if (failed)
                c.status = ST_UNBOUND;
            ok = go && !failed;
        }
        double an[3];
        large_mvs_acc(V, l, n, Q, an);
        if (ok && planet)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                acc[k] = an[k];
                W[k] = fma(hh, acc[k], W[k]);
            }
        large_mvs_momentum(V, T, l, n, mi, W, Pm);
        if (ok) {
#pragma unroll
            for (int k = 0; k < 3; ++k)
                Q[k] = fma(planet ? Pm[k] : W[k], kd, Q[k]);
            finish_step(c, P, last, h, 0.0);
        }
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

hipError_t launch_plain_mvs(const Bucket &B, int waves_per_group, const StepParams &P,
                            hipStream_t s)
{
    if (B.count == 0)
        return hipSuccess;
    const int W = waves_per_group < 1 ? 1 : (waves_per_group > 4 ? 4 : waves_per_group);
    const dim3 grid = grid_for(B.count, 64 * W);
#define FB_L(NN) hipLaunchKernelGGL(k_plain_mvs<NN>, grid, dim3(64 * W), 0, s, B, P)
    FB_SWITCH_MVS(B.n, FB_L)
#undef FB_L
    return hipGetLastError();
}

hipError_t launch_plain_mvs_large(const Bucket &B, const StepParams &P, hipStream_t s)
{
    if (B.count == 0)
        return hipSuccess;
    dim3 grid;
    int T, S;
    if (!large_launch(B, grid, T, S))
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_plain_mvs_large, grid, dim3(T), large_lds_bytes(T), s, B, P, S);
    return hipGetLastError();
}

hipError_t launch_mvs_bpl(const BucketSet &set, const StepParams &P, hipStream_t s)
{
    const int tiles = set.count > 0 ? set.first[set.count] : 0;
    if (tiles == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_mvs_bpl, dim3(tiles), dim3(64), sizeof(BplLds), s, set, P);
    return hipGetLastError();
}

}  // namespace fb
