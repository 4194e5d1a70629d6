// fb_kernels.hip -- gfx950 kernels of libfewbody.
//
// FP64 fourth-order time-symmetrised Hermite P(EC)^2 steps of many
// independent few-body systems (Swarm-NG, arXiv:1208.1157: Eq. 1 and its
// time derivative for the pair forces, Eq. 3 predictor, Eq. 4 corrector
// applied twice per step as in Algorithm 2, many steps per launch as in
// Algorithm 1).  All arithmetic is FP64 on the vector ALUs; the pair sums are
// not a dense contraction, so no MFMA is used.
//
// Two kinds of lane mapping (both read the bucket's structure-of-arrays state with
// consecutive lanes on consecutive slots):
//   SPL  one system per lane.  The whole system lives in VGPRs for the whole
//        step loop; every pair is evaluated once (Newton's third law), no
//        cross-lane traffic.  Used for small n.
//   BPL  one body per lane, floor(64/n) systems per wavefront (lane = body *
//        S + system).  Each lane evaluates its body's n-1 interactions with
//        partner positions/velocities read from the wave's LDS slice; no
//        reduction is needed and every lane does useful work.  Tiles of it
//        are in fb_bpl.h and, unrolled, fb_unrolled.hip; fb_split.h gives a
//        body several lanes.
// In all, each body sums its planet partners in ascending order and the
// star last (Section 4.2), so results are bitwise the same.
//
// The corrector is Eq. 4 read with coefficient 3/20, a (dt)^3 jerk term and
// the predicted state (xp, vp) as the base of every correction:
//   x1 = xp - 3/20 (a0 - ak) h^2 - (7 j0 + 2 jk) h^3 / 60
//   v1 = vp - 1/2 (a0 - ak) h - (5 j0 + jk) h^2 / 12
// The a0/j0 parts are folded into per-step bases, so each correction costs
// four FMAs per component and does not need the corrected velocity.
#include "fb_split.h"

#include <algorithm>
#include <climits>

// Pairs per scheduling group in the system-per-lane evaluation of n >= 5.
#ifndef FB_SPL_PAIR_GROUP
#define FB_SPL_PAIR_GROUP 2
#endif
// Waves per SIMD the register allocator targets for the rolled body-per-lane
// kernels: 3 (168 VGPRs) leaves the adaptive variants unspilled and measured
// faster than 4 (128 VGPRs, with spills) in fixed and adaptive runs.
#ifndef FB_BPL_WAVES
#define FB_BPL_WAVES 3
#endif

namespace fb {
namespace {

// ---------------------------------------------------------------------------
// system-per-lane (SPL)
// ---------------------------------------------------------------------------

// Pair (i, j): r = x_j - x_i, u = v_j - v_i, A = r/|r|^3,
// J = u/|r|^3 - 3 (r.u)/|r|^2 A; body i gains m_j (A, J), body j loses
// m_i (A, J).  With TS, also track max over pairs of
// (|u|^2 + 3 (r.u)^2/|r|^2) / |r|^2 = (|j_ij| / |a_ij|)^2 of the pair's
// two-body relative motion (the step rule's quantity).
template <int N, bool TS>
__device__ __forceinline__ void spl_pair(const int i, const int j, const double (&m)[N],
                                         const double (&x)[N][3], const double (&v)[N][3],
                                         double (&a)[N][3], double (&jk)[N][3], double &wmax)
{
    const double rx = x[j][0] - x[i][0], ry = x[j][1] - x[i][1], rz = x[j][2] - x[i][2];
    const double ux = v[j][0] - v[i][0], uy = v[j][1] - v[i][1], uz = v[j][2] - v[i][2];
    const double r2 = fma(rz, rz, fma(ry, ry, rx * rx));
    const double ru = fma(rz, uz, fma(ry, uy, rx * ux));
    const double ri = rsqrt_nr(r2);
    const double ri2 = ri * ri;
    const double ri3 = ri2 * ri;
    const double al = 3.0 * ru * ri2;
    // J / |r|^-3 = u - 3 (r.u)/|r|^2 r; masses folded into |r|^-3
    const double wx = fma(-al, rx, ux), wy = fma(-al, ry, uy), wz = fma(-al, rz, uz);
    const double mj3 = m[j] * ri3, mi3 = m[i] * ri3;
    a[i][0] = fma(mj3, rx, a[i][0]);
    a[i][1] = fma(mj3, ry, a[i][1]);
    a[i][2] = fma(mj3, rz, a[i][2]);
    a[j][0] = fma(-mi3, rx, a[j][0]);
    a[j][1] = fma(-mi3, ry, a[j][1]);
    a[j][2] = fma(-mi3, rz, a[j][2]);
    jk[i][0] = fma(mj3, wx, jk[i][0]);
    jk[i][1] = fma(mj3, wy, jk[i][1]);
    jk[i][2] = fma(mj3, wz, jk[i][2]);
    jk[j][0] = fma(-mi3, wx, jk[j][0]);
    jk[j][1] = fma(-mi3, wy, jk[j][1]);
    jk[j][2] = fma(-mi3, wz, jk[j][2]);
    if (TS) {
        const double u2 = fma(uz, uz, fma(uy, uy, ux * ux));
        wmax = fmax(wmax, fma(al, ru, u2) * ri2);
        // Keep the running maximum a serial chain through the pairs: left
        // free, the compiler rebalances it into a tree at the end, which
        // keeps every pair's inputs live and spills systems of n >= 6.
        __asm__ __volatile__("" : "+v"(wmax));
    }
}

// Acceleration and jerk of every body: planet-planet pairs first, then the
// star's pairs, so each planet adds the star's contribution last.
template <int N, bool TS>
__device__ __forceinline__ void spl_accjerk(const double (&m)[N], const double (&x)[N][3],
                                            const double (&v)[N][3], double (&a)[N][3],
                                            double (&jk)[N][3], double &wmax)
{
#pragma unroll
    for (int b = 0; b < N; ++b)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            a[b][c] = 0.0;
            jk[b][c] = 0.0;
        }
    // For larger systems, scheduling barriers between groups of pairs keep
    // the scheduler from interleaving (and keeping live) every pair's
    // temporaries at once, which would spill the system's state.
    constexpr int kGroup = N <= 4 ? 1 << 20 : FB_SPL_PAIR_GROUP;
#pragma unroll
    for (int i = 1; i < N; ++i)
#pragma unroll
        for (int j = i + 1; j < N; ++j) {
            spl_pair<N, TS>(i, j, m, x, v, a, jk, wmax);
            if (((i - 1) * (2 * N - i - 2) / 2 + (j - i)) % kGroup == 0)
                __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
    for (int j = 1; j < N; ++j) {
        spl_pair<N, TS>(0, j, m, x, v, a, jk, wmax);
        if (j % kGroup == 0)
            __builtin_amdgcn_sched_barrier(0);
    }
}

// This lane's parking area: [6N + kSplParkClock][64] doubles, lane fastest.
template <int N, bool WIDE>
__device__ __forceinline__ double *spl_park()
{
    return reinterpret_cast<double *>(wave_lds_base<spl_lds_bytes(N), WIDE>()) + (threadIdx.x & 63);
}

// One P(EC)^2 step of size h.  On entry (a, jk) hold the carried a0, j0; on
// exit (x, v) are the corrected state and (a, jk) the last evaluation.
// Returns the step-rule quantity of the last evaluation (TS only).  With
// RELOAD (parked steps only) the caller has parked h in row 6N and the step
// coefficients are rebuilt from it after each evaluation instead of being
// kept in registers through it.
template <int N, bool TS, bool WIDE, bool RELOAD = false>
__device__ __forceinline__ double spl_step(const double (&m)[N], double (&x)[N][3],
                                           double (&v)[N][3], double (&a)[N][3],
                                           double (&jk)[N][3], const Coef &k0)
{
    constexpr bool kPark = N >= FB_SPL_LDS_MIN;
    static_assert(!RELOAD || kPark, "coefficient reload needs the parking area");
    double *park = spl_park<N, WIDE>();
    Coef k = k0;
    double bx[N][3], bv[N][3], xc[N][3], vc[N][3];
#pragma unroll
    for (int b = 0; b < N; ++b)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            predict_comp(k, x[b][c], v[b][c], a[b][c], jk[b][c], xc[b][c], vc[b][c], bx[b][c],
                         bv[b][c]);
            if (kPark) {
                park[(6 * b + c) * 64] = bx[b][c];
                park[(6 * b + 3 + c) * 64] = bv[b][c];
            }
        }
    // The clobbers keep the compiler from forwarding the parked values
    // (which would keep them in registers) or hoisting their reloads above
    // the evaluation.
    if (kPark)
        __asm__ __volatile__("" ::: "memory");
    double w = 0.0;
    spl_accjerk<N, false>(m, xc, vc, a, jk, w);
    if (kPark)
        __asm__ __volatile__("" ::: "memory");
    if (RELOAD)
        k = make_coef(park[6 * N * 64]);
#pragma unroll
    for (int b = 0; b < N; ++b)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            if (kPark) {
                bx[b][c] = park[(6 * b + c) * 64];
                bv[b][c] = park[(6 * b + 3 + c) * 64];
            }
            correct_comp(k, bx[b][c], bv[b][c], a[b][c], jk[b][c], xc[b][c], vc[b][c]);
        }
    if (kPark)
        __asm__ __volatile__("" ::: "memory");
    spl_accjerk<N, TS>(m, xc, vc, a, jk, w);
    if (kPark)
        __asm__ __volatile__("" ::: "memory");
    if (RELOAD)
        k = make_coef(park[6 * N * 64]);
#pragma unroll
    for (int b = 0; b < N; ++b)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            if (kPark) {
                bx[b][c] = park[(6 * b + c) * 64];
                bv[b][c] = park[(6 * b + 3 + c) * 64];
            }
            correct_comp(k, bx[b][c], bv[b][c], a[b][c], jk[b][c], xc[b][c], vc[b][c]);
            x[b][c] = xc[b][c];
            v[b][c] = vc[b][c];
        }
    return w;
}

template <int N>
__device__ __forceinline__ int spl_stop_flags(const double (&m)[N], const double (&x)[N][3],
                                              const double (&v)[N][3], const StepParams &P)
{
    bool fin = true;
#pragma unroll
    for (int b = 0; b < N; ++b)
        fin = fin && finite3(x[b]) && finite3(v[b]);
    if (!fin)
        return 1;
    double r[N];
    r[0] = 0.0;
#pragma unroll
    for (int i = 1; i < N; ++i) {
        const double dx = x[i][0] - x[0][0], dy = x[i][1] - x[0][1], dz = x[i][2] - x[0][2];
        r[i] = sqrt(fma(dz, dz, fma(dy, dy, dx * dx)));
    }
    int fl = 0;
    if (P.stop_rules & 1) {
        const double inv24m0 = 1.0 / (24.0 * m[0]);
#pragma unroll
        for (int i = 1; i < N; ++i)
#pragma unroll
            for (int j = i + 1; j < N; ++j) {
                const double dx = x[i][0] - x[j][0], dy = x[i][1] - x[j][1],
                             dz = x[i][2] - x[j][2];
                const double sep2 = fma(dz, dz, fma(dy, dy, dx * dx));
                if (hill_close(sep2, m[i], m[j], inv24m0, r[i], r[j]))
                    fl |= 2;
            }
    }
    if (P.stop_rules & 2) {
#pragma unroll
        for (int i = 1; i < N; ++i)
            if (r[i] > P.r_eject)
                fl |= 4;
    }
    return fl;
}

// Eq. 5 (Section 4.3.1): tau [sum_i |j_i|^2 / |a_i|^2]^(-1/2) from the
// accelerations and jerks that start the next step, summed in body order.
template <int N>
__device__ __forceinline__ double paper_dt(const double (&a)[N][3], const double (&jk)[N][3],
                                           double tau)
{
    double sum = 0.0;
#pragma unroll
    for (int b = 0; b < N; ++b) {
        const double aa = fma(a[b][2], a[b][2], fma(a[b][1], a[b][1], a[b][0] * a[b][0]));
        const double jj = fma(jk[b][2], jk[b][2], fma(jk[b][1], jk[b][1], jk[b][0] * jk[b][0]));
        sum += jj / aa;
    }
    return tau * rsqrt_nr(sum);
}

// Integrate one system (one lane) for at most P.quantum steps.
template <int N, bool ADV, bool WIDE>
__device__ __forceinline__ void spl_run(const Bucket &B, const int slot, const StepParams &P)
{
    Clock c = load_clock(B, slot);
    if (c.status != ST_ACTIVE)
        return;
    const size_t pitch = B.pitch;
    const double *st = B.st;
    double m[N], x[N][3], v[N][3], a[N][3], jk[N][3];
#pragma unroll
    for (int b = 0; b < N; ++b) {
        m[b] = st[(R_M * N + b) * pitch + slot];
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            x[b][cc] = st[((R_X + cc) * N + b) * pitch + slot];
            v[b][cc] = st[((R_V + cc) * N + b) * pitch + slot];
            a[b][cc] = st[((R_A + cc) * N + b) * pitch + slot];
            jk[b][cc] = st[((R_J + cc) * N + b) * pitch + slot];
        }
    }
    if (!ADV) {
        // Fixed step.  Segment 0 runs the run's whole steps with no per-step
        // bookkeeping; segment 1 the shortened final step, if one is due.
        // One loop serves both so the step body is instantiated once.
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
            const Coef k = make_coef(h);
            constexpr int kStepUnroll = N <= 4 ? 2 : 1;
#pragma unroll kStepUnroll
            for (int q = 0; q < nrun; ++q)
                (void)spl_step<N, false, WIDE>(m, x, v, a, jk, k);
            budget -= nrun;
            c.steps += nrun;
            if (seg == 0) {
                c.k += nrun;
                if (nrun > 0)
                    c.t = fma((double)c.k, c.dt, c.t0);
                if (c.k >= c.nfull) {
                    const double rem = c.t_end - c.t;
                    if (!(rem * c.dt > 1e-9 * c.dt * c.dt)) {
                        c.t = c.t_end;
                        c.status = ST_DONE;
                    }
                }
            } else if (nrun > 0) {
                c.t = c.t_end;
                c.status = ST_DONE;
            }
            if (c.status == ST_ACTIVE && c.steps >= P.max_steps)
                c.status = ST_MAXSTEPS;
        }
    } else {
        // Parked steps also park the step size and the clock across the step
        // (rows 6N..6N+7), so the evaluations keep only the system in VGPRs.
        constexpr bool kParkClock = N >= FB_SPL_LDS_MIN;
        double *pc = kParkClock ? spl_park<N, WIDE>() + 6 * N * 64 : nullptr;
        for (int q = 0; q < P.quantum; ++q) {
            double h = 0.0;
            bool last = false;
            if (!plan_step(c, P, h, last))
                break;
            if constexpr (kParkClock) {
                pc[0] = h;
                pc[64] = c.t;
                pc[2 * 64] = c.t_end;
                pc[3 * 64] = c.dtn;
                pc[4 * 64] = __longlong_as_double(c.k);
                pc[5 * 64] = __longlong_as_double(c.steps);
                pc[6 * 64] = (double)c.status;
                pc[7 * 64] = last ? 1.0 : 0.0;
                __asm__ __volatile__("" ::: "memory");
            }
            const double w = spl_step<N, true, WIDE, kParkClock>(m, x, v, a, jk, make_coef(h));
            if constexpr (kParkClock) {
                __asm__ __volatile__("" ::: "memory");
                h = pc[0];
                c.t = pc[64];
                c.t_end = pc[2 * 64];
                c.dtn = pc[3 * 64];
                c.k = __double_as_longlong(pc[4 * 64]);
                c.steps = __double_as_longlong(pc[5 * 64]);
                c.status = (int)pc[6 * 64];
                last = pc[7 * 64] != 0.0;
            }
            double dtp = P.adaptive == 2 ? paper_dt<N>(a, jk, P.eta) : P.eta * rsqrt_nr(w);
            finish_step(c, P, last, h, dtp);
            const int fl = spl_stop_flags<N>(m, x, v, P);
            if (fl)
                c.status = status_of_flags(fl);
            if (c.status != ST_ACTIVE)
                break;
        }
    }
    if (!ADV) {
        bool fin = true;
#pragma unroll
        for (int b = 0; b < N; ++b)
            fin = fin && finite3(x[b]) && finite3(v[b]);
        if (!fin)
            c.status = ST_NONFINITE;
    }
#pragma unroll
    for (int b = 0; b < N; ++b)
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            B.st[((R_X + cc) * N + b) * pitch + slot] = x[b][cc];
            B.st[((R_V + cc) * N + b) * pitch + slot] = v[b][cc];
            B.st[((R_A + cc) * N + b) * pitch + slot] = a[b][cc];
            B.st[((R_J + cc) * N + b) * pitch + slot] = jk[b][cc];
        }
    store_clock(B, slot, c);
}

// ---------------------------------------------------------------------------
// kernels: plain schedule (one launch per homogeneous bucket)
// ---------------------------------------------------------------------------
// The system-per-lane run of 9 and 10 bodies as a separately compiled
// function: inlined into the kernel, the register allocator spilled 92 and
// 476 bytes per lane to scratch memory; as a callee it spills to AGPRs only.
template <int N, bool ADV>
__device__ __noinline__ void spl_plain_call(const Bucket &B, const int slot, const StepParams &P)
{
    spl_run<N, ADV, false>(B, slot, uniform_params(P));
}

template <int N, bool ADV>
__global__ __launch_bounds__(256) void k_plain_spl(Bucket B, StepParams P)
{
    const int slot = blockIdx.x * blockDim.x + threadIdx.x;
    if (slot >= B.count)
        return;
    if constexpr (N >= 9)
        spl_plain_call<N, ADV>(B, slot, P);
    else
        spl_run<N, ADV, false>(B, slot, P);
}

template <int N, bool ADV>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(FB_BPL_WAVES)))
void k_plain_bpl(Bucket B, StepParams P)
{
    constexpr int S = 64 / N;
    const int wave = threadIdx.x >> 6;
    const int tile = blockIdx.x * (blockDim.x >> 6) + wave;
    const int first = tile * S;
    if (first >= B.count)
        return;
    const int count = min(S, B.count - first);
    int slot;
    bpl_run<N, ADV, false, false>(B, first, count, nullptr, P, slot);
}

// ---------------------------------------------------------------------------
// kernel: persistent schedule (one fused launch over every bucket)
// ---------------------------------------------------------------------------

// Append the systems flagged by `keep` to bucket `bk`'s survivor list
// (wave-aggregated: one atomic per wavefront).
__device__ __forceinline__ void append_survivors(const ActiveLists &AL, int bk, bool keep,
                                                 int slot)
{
    const int lane = threadIdx.x & 63;
    const unsigned long long mask = __ballot(keep);
    if (mask == 0ull)
        return;
    const int cnt = __popcll(mask);
    int base = 0;
    if (lane == 0)
        base = atomicAdd(&AL.next_count[bk], cnt);
    base = __builtin_amdgcn_readfirstlane(base);
    const int pre = __popcll(mask & ((1ull << lane) - 1ull));
    if (keep)
        AL.next[AL.base[bk] + base + pre] = slot;
}

// The tile functions are separately compiled, so their reference arguments
// arrive as generic pointers; the step loop works on a register copy of the
// step parameters (read once), not on memory it would reload after every LDS
// exchange.  The copy is made wave-uniform (scalar registers), so the tests
// on it are scalar branches rather than exec-mask changes.
template <int N, bool ADV>
__device__ __noinline__ bool spl_tile(const Bucket &B, const Tile &T, const int *list,
                                      const StepParams &P, int &slot)
{
    const StepParams Pr = uniform_params(P);
    const int lane = threadIdx.x & 63;
    slot = 0;
    if (lane >= T.count)
        return false;
    slot = list ? list[T.first + lane] : T.first + lane;
    spl_run<N, ADV, true>(B, slot, Pr);
    return B.status[slot] == ST_ACTIVE;
}

// CLS only separates the instances used by the two fused-kernel classes, so
// each is compiled under its own kernel's register budget.
template <int N, bool ADV, bool CLS>
__device__ __noinline__ bool bpl_tile(const Bucket &B, const Tile &T, const int *list,
                                      const StepParams &P, int &slot)
{
    const StepParams Pr = uniform_params(P);
    constexpr bool kRegs = !ADV || N <= kMaxUnrolledAdv;
    return bpl_run<N, ADV, CLS, kRegs>(B, T.first, T.count, list, Pr, slot);
}

template <int N, int G, bool ADV>
__device__ __noinline__ bool split_tile(const Bucket &B, const Tile &T, const int *list,
                                        const StepParams &P, int &slot)
{
    const StepParams Pr = uniform_params(P);
    return split_run<N, G, ADV>(*reinterpret_cast<BplLds *>(wave_lds_base<sizeof(BplLds), false>()), B,
                           T.first, T.count, list, Pr, slot);
}

// Tile dispatch.  The body-per-lane class (SPLC false) keeps the fused
// kernel at 256 VGPRs (2 waves per SIMD) and runs every tile body-per-lane,
// partner loops unrolled (up to 10 bodies with adaptive steps / stop rules);
// the system-per-lane class gives the kernel the full register file (1 wave
// per SIMD) and runs system-per-lane tiles up to n = 10 (n = 8 with
// adaptive steps / stop rules), body-per-lane beyond.
// The body-per-lane class had rolled loops for every n and 3 waves per SIMD
// (168 VGPRs), and a thinned population moved to the other class, one wave per
// SIMD with the loops of up to 8 bodies unrolled.  Two waves serve both: a
// wave alone on its SIMD runs as fast, and of two waves each takes 1.5 times
// as long, not twice.  Best of 3, rolled and unrolled: 65536 systems of 3..15
// bodies, 500 fixed steps 8.87 and 8.40 ms; 65536 of 4..8 bodies, adaptive
// with stop rules, 10 orbits 78.4 and 72.6 ms; 16384 of them, 3 orbits, 11.4
// and 10.6 ms; 24 requests to a server (a few hundred wavefronts) 22.4 and
// 13.9 ms of kernels.  13..16 bodies, fixed steps, 16000 and 65536 systems of 14:
// three waves rolled 707 and 2457 us, two rolled 811 and 2555, two unrolled (the
// partners in three parts) 550 and 2130.  11..16 with rules stay rolled: two
// waves take 0.94 to 0.99 of three waves' time with adaptive steps, and 1.06 to
// 1.11 in fixed steps with stop rules, which have a class of their own
// (k_persistent_rolled).
template <bool ADV, bool SPLC>
__device__ __forceinline__ bool run_tile(const Bucket &B, const Tile &T, const int *list,
                                         const StepParams &P, int &slot)
{
    const int map = T.kind >> 5;
    const int n = T.kind & 31;
    if (map == MAP_SPL) {
        if constexpr (SPLC) {
            switch (n) {
            case 2: return spl_tile<2, ADV>(B, T, list, P, slot);
            case 3: return spl_tile<3, ADV>(B, T, list, P, slot);
            case 4: return spl_tile<4, ADV>(B, T, list, P, slot);
            case 5: return spl_tile<5, ADV>(B, T, list, P, slot);
            case 6: return spl_tile<6, ADV>(B, T, list, P, slot);
            case 7: return spl_tile<7, ADV>(B, T, list, P, slot);
            case 8: return spl_tile<8, ADV>(B, T, list, P, slot);
            default: break;
            }
            if constexpr (!ADV) {
                switch (n) {
                case 9: return spl_tile<9, false>(B, T, list, P, slot);
                case 10: return spl_tile<10, false>(B, T, list, P, slot);
                default: break;
                }
            }
        }
    }
    if constexpr (!SPLC) {
        if (map == MAP_SPLIT4 || map == MAP_SPLIT2) {
            switch (map == MAP_SPLIT4 ? 32 + n : n) {
#define FB_SPLIT_CASE(NN)                                        \
    case NN: return split_tile<NN, 2, ADV>(B, T, list, P, slot);      \
    case 32 + NN: return split_tile<NN, 4, ADV>(B, T, list, P, slot);
                FB_SPLIT_CASE(5) FB_SPLIT_CASE(6) FB_SPLIT_CASE(7) FB_SPLIT_CASE(8)
                FB_SPLIT_CASE(9) FB_SPLIT_CASE(10) FB_SPLIT_CASE(11) FB_SPLIT_CASE(12)
                FB_SPLIT_CASE(13) FB_SPLIT_CASE(14) FB_SPLIT_CASE(15) FB_SPLIT_CASE(16)
#undef FB_SPLIT_CASE
            default: return false;
            }
        }
    }
    switch (n) {
#define FB_BPL_CASE(NN) case NN: return bpl_tile<NN, ADV, SPLC>(B, T, list, P, slot);
        FB_BPL_CASE(2) FB_BPL_CASE(3) FB_BPL_CASE(4) FB_BPL_CASE(5) FB_BPL_CASE(6)
        FB_BPL_CASE(7) FB_BPL_CASE(8) FB_BPL_CASE(9) FB_BPL_CASE(10) FB_BPL_CASE(11)
        FB_BPL_CASE(12) FB_BPL_CASE(13) FB_BPL_CASE(14) FB_BPL_CASE(15) FB_BPL_CASE(16)
#undef FB_BPL_CASE
    default: return false;
    }
}

// Tile of wavefront i in a launch whose tiles, longest first, all run at once,
// more than one a SIMD and at most two.  One-wavefront workgroups are
// dispatched so that i and i + simds share a SIMD.  The longest tiles get the
// SIMDs that no second one comes to, and of the others the longest that may
// share goes with the shortest of all: in index order the second ones joined
// the longest.  16384 systems of 4..8 bodies (1587 tiles), adaptive with stop
// rules, 3 orbits: 10.05 -> 9.16 ms, workgroups of two in index order 10.33.
__device__ __forceinline__ int place_tile(const int i, const int ntiles, const int simds)
{
    const int shared = ntiles - simds;
    return i < shared ? simds - shared + i : i < simds ? i - shared : ntiles - 1 - (i - simds);
}

// Rolled tile of k_persistent_rolled.
template <int N>
__device__ __noinline__ bool rolled_tile(const Bucket &B, const Tile &T, const int *list,
                                         const StepParams &P, int &slot)
{
    const StepParams Pr = uniform_params(P);
    return bpl_run<N, true, false, false>(B, T.first, T.count, list, Pr, slot);
}

__device__ __forceinline__ bool run_rolled_tile(const Bucket &B, const Tile &T, const int *list,
                                                const StepParams &P, int &slot)
{
    static_assert(kMinRolled == 9 && kMaxBodies == 16, "the body counts below");
    switch (T.kind & 31) {
    case 9: return rolled_tile<9>(B, T, list, P, slot);
    case 10: return rolled_tile<10>(B, T, list, P, slot);
    case 11: return rolled_tile<11>(B, T, list, P, slot);
    case 12: return rolled_tile<12>(B, T, list, P, slot);
    case 13: return rolled_tile<13>(B, T, list, P, slot);
    case 14: return rolled_tile<14>(B, T, list, P, slot);
    case 15: return rolled_tile<15>(B, T, list, P, slot);
    case 16: return rolled_tile<16>(B, T, list, P, slot);
    default: return false;
    }
}

template <bool ADV, bool COMPACT, int CLS>
__device__ __forceinline__ void persistent_body(const Bucket *__restrict__ buckets,
                                                const Tile *__restrict__ tiles,
                                                const int *__restrict__ ntiles_p,
                                                int *__restrict__ head, const int *lists,
                                                const StepParams &P, const ActiveLists &AL)
{
    const int ntiles = *ntiles_p;
    const int lane = threadIdx.x & 63;
    // Each wave's first tile is its own index; the rest come from the queue
    // (past the first round).  Workgroups are dispatched across the CUs in
    // index order, so when the tiles are fewer than the resident waves (the
    // population has thinned) they land one per SIMD rather than wherever
    // the queue's atomics happen to be served first.
    const int nwaves = (int)(gridDim.x * (blockDim.x >> 6));
    int first = (int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
    for (;;) {
        int t = 0;
        if (first >= 0) {
            t = first;
            first = -1;
            // (a single round: every tile is some wavefront's first)
            if (ntiles > P.simds && ntiles <= min(2 * P.simds, nwaves) && t < ntiles)
                t = place_tile(t, ntiles, P.simds);
        } else {
            if (lane == 0)
                t = nwaves + atomicAdd(head, 1);
            t = __builtin_amdgcn_readfirstlane(t);
        }
        if (t >= ntiles)
            break;
        const Tile T = tiles[t];
        const Bucket B = buckets[T.bucket];
        int slot = 0;
        bool keep;
        if constexpr (CLS == 2)
            keep = run_rolled_tile(B, T, lists, P, slot);
        else
            keep = run_tile<ADV, CLS == 1>(B, T, lists, P, slot);
        if (COMPACT)
            append_survivors(AL, T.bucket, keep, slot);
    }
}

template <bool ADV, bool COMPACT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void k_persistent(const Bucket *__restrict__ buckets, const Tile *__restrict__ tiles,
                  const int *__restrict__ ntiles_p, int *__restrict__ head, const int *lists,
                  StepParams P, ActiveLists AL)
{
    persistent_body<ADV, COMPACT, 0>(buckets, tiles, ntiles_p, head, lists, P, AL);
}

template <bool ADV, bool COMPACT>
__global__ __launch_bounds__(256) void k_persistent_spl(const Bucket *__restrict__ buckets,
                                                        const Tile *__restrict__ tiles,
                                                        const int *__restrict__ ntiles_p,
                                                        int *__restrict__ head,
                                                        const int *lists, StepParams P,
                                                        ActiveLists AL)
{
    persistent_body<ADV, COMPACT, 1>(buckets, tiles, ntiles_p, head, lists, P, AL);
}

// Fixed steps with stop rules of kMinRolled bodies and more, where the tiles give
// a SIMD more than two wavefronts: three, rolled (persistent_class), since two have
// no room for the partners' state of 11 bodies and more beside that of the rules
// and run rolled too.  60 steps, this class and the other, 40000 systems of 10..16 bodies 1742 and
// 1945 us, compacted every 10 steps 1969 and 2282; 32000 of 10 846 and 1020; 16000 of
// 16 1012 and 1157.  9 bodies alone stay with the other (16000 systems 460 and 381,
// 70000 1445 and 1288), but not beside larger ones: 40000 of 9..16 1728 and 1841.
template <bool COMPACT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
void k_persistent_rolled(const Bucket *__restrict__ buckets, const Tile *__restrict__ tiles,
                         const int *__restrict__ ntiles_p, int *__restrict__ head, const int *lists,
                         StepParams P, ActiveLists AL)
{
    persistent_body<true, COMPACT, 2>(buckets, tiles, ntiles_p, head, lists, P, AL);
}

// Tiles for the next quantum from the survivor counts (one workgroup):
// buckets in the given order (longest work first), tiles of each bucket in
// list order; resets the queue head and the other list's counts.
__global__ void k_build_tiles(const Bucket *__restrict__ buckets, int nb,
                              const int *__restrict__ order, const int *__restrict__ mapping,
                              ActiveLists AL, Tile *__restrict__ tiles, int *ntiles,
                              int *head)
{
    __shared__ int start[kMaxBodies + 2];
    __shared__ int cap[kMaxBodies + 2];
    if (threadIdx.x == 0) {
        int acc = 0;
        for (int i = 0; i < nb; ++i) {
            const int bk = order[i];
            const int n = buckets[bk].n;
            const int c = tile_systems(mapping[bk], n);
            cap[i] = c;
            start[i] = acc;
            acc += (AL.cur_count[bk] + c - 1) / c;
        }
        start[nb] = acc;
        *ntiles = acc;
        *head = 0;
    }
    __syncthreads();
    for (int i = 0; i < nb; ++i) {
        const int bk = order[i];
        const int n = buckets[bk].n;
        const int cnt = AL.cur_count[bk];
        const int c = cap[i];
        for (int t = threadIdx.x; t < start[i + 1] - start[i]; t += blockDim.x) {
            Tile T;
            T.bucket = bk;
            T.first = AL.base[bk] + t * c;
            T.count = min(c, cnt - t * c);
            T.kind = mapping[bk] * 32 + n;
            tiles[start[i] + t] = T;
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nb; i += blockDim.x)
        AL.next_count[order[i]] = 0;
}

__global__ void k_fill_int(int *p, int n, int value)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        p[i] = value;
}

// ---------------------------------------------------------------------------
// set-up, run control, layout and diagnostics kernels (one thread per slot)
// ---------------------------------------------------------------------------

template <int N>
__device__ __forceinline__ void load_xv(const Bucket &B, int s, double (&m)[N], double (&x)[N][3],
                                        double (&v)[N][3])
{
    const size_t pitch = B.pitch;
#pragma unroll
    for (int b = 0; b < N; ++b) {
        m[b] = B.st[(R_M * N + b) * pitch + s];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            x[b][c] = B.st[((R_X + c) * N + b) * pitch + s];
            v[b][c] = B.st[((R_V + c) * N + b) * pitch + s];
        }
    }
}

// Start of a run with adaptive steps (one thread per slot): the clock, and the
// step proposed from the current state when none is carried yet.  One wavefront a
// workgroup, told to the compiler, so that a system's bodies fit the registers
// (6000 x 16 bodies 52 us with the default bound and its scratch, 12 without).
template <int N>
__global__ __launch_bounds__(64) void k_begin_run(Bucket B, RunStart run)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= B.count)
        return;
    if (!begin_run_clock(B, s, B.status[s], B.t[s], run))
        return;
    double m[N], x[N][3], v[N][3], a[N][3], jk[N][3];
    load_xv<N>(B, s, m, x, v);
    if (run.adaptive == 2) {
        const size_t pitch = B.pitch;
#pragma unroll
        for (int b = 0; b < N; ++b)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                a[b][c] = B.st[((R_A + c) * N + b) * pitch + s];
                jk[b][c] = B.st[((R_J + c) * N + b) * pitch + s];
            }
        B.dtn[s] = paper_dt<N>(a, jk, run.eta);
    } else {
        double w = 0.0;
        spl_accjerk<N, true>(m, x, v, a, jk, w);
        B.dtn[s] = run.eta * rsqrt_nr(w);
    }
}

template <int N>
__device__ __forceinline__ void from_mvs(const double (&m)[N], double (&x)[N][3], double (&v)[N][3]);

// Energy (Eq. 6, each pair once) and angular momentum about the origin of
// one system.
template <int N>
__device__ __forceinline__ void sys_energy(const double (&m)[N], const double (&x)[N][3],
                                          const double (&v)[N][3], double &energy,
                                          double (&L)[3])
{
    double kin = 0.0, pot = 0.0, L0 = 0.0, L1 = 0.0, L2 = 0.0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        kin += 0.5 * m[i] * fma(v[i][2], v[i][2], fma(v[i][1], v[i][1], v[i][0] * v[i][0]));
        L0 += m[i] * (x[i][1] * v[i][2] - x[i][2] * v[i][1]);
        L1 += m[i] * (x[i][2] * v[i][0] - x[i][0] * v[i][2]);
        L2 += m[i] * (x[i][0] * v[i][1] - x[i][1] * v[i][0]);
    }
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = i + 1; j < N; ++j) {
            const double dx = x[i][0] - x[j][0], dy = x[i][1] - x[j][1], dz = x[i][2] - x[j][2];
            pot += m[i] * m[j] / sqrt(fma(dz, dz, fma(dy, dy, dx * dx)));
        }
    energy = kin - pot;
    L[0] = L0;
    L[1] = L1;
    L[2] = L2;
}

// Energy and angular momentum of one system in inertial form or (MVS) in MVS
// form, converted first.
template <int N, bool MVS>
__device__ __forceinline__ void diag_run(const Bucket &B, const int s, double *energy,
                                         double *angmom)
{
    double m[N], x[N][3], v[N][3];
    load_xv<N>(B, s, m, x, v);
    if (MVS)
        from_mvs<N>(m, x, v);
    double E, L[3];
    sys_energy<N>(m, x, v, E, L);
    const int o = B.orig[s];
    if (energy)
        energy[o] = E;
    if (angmom) {
        angmom[3 * o + 0] = L[0];
        angmom[3 * o + 1] = L[1];
        angmom[3 * o + 2] = L[2];
    }
}

// Of every system of a set of buckets, 64 a workgroup.
template <bool MVS>
__global__ __launch_bounds__(64) void k_diag(BucketSet set, double *energy, double *angmom)
{
    const int tile = blockIdx.x;
    int k = 0;
    while (k < set.count && tile >= set.first[k + 1])
        ++k;
    if (k >= set.count)
        return;
    const Bucket B = set.b[k];
    const int s = (tile - set.first[k]) * 64 + threadIdx.x;
    if (s >= B.count)
        return;
    switch (B.n) {
#define FB_C(NN) case NN: diag_run<NN, MVS>(B, s, energy, angmom); break;
        FB_C(2) FB_C(3) FB_C(4) FB_C(5) FB_C(6) FB_C(7) FB_C(8) FB_C(9) FB_C(10) FB_C(11)
        FB_C(12) FB_C(13) FB_C(14) FB_C(15) FB_C(16)
#undef FB_C
    default: break;
    }
}

// Monitor record k of every system of a bucket (Section 4.3's logging, with
// Section 4.4's data reduction), into the caller's log buffer:
//   kind 0 (state):  system o's block starts at max_records (o + 6 off[o])
//                    doubles; record k holds t, then pos [n][3], vel [n][3];
//   kind 1 (RV):     [o][k][2] = t and the star's velocity relative to the
//                    system's centre of mass along the unit line of sight l;
//   kind 2 (energy): [o][k][5] = t, E, L.
// Bound as k_begin_run (a record of 6000 x 14 bodies 37 us with scratch, 9.5 without).
template <int N>
__global__ __launch_bounds__(64) void k_log(Bucket B, const long long *__restrict__ orig_off, int kind, double lx,
                      double ly, double lz, int k, int max_records, double *out)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= B.count)
        return;
    double m[N], x[N][3], v[N][3];
    load_xv<N>(B, s, m, x, v);
    const int o = B.orig[s];
    const double t = B.t[s];
    if (kind == 1) {
        double M = 0.0, p0 = 0.0, p1 = 0.0, p2 = 0.0;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            M += m[i];
            p0 = fma(m[i], v[i][0], p0);
            p1 = fma(m[i], v[i][1], p1);
            p2 = fma(m[i], v[i][2], p2);
        }
        const double rv = fma(v[0][2] - p2 / M, lz, fma(v[0][1] - p1 / M, ly, (v[0][0] - p0 / M) * lx));
        double *r = out + ((size_t)o * max_records + k) * 2;
        r[0] = t;
        r[1] = rv;
    } else if (kind == 2) {
        double E, L[3];
        sys_energy<N>(m, x, v, E, L);
        double *r = out + ((size_t)o * max_records + k) * 5;
        r[0] = t;
        r[1] = E;
        r[2] = L[0];
        r[3] = L[1];
        r[4] = L[2];
    } else {
        double *r = out + (size_t)max_records * ((size_t)o + 6 * (size_t)orig_off[o]) +
                    (size_t)k * (1 + 6 * N);
        r[0] = t;
#pragma unroll
        for (int b = 0; b < N; ++b)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                r[1 + 3 * b + c] = x[b][c];
                r[1 + 3 * N + 3 * b + c] = v[b][c];
            }
    }
}

__global__ void k_count_active(Bucket B, int *count)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    const bool act = s < B.count && B.status[s] == ST_ACTIVE;
    const unsigned long long mask = __ballot(act);
    if ((threadIdx.x & 63) == 0 && mask)
        atomicAdd(count, __popcll(mask));
}

// ---------------------------------------------------------------------------
// mixed-variable symplectic (MVS) integrator, Sections 2.2.3 and 4.3.3
// ---------------------------------------------------------------------------
// The paper's five sub-steps (Cartesian drift half step, kick half step,
// Keplerian drift step, kick half step, Cartesian drift half step) are the
// democratic heliocentric splitting (Duncan, Levison & Lee 1998): planets
// move on Kepler orbits about the star with mu = m0 in heliocentric
// positions Q_i = x_i - x_0 and barycentric velocities V_i; kicks apply the
// planet-planet forces only; the drift moves every Q_i by the star's reflex
// motion, dt sum_j m_j V_j / m0, and the centre of mass by dt Vc.
//
// A bucket in MVS form keeps body 0's x and v rows for the centre of mass X
// and its velocity Vc, body i's rows for Q_i and V_i, and the a rows for the
// planet-planet accelerations at Q, which the next step's first kick reuses:
// the drifts move all Q_i together, so the separations do not change.

// MVS form -> inertial in place: x_0 = X - sum m_i Q_i / M, x_i = x_0 + Q_i,
// v_0 = Vc - sum m_i V_i / m0, v_i = Vc + V_i.
template <int N>
__device__ __forceinline__ void from_mvs(const double (&m)[N], double (&x)[N][3], double (&v)[N][3])
{
    double M = 0.0;
#pragma unroll
    for (int i = 0; i < N; ++i)
        M += m[i];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        double sq = 0.0, sp = 0.0;
#pragma unroll
        for (int i = 1; i < N; ++i) {
            sq = fma(m[i], x[i][c], sq);
            sp = fma(m[i], v[i][c], sp);
        }
        const double x0 = x[0][c] - sq / M, Vc = v[0][c];
        x[0][c] = x0;
        v[0][c] = Vc - sp / m[0];
#pragma unroll
        for (int i = 1; i < N; ++i) {
            x[i][c] += x0;
            v[i][c] += Vc;
        }
    }
}

template <int N>
__global__ __launch_bounds__(64) void k_mvs_leave(Bucket B)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= B.count)
        return;
    double m[N], x[N][3], v[N][3], a[N][3];
    load_rows<N>(B, s, m, x, v, a, false);
    from_mvs<N>(m, x, v);
    store_rows<N>(B, s, x, v, a, false);
}

// ---------------------------------------------------------------------------
// large systems (n > 16): one body per lane across a whole workgroup
// ---------------------------------------------------------------------------
// Section 4.2's second gravitation variant, for larger n.  Every lane owns
// one body and sums all n-1 of that body's interactions itself, so each pair
// is evaluated twice (once from either side) and the workgroup's LDS holds
// only the bodies' evaluation state, never per-pair terms.  S = floor(T / n)
// systems share a workgroup of T lanes (lane = system * n + body); a body's
// partners are LDS broadcasts to the lanes of its system.  Two copies of the
// evaluation state alternate, so an evaluation costs one workgroup barrier: a
// lane overwrites a copy only after the next evaluation's barrier, which
// every reader of that copy has passed.

// One interaction of body i with the partner at LDS index idx of one copy
// (Eq. 1 and its time derivative; the terms of bpl_interact).
__device__ __forceinline__ void large_interact(const double2 *__restrict__ xy,
                                               const double2 *__restrict__ zvx,
                                               const double2 *__restrict__ vyvz,
                                               const double *__restrict__ mm, const int idx,
                                               const double (&xi)[3], const double (&vi)[3],
                                               double (&a)[3], double (&jk)[3])
{
    const double2 p0 = xy[idx];
    const double2 p1 = zvx[idx];
    const double2 p2 = vyvz[idx];
    const double mj = mm[idx];
    const double rx = p0.x - xi[0], ry = p0.y - xi[1], rz = p1.x - xi[2];
    const double ux = p1.y - vi[0], uy = p2.x - vi[1], uz = p2.y - vi[2];
    const double r2 = fma(rz, rz, fma(ry, ry, rx * rx));
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
}

// Publish this lane's state in copy `cp`, wait for the workgroup, and (live
// lanes) sum the body's interactions: the other planets in ascending order,
// then the star (the star's lane sums planets 1..n-1).
__device__ __forceinline__ void large_eval(const LargeView &V, const int T, const int cp,
                                           const int tid, const int base, const int b,
                                           const int n, const bool live, const double (&xi)[3],
                                           const double (&vi)[3], double (&a)[3],
                                           double (&jk)[3])
{
    const double2 *xy = V.xy + cp * T;
    const double2 *zvx = V.zvx + cp * T;
    const double2 *vyvz = V.vyvz + cp * T;
    V.xy[cp * T + tid] = make_double2(xi[0], xi[1]);
    V.zvx[cp * T + tid] = make_double2(xi[2], vi[0]);
    V.vyvz[cp * T + tid] = make_double2(vi[1], vi[2]);
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        a[c] = 0.0;
        jk[c] = 0.0;
    }
    if (!live)
        return;
    const int skip = b == 0 ? INT_MAX : b;
#pragma unroll 4
    for (int k = 0; k < n - 2; ++k) {
        const int j = k + 1 + (k + 1 >= skip ? 1 : 0);
        large_interact(xy, zvx, vyvz, V.m, base + j, xi, vi, a, jk);
    }
    large_interact(xy, zvx, vyvz, V.m, base + (b == 0 ? n - 1 : 0), xi, vi, a, jk);
}

// Algorithm 1's "prepare" for large n: (a0, j0) at the current state.
__global__ __launch_bounds__(kLargeMaxLanes) void k_prepare_large(Bucket B, int S)
{
    const int T = blockDim.x, n = B.n;
    const LargeView V = large_view(T);
    const LargeLane l = large_lane(B, S);
    const size_t pitch = B.pitch;
    double mi = 0.0, x[3] = {0.0, 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0};
    if (l.valid) {
        mi = B.st[(R_M * n + l.b) * pitch + l.slot];
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            x[cc] = B.st[((R_X + cc) * n + l.b) * pitch + l.slot];
            v[cc] = B.st[((R_V + cc) * n + l.b) * pitch + l.slot];
        }
    }
    V.m[l.tid] = mi;
    double a[3], jk[3];
    large_eval(V, T, 0, l.tid, l.base, l.b, n, l.valid, x, v, a, jk);
    if (!l.valid)
        return;
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) {
        B.st[((R_A + cc) * n + l.b) * pitch + l.slot] = a[cc];
        B.st[((R_J + cc) * n + l.b) * pitch + l.slot] = jk[cc];
    }
}

// Per-system sums over the bodies of a large-n workgroup, in body order, on
// the star's lane: lane values q[0..4] go through copy 1 of the state arrays.
__device__ __forceinline__ void large_sum5(const LargeView &V, const int T, const LargeLane &l,
                                           const int n, const double (&q)[5], double (&out)[5])
{
    double2 *r0 = V.xy + T, *r1 = V.zvx + T, *r2 = V.vyvz + T;
    r0[l.tid] = make_double2(q[0], q[1]);
    r1[l.tid] = make_double2(q[2], q[3]);
    r2[l.tid] = make_double2(q[4], 0.0);
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 5; ++c)
        out[c] = 0.0;
    if (!l.valid || l.b != 0)
        return;
    for (int k = 0; k < n; ++k) {
        const double2 p = r0[l.base + k], u = r1[l.base + k], w = r2[l.base + k];
        out[0] += p.x;
        out[1] += p.y;
        out[2] += u.x;
        out[3] += u.y;
        out[4] += w.x;
    }
}

// Energy (Eq. 6) and angular momentum parts of this lane's body: its kinetic
// energy, the potential of its pairs with higher-numbered partners (each pair
// once) and m x cross v.
__device__ __forceinline__ void large_energy_terms(const LargeView &V, const int T,
                                                   const LargeLane &l, const int n,
                                                   const double mi, const double (&x)[3],
                                                   const double (&v)[3], double (&q)[5])
{
    V.m[l.tid] = mi;
    V.xy[l.tid] = make_double2(x[0], x[1]);
    V.zvx[l.tid] = make_double2(x[2], 0.0);
    __syncthreads();
    double pot = 0.0;
    if (l.valid)
        for (int j = l.b + 1; j < n; ++j) {
            const double2 p0 = V.xy[l.base + j], p1 = V.zvx[l.base + j];
            const double dx = x[0] - p0.x, dy = x[1] - p0.y, dz = x[2] - p1.x;
            pot += V.m[l.base + j] / sqrt(fma(dz, dz, fma(dy, dy, dx * dx)));
        }
    q[0] = 0.5 * mi * fma(v[2], v[2], fma(v[1], v[1], v[0] * v[0])) - mi * pot;
    q[1] = 0.0;
    q[2] = mi * (x[1] * v[2] - x[2] * v[1]);
    q[3] = mi * (x[2] * v[0] - x[0] * v[2]);
    q[4] = mi * (x[0] * v[1] - x[1] * v[0]);
}

__device__ __forceinline__ void large_load_xv(const Bucket &B, const LargeLane &l, double &mi,
                                              double (&x)[3], double (&v)[3])
{
    mi = 0.0;
    const size_t pitch = B.pitch;
    const int n = B.n;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        x[c] = 0.0;
        v[c] = 0.0;
    }
    if (!l.valid)
        return;
    mi = B.st[(R_M * n + l.b) * pitch + l.slot];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        x[c] = B.st[((R_X + c) * n + l.b) * pitch + l.slot];
        v[c] = B.st[((R_V + c) * n + l.b) * pitch + l.slot];
    }
}

// Run start of a large-n bucket (one body per lane): the clock part on the
// star's lane, then, for systems that need one, the first adaptive step from
// the stored (a0, j0) (Eq. 5) or from the pairwise rule at the current state
// (the proposals of k_begin_run).
__global__ __launch_bounds__(kLargeMaxLanes) void k_begin_run_large(Bucket B, int S, RunStart run)
{
    const int adaptive = run.adaptive;
    const int T = blockDim.x, n = B.n;
    const LargeView V = large_view(T);
    const LargeLane l = large_lane(B, S);
    if (l.valid && l.b == 0)
        V.flag[l.base] = begin_run_clock(B, l.slot, B.status[l.slot], B.t[l.slot], run);
    __syncthreads();
    const bool need = l.valid && V.flag[l.base] != 0;
    if (!__syncthreads_or(need))
        return;
    const size_t pitch = B.pitch;
    double mi, x[3], v[3];
    large_load_xv(B, l, mi, x, v);
    double q = 0.0;
    if (adaptive == 2) {
        if (l.valid) {
            double a[3], jk[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                a[c] = B.st[((R_A + c) * n + l.b) * pitch + l.slot];
                jk[c] = B.st[((R_J + c) * n + l.b) * pitch + l.slot];
            }
            q = fma(jk[2], jk[2], fma(jk[1], jk[1], jk[0] * jk[0])) /
                fma(a[2], a[2], fma(a[1], a[1], a[0] * a[0]));
        }
    } else {
        V.m[l.tid] = mi;
        V.xy[l.tid] = make_double2(x[0], x[1]);
        V.zvx[l.tid] = make_double2(x[2], v[0]);
        V.vyvz[l.tid] = make_double2(v[1], v[2]);
        __syncthreads();
        if (l.valid) {
            for (int j = 0; j < n; ++j) {
                if (j == l.b)
                    continue;
                const double2 p0 = V.xy[l.base + j], p1 = V.zvx[l.base + j],
                              p2 = V.vyvz[l.base + j];
                const double rx = p0.x - x[0], ry = p0.y - x[1], rz = p1.x - x[2];
                const double ux = p1.y - v[0], uy = p2.x - v[1], uz = p2.y - v[2];
                const double r2 = fma(rz, rz, fma(ry, ry, rx * rx));
                const double ru = fma(rz, uz, fma(ry, uy, rx * ux));
                const double u2 = fma(uz, uz, fma(uy, uy, ux * ux));
                const double ri = rsqrt_nr(r2);
                const double ri2 = ri * ri;
                const double al = 3.0 * ru * ri2;
                q = fmax(q, fma(al, ru, u2) * ri2);
            }
        }
    }
    V.red[l.tid] = q;
    __syncthreads();
    if (need && l.b == 0) {
        double r = V.red[l.base];
        for (int b = 1; b < n; ++b)
            r = adaptive == 2 ? r + V.red[l.base + b] : fmax(r, V.red[l.base + b]);
        B.dtn[l.slot] = run.eta * rsqrt_nr(r);
    }
}

__device__ __forceinline__ void large_from_mvs(const LargeView &V, const int T, const LargeLane &l,
                                               const int n, const double mi, double (&x)[3],
                                               double (&v)[3]);

// Energy and angular momentum of every system of a large-n bucket, in
// inertial form or (MVS) in MVS form, converted first.
template <bool MVS>
__global__ __launch_bounds__(kLargeMaxLanes) void k_diag_large(Bucket B, int S, double *energy,
                                                     double *angmom)
{
    const int T = blockDim.x;
    const LargeView V = large_view(T);
    const LargeLane l = large_lane(B, S);
    double mi, x[3], v[3], q[5], sum[5];
    large_load_xv(B, l, mi, x, v);
    if (MVS) {
        V.m[l.tid] = mi;
        large_from_mvs(V, T, l, B.n, mi, x, v);
    }
    large_energy_terms(V, T, l, B.n, mi, x, v, q);
    large_sum5(V, T, l, B.n, q, sum);
    if (!l.valid || l.b != 0)
        return;
    const int o = B.orig[l.slot];
    if (energy)
        energy[o] = sum[0];
    if (angmom) {
        angmom[3 * o + 0] = sum[2];
        angmom[3 * o + 1] = sum[3];
        angmom[3 * o + 2] = sum[4];
    }
}

// Monitor record k of every system of a large-n bucket (layouts of k_log).
__global__ __launch_bounds__(kLargeMaxLanes) void k_log_large(Bucket B, int S,
                                                    const long long *__restrict__ orig_off,
                                                    int kind, double lx, double ly, double lz,
                                                    int k, int max_records, double *out)
{
    const int T = blockDim.x, n = B.n;
    const LargeView V = large_view(T);
    const LargeLane l = large_lane(B, S);
    double mi, x[3], v[3], q[5], sum[5];
    large_load_xv(B, l, mi, x, v);
    const int o = l.valid ? B.orig[l.slot] : 0;
    const double t = l.valid ? B.t[l.slot] : 0.0;
    if (kind == 0) {
        if (!l.valid)
            return;
        double *r = out + (size_t)max_records * ((size_t)o + 6 * (size_t)orig_off[o]) +
                    (size_t)k * (1 + 6 * n);
        if (l.b == 0)
            r[0] = t;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            r[1 + 3 * l.b + c] = x[c];
            r[1 + 3 * n + 3 * l.b + c] = v[c];
        }
        return;
    }
    if (kind == 1) {
        q[0] = mi;
        q[1] = mi * v[0];
        q[2] = mi * v[1];
        q[3] = mi * v[2];
        q[4] = 0.0;
    } else {
        large_energy_terms(V, T, l, n, mi, x, v, q);
    }
    large_sum5(V, T, l, n, q, sum);
    if (!l.valid || l.b != 0)
        return;
    if (kind == 1) {
        const double rv = fma(v[2] - sum[3] / sum[0], lz,
                              fma(v[1] - sum[2] / sum[0], ly, (v[0] - sum[1] / sum[0]) * lx));
        double *r = out + ((size_t)o * max_records + k) * 2;
        r[0] = t;
        r[1] = rv;
    } else {
        double *r = out + ((size_t)o * max_records + k) * 5;
        r[0] = t;
        r[1] = sum[0];
        r[2] = sum[2];
        r[3] = sum[3];
        r[4] = sum[4];
    }
}

// ---------------------------------------------------------------------------
// MVS for larger systems (9..512 bodies): one body per lane across a workgroup
// ---------------------------------------------------------------------------
// The sub-steps of Section 2.2.3 as in k_plain_mvs, laid out like the large-n
// Hermite kernels: each planet's lane drifts it along its own Kepler orbit,
// the planet-planet accelerations are one-sided partner loops over LDS
// broadcasts (planets in ascending order; the same values as the paired
// form), and the sums over a system (the drift's momentum, the centre of
// mass) are fma chains in body order on the star's lane, broadcast through
// LDS.  Every lane reaches every barrier: a system's outcome (unbound,
// Kepler failure) predicates its updates, never the control flow.

// MVS form -> inertial (x, v) of this lane's body (from_mvs): x_0 = X -
// sum m_i Q_i / M, x_i = Q_i + x_0, v_0 = Vc - sum m_i V_i / m_0,
// v_i = V_i + Vc.  V.m must hold the masses.
__device__ __forceinline__ void large_from_mvs(const LargeView &V, const int T, const LargeLane &l,
                                               const int n, const double mi, double (&x)[3],
                                               double (&v)[3])
{
    const double one[3] = {mi, 0.0, 0.0};
    double Ms[3], st[3], sq[3], X[3], sp[3], Vc[3];
    large_sys_wsum3(V, T, l, n, 0, 1.0, one, Ms, st);
    large_sys_wsum3(V, T, l, n, 1, mi, x, sq, X);
    large_sys_wsum3(V, T, l, n, 1, mi, v, sp, Vc);
    const double M = Ms[0], m0 = l.valid ? V.m[l.base] : 1.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double x0 = X[c] - sq[c] / M;
        if (l.b == 0) {
            x[c] = x0;
            v[c] = Vc[c] - sp[c] / m0;
        } else {
            x[c] += x0;
            v[c] += Vc[c];
        }
    }
}

// Inertial -> MVS form of a bucket (X, Vc in row 0, Q_i = x_i - x_0, V_i = v_i - Vc), with the planet-planet
// accelerations at Q in the a0 rows.
__global__ __launch_bounds__(kLargeMaxLanes) void k_mvs_enter_large(Bucket B, int S)
{
    const int T = blockDim.x, n = B.n;
    const LargeView V = large_view(T);
    const LargeLane l = large_lane(B, S);
    double mi, x[3], v[3], a[3];
    large_load_rows(B, l, mi, x, v, a);
    V.m[l.tid] = mi;
    const double one[3] = {mi, 0.0, 0.0};
    double Ms[3], st[3], sx[3], x0[3], sv[3], v0[3];
    large_sys_wsum3(V, T, l, n, 0, 1.0, one, Ms, st);
    large_sys_wsum3(V, T, l, n, 0, mi, x, sx, x0);
    large_sys_wsum3(V, T, l, n, 0, mi, v, sv, v0);
    const double M = Ms[0];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double X = sx[c] / M, Vc = sv[c] / M;
        if (l.b == 0) {
            x[c] = X;
            v[c] = Vc;
        } else {
            x[c] -= x0[c];
            v[c] -= Vc;
        }
    }
    large_mvs_acc(V, l, n, x, a);
    large_store_rows(B, l, x, v, a, true);
}

// MVS form -> inertial of a bucket (from_mvs); the a0 rows are left as they are.
__global__ __launch_bounds__(kLargeMaxLanes) void k_mvs_leave_large(Bucket B, int S)
{
    const int T = blockDim.x;
    const LargeView V = large_view(T);
    const LargeLane l = large_lane(B, S);
    double mi, x[3], v[3], a[3];
    large_load_rows(B, l, mi, x, v, a);
    V.m[l.tid] = mi;
    large_from_mvs(V, T, l, B.n, mi, x, v);
    large_store_rows(B, l, x, v, a, false);
}

// State read-back of a bucket in MVS form, converted to inertial (x, v) on
// the way out.
__global__ __launch_bounds__(kLargeMaxLanes) void k_unpack_mvs_large(Bucket B, int S, StateOut out)
{
    const int T = blockDim.x;
    const LargeView V = large_view(T);
    const LargeLane l = large_lane(B, S);
    double mi, x[3], v[3], a[3];
    large_load_rows(B, l, mi, x, v, a);
    V.m[l.tid] = mi;
    large_from_mvs(V, T, l, B.n, mi, x, v);
    if (!l.valid)
        return;
    const int o = B.orig[l.slot];
    const long long base = out.orig_off[o];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const size_t row = 3 * (base + l.b) + c;
        if (out.pos) out.pos[row] = x[c];
        if (out.vel) out.vel[row] = v[c];
    }
    if (l.b == 0) {
        if (out.t) out.t[o] = B.t[l.slot];
        if (out.status) out.status[o] = B.status[l.slot];
        if (out.steps) out.steps[o] = B.steps[l.slot];
    }
}

// FP64 issue-ceiling probe for the roofline: each lane runs kFmaChains
// independent FMA chains (a <- a*b + c, b slightly below 1 so values stay
// bounded), so the rate is set by VALU issue rather than FMA latency.
constexpr int kFmaChains = 16;

__global__ __launch_bounds__(256) void k_fma_probe(double *out, int iters, double b, double c)
{
    double acc[kFmaChains];
#pragma unroll
    for (int k = 0; k < kFmaChains; ++k)
        acc[k] = 1e-3 * threadIdx.x + k;
    for (int i = 0; i < iters; ++i) {
#pragma unroll
        for (int k = 0; k < kFmaChains; ++k)
            acc[k] = fma(acc[k], b, c);
    }
    double sum = 0.0;
#pragma unroll
    for (int k = 0; k < kFmaChains; ++k)
        sum += acc[k];
    out[(size_t)blockIdx.x * blockDim.x + threadIdx.x] = sum;
}

// The device reciprocal square root of every pair evaluation, elementwise
// over n values (a check of its accuracy against a correctly rounded
// reference).
__global__ void k_rsqrt(const double *__restrict__ in, double *__restrict__ out, long long n)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        out[i] = rsqrt_nr(in[i]);
}

// Checkpoint restore: the carried (a0, j0) rows and each system's clock
// (adaptive step, steps since creation, status) from caller-order arrays.
// Positions, velocities, masses and t were packed already.
__global__ void k_restore(Bucket B, const long long *__restrict__ orig_off,
                          const double *__restrict__ acc, const double *__restrict__ jerk,
                          const double *__restrict__ dtn, const long long *__restrict__ steps,
                          const int *__restrict__ status)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= B.count)
        return;
    const size_t pitch = B.pitch;
    const int n = B.n;
    const int o = B.orig[s];
    const long long base = orig_off[o];
    for (int b = 0; b < n; ++b)
        for (int c = 0; c < 3; ++c) {
            const size_t row = 3 * (base + b) + c;
            B.st[((R_A + c) * n + b) * pitch + s] = acc[row];
            B.st[((R_J + c) * n + b) * pitch + s] = jerk[row];
        }
    B.dtn[s] = dtn[o];
    B.steps[s] = steps[o];
    B.status[s] = status[o];
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
#define FB_SWITCH_N(n, MACRO)                                                           \
    switch (n) {                                                                        \
    case 2: MACRO(2); break;  case 3: MACRO(3); break;  case 4: MACRO(4); break;        \
    case 5: MACRO(5); break;  case 6: MACRO(6); break;  case 7: MACRO(7); break;        \
    case 8: MACRO(8); break;  case 9: MACRO(9); break;  case 10: MACRO(10); break;      \
    case 11: MACRO(11); break; case 12: MACRO(12); break; case 13: MACRO(13); break;    \
    case 14: MACRO(14); break; case 15: MACRO(15); break; case 16: MACRO(16); break;    \
    default: return hipErrorInvalidValue;                                               \
    }

void large_shape(int n, int &T, int &S)
{
    T = 0;
    S = 0;
    long long best_used = -1, best_T = 1;
    for (int t = 64; t <= kLargeMaxLanes; t += 64) {
        const int s = t / n;
        if (s < 1)
            continue;
        // more of the lanes in use (s n / t), compared exactly; ties keep the smaller t
        if ((long long)s * n * best_T > best_used * t) {
            best_used = (long long)s * n;
            best_T = t;
            T = t;
            S = s;
        }
    }
}

hipError_t launch_prepare_large(const Bucket &B, hipStream_t s)
{
    if (B.count == 0)
        return hipSuccess;
    dim3 grid;
    int T, S;
    if (!large_launch(B, grid, T, S))
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_prepare_large, grid, dim3(T), large_lds_bytes(T), s, B, S);
    return hipGetLastError();
}

hipError_t launch_begin_adaptive(const Bucket &B, const RunStart &run, hipStream_t s)
{
    if (B.count == 0)
        return hipSuccess;
    if (B.n > kMaxBodies) {
        dim3 grid;
        int T, S;
        if (!large_launch(B, grid, T, S))
            return hipErrorInvalidValue;
        hipLaunchKernelGGL(k_begin_run_large, grid, dim3(T), large_lds_bytes(T), s, B, S, run);
        return hipGetLastError();
    }
#define FB_L(NN) hipLaunchKernelGGL(k_begin_run<NN>, grid_for(B.count, 64), dim3(64), 0, s, B, run)
    FB_SWITCH_N(B.n, FB_L)
#undef FB_L
    return hipGetLastError();
}

hipError_t launch_plain(const Bucket &B, int mapping, int waves_per_group, const StepParams &P,
                        hipStream_t s)
{
    if (B.count == 0)
        return hipSuccess;
    if (mapping == MAP_BPLU)   // (bpl_mapping)
        return launch_unrolled(B, P, s);
    if (mapping == MAP_SPLIT2 || mapping == MAP_SPLIT4)
        return launch_split(B, mapping == MAP_SPLIT4 ? 4 : 2, P, s);
    const int W = waves_per_group < 1 ? 1 : (waves_per_group > 4 ? 4 : waves_per_group);
    const bool adv = P.adaptive || P.stop_rules;
    if (mapping == MAP_SPL && B.n <= (adv ? kMaxSplAdv : kMaxSplBodies)) {
        const dim3 grid = grid_for(B.count, 64 * W);
#define FB_LA(NN)                                                                       \
    hipLaunchKernelGGL((k_plain_spl<NN, true>), grid, dim3(64 * W), spl_lds_bytes(NN) * W, \
                       s, B, P)
#define FB_LF(NN)                                                                       \
    hipLaunchKernelGGL((k_plain_spl<NN, false>), grid, dim3(64 * W), spl_lds_bytes(NN) * W, \
                       s, B, P)
        if (adv) {
            switch (B.n) {
            case 2: FB_LA(2); break;
            case 3: FB_LA(3); break;
            case 4: FB_LA(4); break;
            case 5: FB_LA(5); break;
            case 6: FB_LA(6); break;
            case 7: FB_LA(7); break;
            case 8: FB_LA(8); break;
            default: return hipErrorInvalidValue;
            }
        } else {
            switch (B.n) {
            case 2: FB_LF(2); break;
            case 3: FB_LF(3); break;
            case 4: FB_LF(4); break;
            case 5: FB_LF(5); break;
            case 6: FB_LF(6); break;
            case 7: FB_LF(7); break;
            case 8: FB_LF(8); break;
            case 9: FB_LF(9); break;
            case 10: FB_LF(10); break;
            default: return hipErrorInvalidValue;
            }
        }
#undef FB_LA
#undef FB_LF
        return hipGetLastError();
    }
    const int S = 64 / B.n;
    const int tiles = (B.count + S - 1) / S;
    const dim3 grid((unsigned)((tiles + W - 1) / W));
    const size_t lds = sizeof(BplLds) * W;
#define FB_L(NN, ADV) case NN: hipLaunchKernelGGL((k_plain_bpl<NN, ADV>), grid, dim3(64 * W), lds, s, B, P); break
#define FB_LN(ADV)                                                                         \
    switch (B.n) {                                                                         \
        FB_L(2, ADV); FB_L(3, ADV); FB_L(4, ADV); FB_L(5, ADV); FB_L(6, ADV); FB_L(7, ADV); \
        FB_L(8, ADV); FB_L(9, ADV); FB_L(10, ADV); FB_L(11, ADV); FB_L(12, ADV);           \
        FB_L(13, ADV); FB_L(14, ADV); FB_L(15, ADV); FB_L(16, ADV);                        \
    default: return hipErrorInvalidValue;                                                  \
    }
    if (adv) {
        FB_LN(true)
    } else {
        FB_LN(false)
    }
#undef FB_LN
#undef FB_L
    return hipGetLastError();
}

size_t persistent_lds_bytes(int cls, int waves_per_group)
{
    const size_t per_wave = cls == 1 ? kWideLdsStride : sizeof(BplLds);
    return per_wave * waves_per_group;
}

int persistent_max_groups_per_cu(int adv, int cls, int waves_per_group)
{
    int blocks = 0;
    const int threads = 64 * waves_per_group;
    const size_t lds = persistent_lds_bytes(cls, waves_per_group);
    hipError_t e;
    if (cls == 2)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, k_persistent_rolled<true>, threads, lds);
    else if (cls == 1)
        e = adv ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, k_persistent_spl<true, true>,
                                                               threads, lds)
                : hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, k_persistent_spl<false, false>,
                                                               threads, lds);
    else
        e = adv ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, k_persistent<true, true>,
                                                               threads, lds)
                : hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, k_persistent<false, false>,
                                                               threads, lds);
    return e == hipSuccess ? blocks : 0;
}

hipError_t launch_persistent(const Bucket *d_buckets, const Tile *d_tiles, const int *d_ntiles,
                             int *d_head, const int *d_lists, const StepParams &P, int adv,
                             int cls, int grid, int waves_per_group, ActiveLists *compact,
                             hipStream_t s)
{
    const int W = waves_per_group < 1 ? 1 : (waves_per_group > 4 ? 4 : waves_per_group);
    const size_t lds = persistent_lds_bytes(cls, W);
    ActiveLists AL = compact ? *compact : ActiveLists{nullptr, nullptr, nullptr, nullptr, nullptr};
    const dim3 g(grid), b(64 * W);
#define FB_P(KERNEL, ...)                                                                \
    hipLaunchKernelGGL((KERNEL<__VA_ARGS__>), g, b, lds, s, d_buckets, d_tiles, d_ntiles, d_head, \
                       d_lists, P, AL)
    if (cls == 2) {
        if (!adv)
            return hipErrorInvalidValue;
        if (compact) FB_P(k_persistent_rolled, true); else FB_P(k_persistent_rolled, false);
    } else if (cls == 1) {
        if (adv) {
            if (compact) FB_P(k_persistent_spl, true, true); else FB_P(k_persistent_spl, true, false);
        } else {
            if (compact) FB_P(k_persistent_spl, false, true); else FB_P(k_persistent_spl, false, false);
        }
    } else {
        if (adv) {
            if (compact) FB_P(k_persistent, true, true); else FB_P(k_persistent, true, false);
        } else {
            if (compact) FB_P(k_persistent, false, true); else FB_P(k_persistent, false, false);
        }
    }
#undef FB_P
    return hipGetLastError();
}

hipError_t launch_build_tiles(const Bucket *d_buckets, int n_buckets, const int *d_order,
                              const int *d_mapping, ActiveLists L, Tile *d_tiles, int *d_ntiles,
                              int *d_head, hipStream_t s)
{
    if (n_buckets < 0 || n_buckets > kMaxBodies + 1)   // the kernel's tables hold kMaxBodies + 2
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_build_tiles, dim3(1), dim3(256), 0, s, d_buckets, n_buckets, d_order,
                       d_mapping, L, d_tiles, d_ntiles, d_head);
    return hipGetLastError();
}

hipError_t launch_reset_counter(int *p, int n, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill_int, grid_for(n, 256), dim3(256), 0, s, p, n, 0);
    return hipGetLastError();
}

hipError_t launch_diag(const Bucket *b, int nb, double *energy, double *angmom, bool mvs_form,
                       hipStream_t s)
{
    BucketSet set;
    set.clear();
    for (int i = 0; i < nb; ++i) {
        const Bucket &B = b[i];
        if (B.count == 0)
            continue;
        if (B.n <= kMaxBodies) {   // at most one bucket of each n
            if (set.count == BucketSet::kMost)
                return hipErrorInvalidValue;
            set.add(B, (B.count + 63) / 64);
            continue;
        }
        dim3 grid;
        int T, S;
        if (!large_launch(B, grid, T, S))
            return hipErrorInvalidValue;
        if (mvs_form)
            hipLaunchKernelGGL(k_diag_large<true>, grid, dim3(T), large_lds_bytes(T), s, B, S,
                               energy, angmom);
        else
            hipLaunchKernelGGL(k_diag_large<false>, grid, dim3(T), large_lds_bytes(T), s, B, S,
                               energy, angmom);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    if (set.count == 0)
        return hipSuccess;
    const dim3 grid((unsigned)set.first[set.count]);
    if (mvs_form)
        hipLaunchKernelGGL(k_diag<true>, grid, dim3(64), 0, s, set, energy, angmom);
    else
        hipLaunchKernelGGL(k_diag<false>, grid, dim3(64), 0, s, set, energy, angmom);
    return hipGetLastError();
}

#define FB_SWITCH_MVS(n, MACRO)                                                         \
    switch (n) {                                                                        \
    case 2: MACRO(2); break;  case 3: MACRO(3); break;  case 4: MACRO(4); break;        \
    case 5: MACRO(5); break;  case 6: MACRO(6); break;  case 7: MACRO(7); break;        \
    case 8: MACRO(8); break;                                                            \
    default: return hipErrorInvalidValue;                                               \
    }
static_assert(kMaxMvsBodies == 8, "FB_SWITCH_MVS covers n = 2..kMaxMvsBodies");

hipError_t launch_mvs_enter_large(const Bucket &B, hipStream_t s)
{
    if (B.count == 0)
        return hipSuccess;
    dim3 grid;
    int T, S;
    if (!large_launch(B, grid, T, S))
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_mvs_enter_large, grid, dim3(T), large_lds_bytes(T), s, B, S);
    return hipGetLastError();
}

hipError_t launch_mvs_leave(const Bucket &B, hipStream_t s)
{
    if (B.count == 0)
        return hipSuccess;
    if (B.n > kMaxMvsBodies) {
        dim3 grid;
        int T, S;
        if (!large_launch(B, grid, T, S))
            return hipErrorInvalidValue;
        hipLaunchKernelGGL(k_mvs_leave_large, grid, dim3(T), large_lds_bytes(T), s, B, S);
        return hipGetLastError();
    }
#define FB_L(NN) hipLaunchKernelGGL(k_mvs_leave<NN>, grid_for(B.count, 64), dim3(64), 0, s, B)
    FB_SWITCH_MVS(B.n, FB_L)
#undef FB_L
    return hipGetLastError();
}

hipError_t launch_unpack_mvs_large(const Bucket &B, const StateOut &out, hipStream_t s)
{
    if (B.count == 0)
        return hipSuccess;
    dim3 grid;
    int T, S;
    if (!large_launch(B, grid, T, S))
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_unpack_mvs_large, grid, dim3(T), large_lds_bytes(T), s, B, S, out);
    return hipGetLastError();
}

hipError_t launch_count_active(const Bucket &B, int *count, hipStream_t s)
{
    if (B.count == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_count_active, grid_for(B.count, 256), dim3(256), 0, s, B, count);
    return hipGetLastError();
}

hipError_t launch_log(const Bucket &B, const long long *orig_off, int kind, const double *los,
                      int k, int max_records, double *out, hipStream_t s)
{
    if (B.count == 0)
        return hipSuccess;
    if (B.n > kMaxBodies) {
        dim3 grid;
        int T, S;
        if (!large_launch(B, grid, T, S))
            return hipErrorInvalidValue;
        hipLaunchKernelGGL(k_log_large, grid, dim3(T), large_lds_bytes(T), s, B, S, orig_off,
                           kind, los[0], los[1], los[2], k, max_records, out);
        return hipGetLastError();
    }
#define FB_L(NN) hipLaunchKernelGGL(k_log<NN>, grid_for(B.count, 64), dim3(64), 0, s, B, orig_off, \
                                    kind, los[0], los[1], los[2], k, max_records, out)
    FB_SWITCH_N(B.n, FB_L)
#undef FB_L
    return hipGetLastError();
}

hipError_t launch_fma_probe(double *out, int blocks, int iters, hipStream_t s)
{
    hipLaunchKernelGGL(k_fma_probe, dim3(blocks), dim3(256), 0, s, out, iters, 0.999999, 1e-6);
    return hipGetLastError();
}

hipError_t launch_rsqrt(const double *in, double *out, long long n, hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    const long long blocks = (n + 255) / 256;
    if (blocks > INT_MAX)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_rsqrt, dim3((unsigned)blocks), dim3(256), 0, s, in, out, n);
    return hipGetLastError();
}

hipError_t launch_restore(const Bucket &B, const long long *orig_off, const double *acc,
                          const double *jerk, const double *dtn, const long long *steps,
                          const int *status, hipStream_t s)
{
    if (B.count == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_restore, grid_for(B.count, 256), dim3(256), 0, s, B, orig_off, acc, jerk,
                       dtn, steps, status);
    return hipGetLastError();
}

}  // namespace fb
