// fb_large.hip -- Hermite steps of large systems (n > kMaxBodies), Section
// 4.2's second gravitation variant: every pair from either side, only
// per-body values in LDS.
#include "fb_bpl.h"

#include <algorithm>
#include <cmath>

namespace fb {
namespace {

// ---------------------------------------------------------------------------
// layout
// ---------------------------------------------------------------------------
// Lanes hold K bodies each and sum their interactions one partner after
// another (planets 1..n-1 in ascending order, then the star); or G (2, 4 or 8)
// lanes share them, so that a few systems still use the device: lane g of them
// sums the partners g, g + G, ... of that order, and the shares are added
// across the lanes in a binary tree (so a system's rounding depends on the
// layout, which n and the number of systems of that n choose; 16 lanes were
// never the fastest from 17 bodies up).  A system takes L = ceil(n / K) G
// consecutive lanes of a workgroup, which holds S systems.  The bodies'
// evaluation state sits in LDS in summation order as 48-byte records, so a
// partner is three ds_read_b128 at immediate offsets from one address; two
// copies alternate between the two evaluations of a step, so an evaluation
// costs one workgroup barrier.

// Position of body b in summation order.
__device__ __forceinline__ int large_slot(const int b, const int n)
{
    return b == 0 ? n - 1 : b - 1;
}

template <int CTRL>
__device__ __forceinline__ double dpp_read(const double v)
{
    const unsigned long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)(u & 0xffffffffull), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(u >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

constexpr int kRowHalfMirror = 0x141;
constexpr int kQuadXor2 = 2 | (3 << 2) | (0 << 4) | (1 << 6), kQuadXor1 = 1 | (0 << 2) | (3 << 4) | (2 << 6);

template <int CTRL>
__device__ __forceinline__ void large_add_lanes(double (&a)[3], double (&jk)[3])
{
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        a[c] += dpp_read<CTRL>(a[c]);
        jk[c] += dpp_read<CTRL>(jk[c]);
    }
}

template <int CTRL>
__device__ __forceinline__ double large_max_lanes(const double v)
{
    return fmax(v, dpp_read<CTRL>(v));
}

// Sums, and maximum, over the G lanes of a body, to all of them.
__device__ __forceinline__ void large_add_shares(const int G, double (&a)[3], double (&jk)[3])
{
    if (G >= 8)
        large_add_lanes<kRowHalfMirror>(a, jk);
    if (G >= 4)
        large_add_lanes<kQuadXor2>(a, jk);
    if (G >= 2)
        large_add_lanes<kQuadXor1>(a, jk);
}

__device__ __forceinline__ double large_max_shares(const int G, double v)
{
    if (G >= 8)
        v = large_max_lanes<kRowHalfMirror>(v);
    if (G >= 4)
        v = large_max_lanes<kQuadXor2>(v);
    if (G >= 2)
        v = large_max_lanes<kQuadXor1>(v);
    return v;
}

// Evaluation state of one body.
struct LargeBody {
    double2 xy, zvx, vyvz;
};

// A workgroup's dynamic LDS for E bodies: two copies of their evaluation
// state, masses, one reduction double and one int each.
struct LargeStepView {
    LargeBody *st;   // copy c of entry e at [c * E + e]
    double *m;
    double *red;
    int *flag;
};

constexpr size_t large_step_lds_bytes(int E)
{
    return (size_t)E * (2 * sizeof(LargeBody) + 2 * sizeof(double) + sizeof(int));
}

__device__ __forceinline__ LargeStepView large_step_view(const int E)
{
    extern __shared__ char fb_dyn_lds[];
    LargeStepView V;
    V.st = reinterpret_cast<LargeBody *>(fb_dyn_lds);
    V.m = reinterpret_cast<double *>(V.st + 2 * E);
    V.red = V.m + E;
    V.flag = reinterpret_cast<int *>(V.red + E);
    return V;
}

// A lane's place: its system's first LDS entry, its bodies (own: they exist;
// lead: this lane writes them), its share of the partners (share, share + G,
// ...).
template <int K>
struct LargeSeat {
    int base, n, G, log_g, share;
    int body[K], slot[K];
    bool own[K], lead[K], valid;
};

// One interaction of body i with a partner (Eq. 1 and its time derivative,
// the terms of bpl_interact).  With TS, also the pair's step-rule quantity
// (|u|^2 + 3 (r.u)^2/|r|^2) / |r|^2 into wmax (zero for the self term).
template <bool TS>
__device__ __forceinline__ void large_interact_p(const LargeBody &p, const double mj,
                                                 const double (&xi)[3], const double (&vi)[3],
                                                 double (&a)[3], double (&jk)[3], double &wmax)
{
    const double rx = p.xy.x - xi[0], ry = p.xy.y - xi[1], rz = p.zvx.x - xi[2];
    const double ux = p.zvx.y - vi[0], uy = p.vyvz.x - vi[1], uz = p.vyvz.y - vi[2];
    const double r2 = fmax(fma(rz, rz, fma(ry, ry, rx * rx)), kLargeMinR2);
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

// Publish this lane's bodies in copy `cp`, wait for the workgroup, and sum
// each owned body's interactions (its own record contributes zeros).
template <int K, bool TS, bool SPLIT>
__device__ __forceinline__ void large_eval_k(const LargeStepView &V, const int E, const int cp,
                                             const LargeSeat<K> &s, const bool live,
                                             const double (&xi)[K][3], const double (&vi)[K][3],
                                             double (&a)[K][3], double (&jk)[K][3],
                                             double (&w)[K])
{
    LargeBody *st = V.st + cp * E + s.base;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        w[k] = 0.0;
        if (s.lead[k]) {
            LargeBody &q = st[s.slot[k]];
            q.xy = make_double2(xi[k][0], xi[k][1]);
            q.zvx = make_double2(xi[k][2], vi[k][0]);
            q.vyvz = make_double2(vi[k][1], vi[k][2]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            a[k][c] = 0.0;
            jk[k][c] = 0.0;
        }
    if (!live)
        return;
    const double *mm = V.m + s.base;
    if constexpr (K == 2 && !SPLIT) {
#pragma unroll 4
        for (int p = 0; p < s.n; ++p) {
            const LargeBody q = st[p];
            const double mj = mm[p];
#pragma unroll
            for (int k = 0; k < K; ++k)
                large_interact_p<TS>(q, mj, xi[k], vi[k], a[k], jk[k], w[k]);
        }
        return;
    }
    // Every lane takes n / G partners (a scalar count), some one more.  The
    // next one is read before the interaction with this one: 1024 x 64 12.4 ->
    // 11.6 us a step, unrolling by 4 instead 12.05; a full device of two bodies
    // a lane, above, prefers the latter (4096 x 64: 38.6 against 39.2).
    const int G = SPLIT ? s.G : 1, whole = SPLIT ? s.n >> s.log_g : s.n;
    int p = SPLIT ? s.share : 0;
    LargeBody q = st[p];
    double mj = mm[p];
#pragma unroll 2
    for (int i = 1; i < whole; ++i) {
        p += G;
        const LargeBody next = st[p];
        const double m_next = mm[p];
#pragma unroll
        for (int k = 0; k < K; ++k)
            large_interact_p<TS>(q, mj, xi[k], vi[k], a[k], jk[k], w[k]);
        q = next;
        mj = m_next;
    }
#pragma unroll
    for (int k = 0; k < K; ++k)
        large_interact_p<TS>(q, mj, xi[k], vi[k], a[k], jk[k], w[k]);
    p += G;
    if (SPLIT && p < s.n) {
        q = st[p];
        mj = mm[p];
#pragma unroll
        for (int k = 0; k < K; ++k)
            large_interact_p<TS>(q, mj, xi[k], vi[k], a[k], jk[k], w[k]);
    }
    if constexpr (SPLIT)
#pragma unroll
        for (int k = 0; k < K; ++k) {
            large_add_shares(s.G, a[k], jk[k]);
            if (TS)
                w[k] = large_max_shares(s.G, w[k]);
        }
}

// Per-system reduction of one value per body, in body order (max, or sum);
// every valid lane gets its system's result.  Two barriers.
template <int K, bool MAXOP>
__device__ __forceinline__ double large_sys_reduce(const LargeStepView &V, const LargeSeat<K> &s,
                                                   const double (&val)[K])
{
    double *red = V.red + s.base;
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (s.lead[k])
            red[s.slot[k]] = val[k];
    __syncthreads();
    double r = 0.0;
    if (s.valid) {
        r = red[s.n - 1];   // the star
        for (int p = 0; p < s.n - 1; ++p)
            r = MAXOP ? fmax(r, red[p]) : r + red[p];
    }
    __syncthreads();
    return r;
}

// Stop-rule flags of each system after a committed step (the bits of
// bpl_stop_flags: 1 non-finite, 2 two planets within one mutual Hill radius,
// 4 a planet beyond r_eject), OR-ed over the system; positions go through
// copy 0 of the evaluation state, free until the next step's first
// evaluation.
template <int K>
__device__ __forceinline__ int large_stop_flags(const LargeStepView &V, const LargeSeat<K> &s,
                                                const double (&x)[K][3], const double (&v)[K][3],
                                                const StepParams &P)
{
    const int n = s.n;
    LargeBody *st = V.st + s.base;
    int fl = 0;
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (s.own[k]) {
            fl |= (finite3(x[k]) && finite3(v[k])) ? 0 : 1;
            if (s.lead[k]) {
                st[s.slot[k]].xy = make_double2(x[k][0], x[k][1]);
                st[s.slot[k]].zvx.x = x[k][2];
            }
        }
    __syncthreads();
    double rb[K];
    if (s.valid) {
        const LargeBody s0 = st[n - 1];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const double dx = x[k][0] - s0.xy.x, dy = x[k][1] - s0.xy.y, dz = x[k][2] - s0.zvx.x;
            rb[k] = sqrt(fma(dz, dz, fma(dy, dy, dx * dx)));
            if (s.lead[k])
                V.red[s.base + s.slot[k]] = rb[k];
        }
    }
    __syncthreads();
    if (s.valid) {
        const double inv24m0 = 1.0 / (24.0 * V.m[s.base + n - 1]);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (!s.own[k] || s.body[k] == 0)
                continue;
            if ((P.stop_rules & 2) && rb[k] > P.r_eject)
                fl |= 4;
            if (P.stop_rules & 1) {
                const double mi = V.m[s.base + s.slot[k]];
                for (int p = s.share; p < n - 1; p += s.G) {   // this lane's share of the planets
                    if (p == s.slot[k])
                        continue;
                    const LargeBody q = st[p];
                    const double ex = x[k][0] - q.xy.x, ey = x[k][1] - q.xy.y, ez = x[k][2] - q.zvx.x;
                    const double sep2 = fma(ez, ez, fma(ey, ey, ex * ex));
                    if (hill_close(sep2, mi, V.m[s.base + p], inv24m0, rb[k], V.red[s.base + p]))
                        fl |= 2;
                }
            }
        }
    }
    // the lanes of a body, then its system, one bit at a time
    int r = 0;
    const bool one = (fl & 1) != 0, two = (fl & 2) != 0, four = (fl & 4) != 0;
    if (__syncthreads_or(fl)) {   // rare: which systems
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (s.lead[k])
                V.flag[s.base + s.slot[k]] = 0;
        __syncthreads();
        if (s.valid && fl)
            atomicOr(&V.flag[s.base], (one ? 1 : 0) | (two ? 2 : 0) | (four ? 4 : 0));
        __syncthreads();
        if (s.valid)
            r = V.flag[s.base];
        __syncthreads();
    }
    return r;
}

// Hermite P(EC)^2 steps (Algorithm 1's loop, Algorithm 2's step) for at most
// P.quantum steps.  Every lane commits every iteration (so the pre-step state
// need not stay live through the evaluations); a system's state is written
// back as soon as it stops stepping, and its registers are ignored after
// that.
//
// Few systems are bound by the chain of a body's interactions, a full device
// by FP64 issue (33 instructions an interaction, two a pair).  Hence the two
// dimensions of the layout; loops over partners with scalar trip counts (a
// divergent count cost a mask and a branch an interaction, 1.3x); records of
// a body together, so a partner is three 16-byte reads off one address; two
// copies of them instead of a second barrier an evaluation.  256 VGPRs: two
// bodies a lane would spill at 128.  Fixed steps, us a step, against one
// lane per one to four bodies with a structure of arrays in LDS: 17 bodies
// 4.2 -> 2.0 (64 systems), 6.6 -> 6.5 (4096); 64 bodies 20.8 -> 4.3,
// 22.3 -> 11.6 (1024), 39.3 -> 38.6 (4096: 26 us of FP64 issue, both sides of
// every pair); 128 bodies 40.8 -> 11.6 (256); 512 bodies 161 -> 144.
template <int K, bool SPLIT, bool ADV>
__global__ __launch_bounds__(kLargeMaxLanes) __attribute__((amdgpu_waves_per_eu(2)))
void k_plain_large(Bucket B, StepParams P, int S, int log_g)
{
    const int G = SPLIT ? 1 << log_g : 1;
    const int n = B.n, H = (n + K - 1) / K, L = H * G, E = S * n;
    const LargeStepView V = large_step_view(E);
    const int tid = threadIdx.x;
    const int sys = tid / L, rem = tid - sys * L;
    const int h = SPLIT ? rem >> log_g : rem, pos = rem - h * G;
    const int slot0 = blockIdx.x * S + sys;
    LargeSeat<K> s;
    s.valid = sys < S && slot0 < B.count;
    s.base = s.valid ? sys * n : 0;
    s.n = n;
    s.G = G;
    s.log_g = log_g;
    s.share = pos;
    const int slot = s.valid ? slot0 : 0;
    const size_t pitch = B.pitch;
    double x[K][3], v[K][3], a0[K][3], j0[K][3];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        s.body[k] = h + k * H;
        s.own[k] = s.valid && s.body[k] < n;
        s.lead[k] = s.own[k] && pos == 0;
        const int b = s.own[k] ? s.body[k] : 0;
        s.slot[k] = large_slot(b, n);
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) {
            x[k][cc] = v[k][cc] = a0[k][cc] = j0[k][cc] = 0.0;
            if (s.own[k]) {
                x[k][cc] = B.st[((R_X + cc) * n + b) * pitch + slot];
                v[k][cc] = B.st[((R_V + cc) * n + b) * pitch + slot];
                a0[k][cc] = B.st[((R_A + cc) * n + b) * pitch + slot];
                j0[k][cc] = B.st[((R_J + cc) * n + b) * pitch + slot];
            }
        }
        if (s.lead[k])   // ordered before any read by the loop's first barrier
            V.m[s.base + s.slot[k]] = B.st[(R_M * n + b) * pitch + slot];
    }
    Clock c;
    c.status = ST_DONE;
    if (s.valid)
        c = load_clock(B, slot);
    bool pending = false;   // registers hold committed steps not yet written back
    int bad = 0;            // non-finite state written back
    auto write_back = [&]() {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (!s.lead[k])
                continue;
            const int b = s.body[k];
            bad |= (finite3(x[k]) && finite3(v[k])) ? 0 : 1;
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                B.st[((R_X + cc) * n + b) * pitch + slot] = x[k][cc];
                B.st[((R_V + cc) * n + b) * pitch + slot] = v[k][cc];
                B.st[((R_A + cc) * n + b) * pitch + slot] = a0[k][cc];
                B.st[((R_J + cc) * n + b) * pitch + slot] = j0[k][cc];
            }
        }
        pending = false;
    };
#pragma unroll 1
    for (int q = 0; q < P.quantum; ++q) {
        double hs = 0.0;
        bool last = false;
        const bool act = s.valid && plan_step(c, P, hs, last);
        if (pending && !act)
            write_back();
        if (!__syncthreads_or(act))
            break;
        const Coef cf = make_coef(hs);
        double xc[K][3], vc[K][3], bx[K][3], bv[K][3], ak[K][3], jk[K][3];
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int cc = 0; cc < 3; ++cc)
                predict_comp(cf, x[k][cc], v[k][cc], a0[k][cc], j0[k][cc], xc[k][cc], vc[k][cc],
                             bx[k][cc], bv[k][cc]);
        double w[K];
        large_eval_k<K, false, SPLIT>(V, E, 0, s, act, xc, vc, ak, jk, w);
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int cc = 0; cc < 3; ++cc)
                correct_comp(cf, bx[k][cc], bv[k][cc], ak[k][cc], jk[k][cc], xc[k][cc], vc[k][cc]);
        large_eval_k<K, ADV, SPLIT>(V, E, 1, s, act, xc, vc, ak, jk, w);
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                correct_comp(cf, bx[k][cc], bv[k][cc], ak[k][cc], jk[k][cc], x[k][cc], v[k][cc]);
                a0[k][cc] = ak[k][cc];
                j0[k][cc] = jk[k][cc];
            }
        double dtp = 0.0;
        if (ADV && P.adaptive == 1)   // the pairwise rule: max over the system's pairs
            dtp = P.eta * rsqrt_nr(large_sys_reduce<K, true>(V, s, w));
        if (ADV && P.adaptive == 2) { // Eq. 5: sum over the system's bodies
            double qq[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const double aa = fma(ak[k][2], ak[k][2], fma(ak[k][1], ak[k][1], ak[k][0] * ak[k][0]));
                const double jj = fma(jk[k][2], jk[k][2], fma(jk[k][1], jk[k][1], jk[k][0] * jk[k][0]));
                qq[k] = jj / aa;
            }
            dtp = P.eta * rsqrt_nr(large_sys_reduce<K, false>(V, s, qq));
        }
        if (act) {
            finish_step(c, P, last, hs, dtp);
            pending = true;
        }
        if (ADV) {
            const int fl = large_stop_flags<K>(V, s, x, v, P);
            if (act && fl)
                c.status = status_of_flags(fl);
        }
    }
    if (pending)
        write_back();
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (s.lead[k])
            V.flag[s.base + s.slot[k]] = bad;
    __syncthreads();
    if (s.valid && h == 0 && pos == 0) {   // the lane of the star
        int fl = 0;
        if (!ADV)                          // (with ADV the stop flags checked every step)
            for (int b = 0; b < n; ++b)
                fl |= V.flag[s.base + b];
        if (fl)
            c.status = ST_NONFINITE;
        store_clock(B, slot, c);
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// launch
// ---------------------------------------------------------------------------
namespace {

struct LargeShape {
    int K, G, T, S;
};

// What a run does besides fixed steps.
struct LargeRules {
    bool adaptive, stops;
};

// Estimated time (us) of a step while `now` workgroups of `waves` wavefronts
// share a CU: either the chain of one lane's interactions (0.17 us a partner
// of one body, 0.29 us of two; 0.2 us to add the shares of two lanes; 0.13 us
// of barrier a wavefront) or the issue of a SIMD's wavefronts (0.16 or 0.29 us
// a partner and wavefront, 0.6 us a body and wavefront for the rest of the
// step), the larger and a little more.  Workgroups of 2 or 3 wavefronts load
// the SIMDs unevenly.  The rules add to it: two bodies a lane cost a little more
// a partner (their step-rule quantities; more where lanes share partners), the
// stop rules a pass over the partners, the step rule a pass over the system.
double large_step_us(int K, int log_g, int n, int waves, int now, LargeRules r)
{
    const int parts = (n + (1 << log_g) - 1) >> log_g;
    double per_simd = (now * waves + 3) / 4;
    if (now > 1 && (waves == 2 || waves == 3))
        per_simd = 1.2 * std::max(2.0, per_simd);
    double chain = 0.7 + parts * (K == 1 ? 0.17 : 0.29) + 0.2 * K * log_g + 0.13 * waves;
    double issue = per_simd * (parts * (K == 1 ? 0.16 : 0.29) + 0.6 * K);
    if (r.adaptive || r.stops) {
        const double pair = K == 1 ? 0.0 : log_g == 0 ? 0.0053 : 0.0202;
        chain += pair * parts;
        issue += per_simd * pair * parts;
    }
    if (r.stops) {
        chain += (K == 1 ? 0.0552 : 0.0448) * parts;
        issue += per_simd * (K == 1 ? 0.0079 : 0.0302) * parts;
    }
    if (r.adaptive)
        chain += 0.0517 * n;
    const double c2 = chain * chain, c4 = c2 * c2, i2 = issue * issue, i4 = i2 * i2;
    return std::sqrt(std::sqrt(std::sqrt(c4 * c4 + i4 * i4)));   // (8th powers)
}

// Estimated time (us a step) of a run of `count` systems.  A CU takes 8
// wavefronts at a time, 2 a SIMD, so a run is so many full rounds and one of
// the workgroups left over.  With adaptive steps the systems take different
// numbers of steps, and the slowest several times the mean: a workgroup lasts
// as long as the slowest of its S systems (0.186 ln S more), and the last ones
// run with the device to themselves (3.59 steps more).
double large_run_us(const LargeShape &f, int n, int count, int num_cu, LargeRules r)
{
    int log_g = 0;
    while ((1 << log_g) < f.G)
        ++log_g;
    const int waves = f.T / 64, at_once = std::max(1, 8 / waves);
    const int per_cu = ((count + f.S - 1) / f.S + num_cu - 1) / num_cu;   // workgroups
    const int left = per_cu % at_once;
    const double t = per_cu / at_once * large_step_us(f.K, log_g, n, waves, at_once, r) +
                     (left ? large_step_us(f.K, log_g, n, waves, left, r) : 0.0);
    if (!r.adaptive)
        return t;
    return t * (1.0 + 0.186 * std::log((double)f.S)) + 3.59 * large_step_us(f.K, log_g, n, waves, 1, r);
}

LargeShape large_best(int n, int count, int num_cu, LargeRules r)
{
    LargeShape best{1, 1, 0, 0};
    double least = 0.0;
    for (int K = 1; K <= 2; ++K)
        for (int G = 1; G <= 8; G *= 2) {
            const int L = (n + K - 1) / K * G;
            for (int T = 64; T <= kLargeMaxLanes; T += 64) {
                const int S = std::min(std::min(T / L, kLargeMaxLanes / n), count);
                if (S < 1 || S * L <= T - 64)   // (a smaller T holds as many)
                    continue;
                const LargeShape f{K, G, T, S};
                const double t = large_run_us(f, n, count, num_cu, r);
                if (best.S == 0 || t < least) {
                    least = t;
                    best = f;
                }
            }
        }
    return best;
}

// The layout with the least estimated time.  For fixed steps the constants are
// a fit to 3300 timed layouts (31 body counts of 17..512, 1..6000 systems); the
// pick is 1.5% slower than the best of them on average and 14% at worst (350
// bodies, 1024 systems: 425 against 373 us).  Few systems spread out (64 bodies:
// 8 lanes a body up to 256 systems, 4.2-5.1 us a step against 11-12.5 with one;
// 4 lanes to 512, 7.9 us); a full device does not split (4096 x 64: two bodies a
// lane 40 us, one body on 4 lanes 46-56).
// Runs with rules spread out more.  The rules' constants are a fit to 372 runs
// (17..512 bodies, 4..6000 systems; adaptive with and without stop rules, fixed
// steps with them; 28 layouts each on average): the pick is 2% slower than the
// best on average and 38% at worst (40 bodies, 3000 systems), the layout for
// fixed steps 11% and 3.2 times.  80 bodies, 3000 systems, adaptive 14.9 -> 6.6
// ms, 200 bodies, 1000 systems 22.2 -> 15.7.  The layout for fixed steps stays
// where another is not clearly better, a tenth with adaptive steps alone and a
// twentieth with stop rules alone: closer ones the estimate does not tell apart
// (33 bodies, 1000 systems, adaptive, 303 and 343 us; 200 bodies, 4 systems, stop
// rules, 1.20 and 1.26 ms).  With stop rules alone one lane a body is taken wherever
// it is estimated best: 30 sizes where it was closer were 2 to 7% faster (80 bodies,
// 1000 systems, 62 steps 2.54 and 2.63 ms; 400 bodies, 8 systems, 10 steps 1.76
// and 1.86), 16 others of the same distance with more lanes 3 to 10% slower.
LargeShape large_layout(int n, int count, int num_cu, LargeRules r)
{
    const LargeShape f = large_best(n, count, num_cu, r);
    if (r.adaptive == r.stops)
        return f;
    const LargeShape g = large_best(n, count, num_cu, LargeRules{false, false});
    const double clear = r.adaptive ? 0.9 : f.G == 1 ? 1.0 : 0.95;
    return large_run_us(f, n, count, num_cu, r) > clear * large_run_us(g, n, count, num_cu, r) ? g : f;
}

template <int K, bool SPLIT>
void large_launch_as(const Bucket &B, const StepParams &P, const LargeShape &f, hipStream_t s)
{
    const dim3 grid((unsigned)((B.count + f.S - 1) / f.S));
    const size_t lds = large_step_lds_bytes(f.S * B.n);
    int log_g = 0;
    while ((1 << log_g) < f.G)
        ++log_g;
    if (P.adaptive || P.stop_rules)
        hipLaunchKernelGGL((k_plain_large<K, SPLIT, true>), grid, dim3(f.T), lds, s, B, P, f.S, log_g);
    else
        hipLaunchKernelGGL((k_plain_large<K, SPLIT, false>), grid, dim3(f.T), lds, s, B, P, f.S, log_g);
}

}  // namespace

hipError_t launch_large(const Bucket &B, const StepParams &P, int num_cu, hipStream_t s)
{
    if (B.count == 0)
        return hipSuccess;
    const LargeShape f = large_layout(B.n, B.count, num_cu, LargeRules{P.adaptive != 0, P.stop_rules != 0});
    if (f.S < 1)
        return hipErrorInvalidValue;
    if (f.K == 1 && f.G == 1)
        large_launch_as<1, false>(B, P, f, s);
    else if (f.K == 1)
        large_launch_as<1, true>(B, P, f, s);
    else if (f.G == 1)
        large_launch_as<2, false>(B, P, f, s);
    else
        large_launch_as<2, true>(B, P, f, s);
    return hipGetLastError();
}

}  // namespace fb
