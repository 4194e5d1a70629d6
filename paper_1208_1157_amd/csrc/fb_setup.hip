// fb_setup.hip -- set-up, start of a run and read-back of every bucket of an
// ensemble (or of a server request's slot ranges) at once.
//
// A launch per bucket and kernel cost a mixed ensemble dozens of launches of a
// few workgroups each, one after another: 65536 systems of 3..15 bodies took
// 205 us to lay out, 400 for the first evaluation (a system per lane: the
// larger ones spilled), 290 to read back; a server request as much for each of
// its slot ranges.  Here the buckets of a set share a launch and a lane has
// one body, so the caller's rows are read and written 24 bytes a lane side by
// side: 65536 x 3..15 in 35 us, the evaluation included, and 30 us back;
// 131072 x 3 in 20 us (20 before) and 18 (29).
#include "fb_bpl.h"

#include <algorithm>

namespace fb {
namespace {

constexpr int kBlock = 256, kWaves = kBlock / 64;

// Bucket of the set whose tiles include `tile` (set.count: none).
__device__ __forceinline__ int bucket_of(const BucketSet &set, const int tile)
{
    int k = 0;
    while (k < set.count && tile >= set.first[k + 1])
        ++k;
    return k;
}

// The caller's system in a slot; the storing lane keeps it in the tables.
__device__ __forceinline__ int origin_of(const CallerArrays &in, const Bucket &B, const int slot,
                                         const bool store)
{
    if (in.identity) {
        if (store && in.orig_off) {
            B.orig[slot] = slot;
            in.orig_off[slot] = (long long)slot * B.n;
            if (slot == B.count - 1)
                in.orig_off[slot + 1] = (long long)(slot + 1) * B.n;
        }
        return slot;
    }
    if (!in.origins)
        return B.orig[slot];
    const int o = in.origins[B.pad + slot];
    if (store)
        B.orig[slot] = o;
    return o;
}

// Layout of the caller's arrays (or, AOS false, of the rows already there)
// and the set-up evaluation of (a0, j0), Algorithm 1's "prepare"; and the
// start of a run, if run.on.  A tile of 64 / n systems a wavefront, a lane a
// body; the evaluation sums the partners in the order of bpl_eval, so its bits
// are those of every other mapping.  Bound by the copies' memory traffic.
template <bool AOS>
__global__ __launch_bounds__(kBlock) void k_create(BucketSet set, CallerArrays in, RunStart run)
{
    __shared__ BplLds lds[kWaves];
    const int lane = threadIdx.x & 63;
    const int tile = uniform_i(blockIdx.x * kWaves + (threadIdx.x >> 6));
    const int k = bucket_of(set, tile);
    if (k >= set.count)   // the whole wavefront; no workgroup barrier below
        return;
    BplLds &L = lds[threadIdx.x >> 6];
    const Bucket B = set.b[k];
    const size_t pitch = B.pitch;
    const int n = B.n, S = 64 / n;
    const int sys = lane / n, b = lane - sys * n;
    const int slot = (tile - set.first[k]) * S + sys;
    const bool own = sys < S && slot < B.count;
    if (AOS && !own && sys < S && b == 0 && in.pad && slot < B.pitch) {   // padding: inert, finished
        B.status[slot] = ST_DONE;
        B.t[slot] = 0.0;
        B.steps[slot] = 0;
    }
    double m = 0.0, x[3] = {0.0, 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0};
    if (own) {
        if (AOS) {
            const int o = origin_of(in, B, slot, b == 0);
            const long long row = (in.identity ? (long long)slot * n : in.orig_off[o]) + b;
            m = in.mass[row];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                x[c] = in.pos[3 * row + c];
                v[c] = in.vel[3 * row + c];
            }
            const double t = in.t0 ? in.t0[o] : 0.0;
            if (in.bad && !(__builtin_isfinite(m) && m >= 0.0 && finite3(x) && finite3(v) &&
                            __builtin_isfinite(t)))
                atomicOr(in.bad, 1);
            B.st[(R_M * n + b) * pitch + slot] = m;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                B.st[((R_X + c) * n + b) * pitch + slot] = x[c];
                B.st[((R_V + c) * n + b) * pitch + slot] = v[c];
            }
            if (b == 0) {
                B.t[slot] = t;
                B.dtn[slot] = 0.0;
                B.steps[slot] = 0;
                if (run.on) {
                    begin_run_clock(B, slot, ST_DONE, t, run);
                } else {
                    B.t0run[slot] = t;
                    B.t_end[slot] = t;
                    B.dt[slot] = 0.0;
                    B.krun[slot] = 0;
                    B.nfull[slot] = 0;
                    B.status[slot] = ST_DONE;
                }
            }
        } else {
            m = B.st[(R_M * n + b) * pitch + slot];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                x[c] = B.st[((R_X + c) * n + b) * pitch + slot];
                v[c] = B.st[((R_V + c) * n + b) * pitch + slot];
            }
        }
    }
    L.xy[lane] = make_double2(x[0], x[1]);
    L.zvx[lane] = make_double2(x[2], v[0]);
    L.vyvz[lane] = make_double2(v[1], v[2]);
    L.mr[lane] = make_double2(m, 0.0);
    wave_sync();
    double a[3] = {0.0, 0.0, 0.0}, jk[3] = {0.0, 0.0, 0.0}, w = 0.0;
    const int base = own ? lane - b : 0, skip = b == 0 ? n : b;
#pragma unroll 1
    for (int p = 1; p < n - 1; ++p)
        bpl_interact<false>(L, base + p + (p >= skip ? 1 : 0), x, v, a, jk, w);
    bpl_interact<false>(L, base + (b == 0 ? n - 1 : 0), x, v, a, jk, w);
    if (!own)
        return;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        B.st[((R_A + c) * n + b) * pitch + slot] = a[c];
        B.st[((R_J + c) * n + b) * pitch + slot] = jk[c];
    }
}

// Caller's arrays -> rows without the evaluation, a lane a body of any n
// (systems of more than kMaxBodies bodies: k_prepare_large evaluates).
__global__ __launch_bounds__(kBlock) void k_layout(Bucket B, CallerArrays in)
{
    const size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x, pitch = B.pitch;
    const int n = B.n, slot = (int)(i / n), b = (int)(i - (size_t)slot * n);
    if (slot >= B.pitch)
        return;
    if (slot >= B.count) {
        if (in.pad && b == 0) {
            B.status[slot] = ST_DONE;
            B.t[slot] = 0.0;
            B.steps[slot] = 0;
        }
        return;
    }
    const int o = origin_of(in, B, slot, b == 0);
    const long long row = (in.identity ? (long long)slot * n : in.orig_off[o]) + b;
    const double m = in.mass[row];
    bool ok = __builtin_isfinite(m) && m >= 0.0;
    B.st[(R_M * n + b) * pitch + slot] = m;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double x = in.pos[3 * row + c], v = in.vel[3 * row + c];
        ok = ok && __builtin_isfinite(x) && __builtin_isfinite(v);
        B.st[((R_X + c) * n + b) * pitch + slot] = x;
        B.st[((R_V + c) * n + b) * pitch + slot] = v;
    }
    if (b == 0) {
        const double t = in.t0 ? in.t0[o] : 0.0;
        ok = ok && __builtin_isfinite(t);
        B.t[slot] = t;
        B.t0run[slot] = t;
        B.t_end[slot] = t;
        B.dt[slot] = 0.0;
        B.dtn[slot] = 0.0;
        B.krun[slot] = 0;
        B.nfull[slot] = 0;
        B.steps[slot] = 0;
        B.status[slot] = ST_DONE;
    }
    if (in.bad && !ok)
        atomicOr(in.bad, 1);
}

// The clocks' start of a run that proposes no adaptive step from the state.
__global__ __launch_bounds__(kBlock) void k_begin_clock(BucketSet set, RunStart run)
{
    const int k = bucket_of(set, blockIdx.x);
    if (k >= set.count)
        return;
    const Bucket B = set.b[k];
    const int slot = (blockIdx.x - set.first[k]) * kBlock + threadIdx.x;
    if (slot < B.count)
        begin_run_clock(B, slot, B.status[slot], B.t[slot], run);
}

// ... of one bucket: without the set among the kernel's arguments (1.6 KB).  A call
// of one step, 40000 x 3 bodies, 11.9 us through the set and 10.8 so.  Workgroups of
// a wavefront would leave the SIMDs of a CU unevenly taken where the next launch
// starts: 200 steps with stop rules of 8192 x 16 bodies 1671 us after this kernel,
// 2324 after one with 64 lanes a workgroup.
__global__ __launch_bounds__(kBlock) void k_begin_clock_of(Bucket B, RunStart run)
{
    const int slot = blockIdx.x * kBlock + threadIdx.x;
    if (slot < B.count)
        begin_run_clock(B, slot, B.status[slot], B.t[slot], run);
}

// Rows -> the caller's arrays (any output may be null), a lane a body of any
// n.  Bound by memory traffic.
__global__ __launch_bounds__(kBlock) void k_read_back(BucketSet set, StateOut out)
{
    const int k = bucket_of(set, blockIdx.x);
    if (k >= set.count)
        return;
    const Bucket B = set.b[k];
    const size_t i = (size_t)(blockIdx.x - set.first[k]) * kBlock + threadIdx.x, pitch = B.pitch;
    const int n = B.n, slot = (int)(i / n), b = (int)(i - (size_t)slot * n);
    if (slot >= B.count)
        return;
    const int o = out.orig_off ? B.orig[slot] : slot;
    const long long row = 3 * ((out.orig_off ? out.orig_off[o] : (long long)slot * n) + b);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        if (out.pos)
            out.pos[row + c] = B.st[((R_X + c) * n + b) * pitch + slot];
        if (out.vel)
            out.vel[row + c] = B.st[((R_V + c) * n + b) * pitch + slot];
        if (out.acc)
            out.acc[row + c] = B.st[((R_A + c) * n + b) * pitch + slot];
        if (out.jerk)
            out.jerk[row + c] = B.st[((R_J + c) * n + b) * pitch + slot];
    }
    if (b == 0) {
        if (out.t)
            out.t[o] = B.t[slot];
        if (out.status)
            out.status[o] = B.status[slot];
        if (out.steps)
            out.steps[o] = B.steps[slot];
        if (out.dtn)
            out.dtn[o] = B.dtn[slot];
    }
}

// The same of buckets in MVS form, converted to inertial positions and
// velocities on the way (the stored form stays): x_0 = X - sum m_i Q_i / M,
// x_i = x_0 + Q_i, v_0 = Vc - sum m_i V_i / m_0, v_i = Vc + V_i.  Every lane
// sums for itself over its system's bodies in LDS, in the order of from_mvs.
__global__ __launch_bounds__(kBlock) void k_read_back_mvs(BucketSet set, StateOut out)
{
    __shared__ BplLds lds[kWaves];
    const int lane = threadIdx.x & 63;
    const int tile = uniform_i(blockIdx.x * kWaves + (threadIdx.x >> 6));
    const int k = bucket_of(set, tile);
    if (k >= set.count)
        return;
    BplLds &L = lds[threadIdx.x >> 6];
    const Bucket B = set.b[k];
    const size_t pitch = B.pitch;
    const int n = B.n, S = 64 / n;
    const int sys = lane / n, b = lane - sys * n;
    const int slot = (tile - set.first[k]) * S + sys;
    const bool own = sys < S && slot < B.count;
    double m = 0.0, x[3] = {0.0, 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0};
    if (own) {
        m = B.st[(R_M * n + b) * pitch + slot];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            x[c] = B.st[((R_X + c) * n + b) * pitch + slot];
            v[c] = B.st[((R_V + c) * n + b) * pitch + slot];
        }
    }
    L.xy[lane] = make_double2(x[0], x[1]);
    L.zvx[lane] = make_double2(x[2], v[0]);
    L.vyvz[lane] = make_double2(v[1], v[2]);
    L.mr[lane] = make_double2(m, 0.0);
    wave_sync();
    const int base = own ? lane - b : 0;
    const double m0 = L.mr[base].x;
    double M = 0.0 + m0, sq[3] = {0.0, 0.0, 0.0}, sp[3] = {0.0, 0.0, 0.0};
#pragma unroll 1
    for (int i = 1; i < n; ++i) {
        const double mi = L.mr[base + i].x;
        const double2 p0 = L.xy[base + i], p1 = L.zvx[base + i], p2 = L.vyvz[base + i];
        M += mi;
        sq[0] = fma(mi, p0.x, sq[0]);
        sq[1] = fma(mi, p0.y, sq[1]);
        sq[2] = fma(mi, p1.x, sq[2]);
        sp[0] = fma(mi, p1.y, sp[0]);
        sp[1] = fma(mi, p2.x, sp[1]);
        sp[2] = fma(mi, p2.y, sp[2]);
    }
    if (!own)
        return;
    const double2 c0 = L.xy[base], c1 = L.zvx[base], c2 = L.vyvz[base];
    const double X[3] = {c0.x, c0.y, c1.x}, V[3] = {c1.y, c2.x, c2.y};
    const int o = B.orig[slot];
    const long long row = 3 * (out.orig_off[o] + b);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double x0 = X[c] - sq[c] / M;
        if (out.pos)
            out.pos[row + c] = b == 0 ? x0 : x[c] + x0;
        if (out.vel)
            out.vel[row + c] = b == 0 ? V[c] - sp[c] / m0 : v[c] + V[c];
    }
    if (b == 0) {
        if (out.t)
            out.t[o] = B.t[slot];
        if (out.status)
            out.status[o] = B.status[slot];
        if (out.steps)
            out.steps[o] = B.steps[slot];
    }
}

// Inertial (x, v) -> MVS form in place: X, Vc in row 0, Q_i = x_i - x_0, V_i =
// v_i - Vc, and the planet-planet accelerations at Q (mvs_acc, in its order); a
// lane a body, as k_read_back_mvs.  4099 systems of 5..12 bodies in 8 us, 45
// as a launch per body count.
__global__ __launch_bounds__(kBlock) void k_enter_mvs(BucketSet set)
{
    __shared__ BplLds lds[kWaves];
    const int lane = threadIdx.x & 63;
    const int tile = uniform_i(blockIdx.x * kWaves + (threadIdx.x >> 6));
    const int k = bucket_of(set, tile);
    if (k >= set.count)
        return;
    BplLds &L = lds[threadIdx.x >> 6];
    const Bucket B = set.b[k];
    const size_t pitch = B.pitch;
    const int n = B.n, S = 64 / n;
    const int sys = lane / n, b = lane - sys * n;
    const int slot = (tile - set.first[k]) * S + sys;
    const bool own = sys < S && slot < B.count;
    double m = 0.0, x[3] = {0.0, 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0};
    if (own) {
        m = B.st[(R_M * n + b) * pitch + slot];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            x[c] = B.st[((R_X + c) * n + b) * pitch + slot];
            v[c] = B.st[((R_V + c) * n + b) * pitch + slot];
        }
    }
    L.xy[lane] = make_double2(x[0], x[1]);
    L.zvx[lane] = make_double2(x[2], v[0]);
    L.vyvz[lane] = make_double2(v[1], v[2]);
    L.mr[lane] = make_double2(m, 0.0);
    wave_sync();
    const int base = own ? lane - b : 0;
    double M = 0.0, sx[3] = {0.0, 0.0, 0.0}, sv[3] = {0.0, 0.0, 0.0};
#pragma unroll 1
    for (int i = 0; i < n; ++i) {
        const double mi = L.mr[base + i].x;
        const double2 p0 = L.xy[base + i], p1 = L.zvx[base + i], p2 = L.vyvz[base + i];
        M += mi;
        sx[0] = fma(mi, p0.x, sx[0]);
        sx[1] = fma(mi, p0.y, sx[1]);
        sx[2] = fma(mi, p1.x, sx[2]);
        sv[0] = fma(mi, p1.y, sv[0]);
        sv[1] = fma(mi, p2.x, sv[1]);
        sv[2] = fma(mi, p2.y, sv[2]);
    }
    const double2 s0 = L.xy[base];
    const double x0[3] = {s0.x, s0.y, L.zvx[base].x};
    wave_sync();
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double X = sx[c] / M, Vc = sv[c] / M;
        x[c] = b == 0 ? X : x[c] - x0[c];
        v[c] = b == 0 ? Vc : v[c] - Vc;
    }
    L.xy[lane] = make_double2(x[0], x[1]);
    L.zvx[lane] = make_double2(x[2], 0.0);
    wave_sync();
    double a[3] = {0.0, 0.0, 0.0};
    const int skip = b == 0 ? n : b;
#pragma unroll 1
    for (int p = 1; p < n - 1; ++p) {   // the other planets (the star's lane: not used)
        const int at = base + p + (p >= skip ? 1 : 0);
        const double2 p0 = L.xy[at];
        const double d0 = p0.x - x[0], d1 = p0.y - x[1], d2 = L.zvx[at].x - x[2];
        const double s = rsqrt_nr(fma(d2, d2, fma(d1, d1, d0 * d0)));
        const double mj = L.mr[at].x * (s * s * s);
        a[0] = fma(mj, d0, a[0]);
        a[1] = fma(mj, d1, a[1]);
        a[2] = fma(mj, d2, a[2]);
    }
    if (!own)
        return;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        B.st[((R_X + c) * n + b) * pitch + slot] = x[c];
        B.st[((R_V + c) * n + b) * pitch + slot] = v[c];
        B.st[((R_A + c) * n + b) * pitch + slot] = b == 0 ? 0.0 : a[c];
    }
}

__global__ __launch_bounds__(kBlock) void k_persistent_tables(BucketSet set, PersistentTables t)
{
    int base = t.first_entry;
    for (int k = 0; k < set.count; ++k) {
        const Bucket &B = set.b[k];
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            const int i = t.first_bucket + k;
            t.buckets[i] = B;
            t.order[k] = i;   // buckets are laid out in descending n: longest work first
            t.mapping[i] = t.map[k];
            t.list_base[i] = base;
            if (t.lists)
                t.counts[i] = B.count;
        }
        if (t.lists && (int)blockIdx.x >= set.first[k] && (int)blockIdx.x < set.first[k + 1]) {
            const int slot = (blockIdx.x - set.first[k]) * kBlock + threadIdx.x;
            if (slot < B.pitch)
                t.lists[base + slot] = slot;
        }
        base += B.pitch;
    }
}

// Launch over the buckets for which take(B) holds, a set at a time; units(B)
// is a bucket's number of tiles and `per` the tiles a workgroup takes.
template <class Take, class Units, class Launch>
hipError_t for_sets(const Bucket *b, int nb, Take take, Units units, int per, Launch launch)
{
    BucketSet set;
    set.clear();
    for (int i = 0; i <= nb; ++i) {
        if (i < nb && take(b[i]) && b[i].count > 0)
            set.add(b[i], units(b[i]));
        if (set.count == BucketSet::kMost || (i == nb && set.count > 0)) {
            launch(set, dim3((unsigned)((set.first[set.count] + per - 1) / per)));
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess)
                return e;
            set.clear();
        }
    }
    return hipSuccess;
}

bool is_small(const Bucket &B) { return B.n <= kMaxBodies; }
bool any_n(const Bucket &) { return true; }
int body_tiles(const Bucket &B) { return (B.count + 64 / B.n - 1) / (64 / B.n); }
int body_blocks(const Bucket &B) { return (int)(((size_t)B.count * B.n + kBlock - 1) / kBlock); }
int slot_blocks(const Bucket &B) { return (B.count + kBlock - 1) / kBlock; }

}  // namespace

hipError_t launch_create(const Bucket *b, int nb, const CallerArrays &in, const RunStart &run,
                         hipStream_t s)
{
    hipError_t e = for_sets(
        b, nb, is_small,
        [&](const Bucket &B) { return in.pad ? (B.pitch + 64 / B.n - 1) / (64 / B.n) : body_tiles(B); },
        kWaves, [&](const BucketSet &set, dim3 grid) {
            hipLaunchKernelGGL(k_create<true>, grid, dim3(kBlock), 0, s, set, in, run);
        });
    for (int i = 0; i < nb && e == hipSuccess; ++i)
        if (!is_small(b[i]) && b[i].count > 0) {
            if (run.on)
                return hipErrorInvalidValue;
            const size_t bodies = (size_t)(in.pad ? b[i].pitch : b[i].count) * b[i].n;
            hipLaunchKernelGGL(k_layout, dim3((unsigned)((bodies + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, b[i], in);
            e = hipGetLastError();
            if (e == hipSuccess)
                e = launch_prepare_large(b[i], s);
        }
    return e;
}

hipError_t launch_prepare(const Bucket *b, int nb, hipStream_t s)
{
    hipError_t e = for_sets(b, nb, is_small, body_tiles, kWaves, [&](const BucketSet &set, dim3 grid) {
        hipLaunchKernelGGL(k_create<false>, grid, dim3(kBlock), 0, s, set, CallerArrays(), RunStart());
    });
    for (int i = 0; i < nb && e == hipSuccess; ++i)
        if (!is_small(b[i]))
            e = launch_prepare_large(b[i], s);
    return e;
}

hipError_t launch_mvs_enter(const Bucket *b, int nb, hipStream_t s)
{
    hipError_t e = for_sets(b, nb, is_small, body_tiles, kWaves, [&](const BucketSet &set, dim3 grid) {
        hipLaunchKernelGGL(k_enter_mvs, grid, dim3(kBlock), 0, s, set);
    });
    for (int i = 0; i < nb && e == hipSuccess; ++i)
        if (!is_small(b[i]))
            e = launch_mvs_enter_large(b[i], s);
    return e;
}

hipError_t launch_begin_run(const Bucket *b, int nb, const RunStart &run, hipStream_t s)
{
    if (run.adaptive == 1 || run.adaptive == 2) {   // a step is proposed from the state
        for (int i = 0; i < nb; ++i) {
            const hipError_t e = launch_begin_adaptive(b[i], run, s);
            if (e != hipSuccess)
                return e;
        }
        return hipSuccess;
    }
    if (nb == 1) {
        if (b->count > 0)
            hipLaunchKernelGGL(k_begin_clock_of, dim3((unsigned)slot_blocks(*b)), dim3(kBlock), 0, s, *b, run);
        return hipGetLastError();
    }
    return for_sets(b, nb, any_n, slot_blocks, 1, [&](const BucketSet &set, dim3 grid) {
        hipLaunchKernelGGL(k_begin_clock, grid, dim3(kBlock), 0, s, set, run);
    });
}

hipError_t launch_read_back(const Bucket *b, int nb, const StateOut &out, bool mvs_form, hipStream_t s)
{
    if (!mvs_form)
        return for_sets(b, nb, any_n, body_blocks, 1, [&](const BucketSet &set, dim3 grid) {
            hipLaunchKernelGGL(k_read_back, grid, dim3(kBlock), 0, s, set, out);
        });
    hipError_t e = for_sets(b, nb, is_small, body_tiles, kWaves, [&](const BucketSet &set, dim3 grid) {
        hipLaunchKernelGGL(k_read_back_mvs, grid, dim3(kBlock), 0, s, set, out);
    });
    for (int i = 0; i < nb && e == hipSuccess; ++i)
        if (!is_small(b[i]))
            e = launch_unpack_mvs_large(b[i], out, s);
    return e;
}

hipError_t launch_persistent_tables(const Bucket *small, int nb, const PersistentTables &t,
                                    hipStream_t s)
{
    if (nb > BucketSet::kMost)
        return hipErrorInvalidValue;
    BucketSet set;
    set.clear();
    for (int i = 0; i < nb; ++i)
        set.add(small[i], t.lists ? (small[i].pitch + kBlock - 1) / kBlock : 0);
    hipLaunchKernelGGL(k_persistent_tables, dim3((unsigned)std::max(1, set.first[nb])), dim3(kBlock), 0,
                       s, set, t);
    return hipGetLastError();
}

}  // namespace fb
