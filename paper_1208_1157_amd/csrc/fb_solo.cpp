// fb_solo.cpp -- stateless fixed-step Hermite integration of one homogeneous
// batch of systems held in the caller's device arrays.
//
// A small batch (n_sys systems of n bodies, body-major rows as everywhere in
// the ABI) is one launch: its kernel loads the caller's rows, evaluates
// (Algorithm 1's "prepare"), takes the steps (Eq. 3 predictor, Eq. 4 corrector
// twice per step as in Algorithm 2) and stores the rows back.  A larger one is
// laid out as one structure-of-arrays bucket with its set-up evaluation,
// advanced by a plain launch of the same kernels an ensemble uses, and
// unpacked back in place.  Nothing is read back to the host and nothing
// outlives the call, so the call is pure stream work.  The bucket lives either
// in a caller workspace or, for callers that cannot allocate device memory, in
// a fixed per-device array of this file.
#include "fewbody.h"
#include "fb_internal.h"
#include "fb_runtime_internal.h"

#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <mutex>

using namespace fb;
using namespace fb::rt;

namespace {

// Largest batch the allocation-free entry point takes: the bucket of, e.g.,
// 170000 three-body or 38000 sixteen-body systems.
constexpr size_t kScratchBytes = (size_t)64 << 20;
constexpr int kMaxDevices = 64;

// The allocation-free entry point's bucket.  Host code never uses this name
// as an address: every device gets its own copy, whose address is looked up
// once per device (g_scratch_ptr).
static __device__ __align__(256) char scratch[kScratchBytes];

std::mutex g_scratch_mu;
char *g_scratch_ptr[kMaxDevices];

// Batches above this many systems are rejected before any size arithmetic.
constexpr int32_t kMaxSoloSystems = 1 << 26;

// Byte offsets of the batch's bucket inside a workspace; plain arithmetic (no
// heap).
struct SoloLayout {
    BucketLayout b;
    size_t total;
};

bool solo_layout(int32_t n_sys, int32_t n, SoloLayout &L)
{
    if (n_sys < 0 || n_sys > kMaxSoloSystems || n < 2 || n > kMaxBodies)
        return false;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off = align_up(off + bytes, 256);
        return o;
    };
    BucketLayout &bl = L.b;
    bl.n = n;
    bl.count = n_sys;
    bl.pitch = (int)align_up((size_t)n_sys, 64);
    const size_t P = bl.pitch;
    bl.st = take(sizeof(double) * R_COUNT * n * P);
    bl.t = take(8 * P);
    bl.t_end = take(8 * P);
    bl.dt = take(8 * P);
    bl.dtn = take(8 * P);
    bl.t0run = take(8 * P);
    bl.krun = take(8 * P);
    bl.nfull = take(8 * P);
    bl.steps = take(8 * P);
    bl.status = take(4 * P);
    bl.orig = take(4 * P);
    L.total = off;
    return true;
}

Bucket solo_view(char *base, const SoloLayout &L)
{
    const BucketLayout &bl = L.b;
    Bucket B;
    B.st = reinterpret_cast<double *>(base + bl.st);
    B.t = reinterpret_cast<double *>(base + bl.t);
    B.t_end = reinterpret_cast<double *>(base + bl.t_end);
    B.dt = reinterpret_cast<double *>(base + bl.dt);
    B.dtn = reinterpret_cast<double *>(base + bl.dtn);
    B.t0run = reinterpret_cast<double *>(base + bl.t0run);
    B.krun = reinterpret_cast<long long *>(base + bl.krun);
    B.nfull = reinterpret_cast<long long *>(base + bl.nfull);
    B.steps = reinterpret_cast<long long *>(base + bl.steps);
    B.status = reinterpret_cast<int *>(base + bl.status);
    B.orig = reinterpret_cast<int *>(base + bl.orig);
    B.n = bl.n;
    B.pitch = bl.pitch;
    B.count = bl.count;
    B.pad = 0;
    return B;
}

fb_status solo_check(int32_t n_sys, int32_t n, const double *d_mass, const double *d_pos,
                     const double *d_vel, int64_t n_steps, double dt, SoloLayout &L)
{
    if (!solo_layout(n_sys, n, L))
        return fail(FB_E_INVAL, "n_sys must be in 0..%d and n in 2..%d", kMaxSoloSystems,
                    kMaxBodies);
    if (n_sys > 0 && (!d_mass || !d_pos || !d_vel))
        return fail(FB_E_INVAL, "d_mass, d_pos and d_vel are required");
    if (n_steps < 0)
        return fail(FB_E_INVAL, "n_steps must be >= 0");
    if (n_steps > 0 && !(std::isfinite(dt) && dt != 0.0))
        return fail(FB_E_INVAL, "dt must be finite and non-zero");
    return FB_OK;
}

// Enqueue layout, set-up evaluation, n_steps fixed steps and read-back of the
// batch on stream s, with the bucket at `base`.  The steps use the plan of
// body count n and the same launch as an ensemble's plain schedule.
fb_status solo_run(char *base, const SoloLayout &L, const double *d_mass, double *d_pos,
                   double *d_vel, int32_t *d_status, int64_t n_steps, double dt, hipStream_t s,
                   bool timed)
{
    const Bucket B = solo_view(base, L);
    int dev = 0, num_cu = 0;
    FB_HIP(hipGetDevice(&dev));
    FB_HIP(hipDeviceGetAttribute(&num_cu, hipDeviceAttributeMultiprocessorCount, dev));
    const Plan p = get_plan(B.n);
    StepParams P;
    P.adaptive = 0;
    P.stop_rules = 0;
    P.eta = 0.01;
    P.r_eject = 100.0;
    P.max_steps = LLONG_MAX;
    P.quantum = INT_MAX;
    P.simds = 0;
    const int map = plain_mapping(p, B, false, false, num_cu > 0 ? num_cu : 256, INT_MAX);
    if (n_steps > 0 && solo_in_one(B.n, map)) {
        // A small batch: one launch, the bucket not used.  16 x 3 bodies, 10
        // steps: 18.6 us; 24.9 as three launches.
        const SoloIO io{d_mass, d_pos, d_vel, d_status, B.count, (long long)n_steps, dt};
        auto launch = [&]() {
            return map == MAP_BPLU ? launch_solo_quads(io, B.n, P, s)
                                   : launch_solo_split(io, B.n, map == MAP_SPLIT4 ? 4 : 2, P, s);
        };
        if (timed) {
            ProfScope ps(s);
            FB_HIP(launch());
        } else {
            FB_HIP(launch());
        }
        return FB_OK;
    }
    CallerArrays in;
    in.mass = d_mass;
    in.pos = d_pos;
    in.vel = d_vel;
    in.identity = 1;
    in.pad = 1;
    FB_HIP(launch_create(&B, 1, in, n_steps > 0 ? start_steps(n_steps, dt) : RunStart(), s));
    if (n_steps > 0) {
        if (timed) {
            ProfScope ps(s);
            FB_HIP(launch_plain(B, map, p.waves_per_group, P, s));
        } else {
            FB_HIP(launch_plain(B, map, p.waves_per_group, P, s));
        }
    }
    StateOut out;
    out.pos = d_pos;
    out.vel = d_vel;
    out.status = d_status;
    FB_HIP(launch_read_back(&B, 1, out, false, s));
    return FB_OK;
}

// This device's copy of `scratch`, looked up on the first call on the device
// (with the device current) and kept for the process.
fb_status device_scratch(char *&out)
{
    int dev = 0;
    FB_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices)
        return fail(FB_E_DEVICE, "device %d is beyond the %d devices the static scratch serves",
                    dev, kMaxDevices);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess)
            return hip_fail(e, "hipGetSymbolAddress(scratch)");
        if (!ptr || reinterpret_cast<uintptr_t>(ptr) % 256)
            return fail(FB_E_DEVICE, "static scratch at an unusable address");
        g_scratch_ptr[dev] = static_cast<char *>(ptr);
    }
    out = g_scratch_ptr[dev];
    return FB_OK;
}

}  // namespace

extern "C" {

fb_status fb_hermite_steps_device(int32_t n_sys, int32_t n, const double *d_mass, double *d_pos,
                                  double *d_vel, int32_t *d_status, int64_t n_steps, double dt,
                                  void *d_workspace, size_t ws_bytes, void *hip_stream)
{
    SoloLayout L;
    fb_status st = solo_check(n_sys, n, d_mass, d_pos, d_vel, n_steps, dt, L);
    if (st != FB_OK)
        return st;
    if (n_sys == 0)
        return FB_OK;
    if (!d_workspace || ws_bytes < L.total)
        return fail(FB_E_NOMEM, "workspace of %zu bytes needed, %zu given", L.total, ws_bytes);
    if (reinterpret_cast<uintptr_t>(d_workspace) % 256)
        return fail(FB_E_INVAL, "workspace must be 256-byte aligned");
    return solo_run(static_cast<char *>(d_workspace), L, d_mass, d_pos, d_vel, d_status, n_steps,
                    dt, (hipStream_t)hip_stream, true);
}

fb_status fb_hermite_steps_device_noalloc(int32_t n_sys, int32_t n, const double *d_mass,
                                          double *d_pos, double *d_vel, int32_t *d_status,
                                          int64_t n_steps, double dt, void *hip_stream)
{
    SoloLayout L;
    fb_status st = solo_check(n_sys, n, d_mass, d_pos, d_vel, n_steps, dt, L);
    if (st != FB_OK)
        return st;
    if (n_sys == 0)
        return FB_OK;
    if (L.total > kScratchBytes)
        return fail(FB_E_NOMEM,
                    "%d systems of %d bodies need %zu bytes; the static scratch holds %zu "
                    "(use fb_hermite_steps_device with a workspace)",
                    n_sys, n, L.total, kScratchBytes);
    char *base = nullptr;
    st = device_scratch(base);
    if (st != FB_OK)
        return st;
    return solo_run(base, L, d_mass, d_pos, d_vel, d_status, n_steps, dt,
                    (hipStream_t)hip_stream, false);
}

size_t fb_hermite_steps_workspace_bytes(int32_t n_sys, int32_t n)
{
    SoloLayout L;
    return solo_layout(n_sys, n, L) ? L.total : 0;
}

}  // extern "C"
