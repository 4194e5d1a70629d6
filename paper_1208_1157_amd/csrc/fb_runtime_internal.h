// Host-runtime internals shared by fb_runtime.cpp (ensembles, plans, timing)
// and fb_server.cpp (continuous-batching server).  Not part of the ABI.
#pragma once

#include "fewbody.h"
#include "fb_internal.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <vector>

namespace fb {
namespace rt {

// Record an error message for fb_last_error() and return `code`.
fb_status fail(fb_status code, const char *fmt, ...);
fb_status hip_fail(hipError_t e, const char *what);

#define FB_HIP(call)                                  \
    do {                                              \
        hipError_t e_ = (call);                       \
        if (e_ != hipSuccess)                         \
            return ::fb::rt::hip_fail(e_, #call);     \
    } while (0)

struct Plan {
    int mapping;          // MAP_SPL / MAP_BPL (entry 0: fused-kernel class, 0 = auto)
    int waves_per_group;  // 1..4
    int groups_per_cu;    // persistent schedule only (entry 0)
};
Plan get_plan(int n);

// Wavefronts of `count` n-body systems with a body's partners shared by
// several lanes, as a SIMD counts them: 5 and 6 bodies fill one with four
// lanes a body as fast as with two, so they are counted twice there.
inline long long split_tiles(int n, long long count, int map)
{
    const int S = tile_systems(map, n);
    return (count + S - 1) / S * (map == MAP_SPLIT4 && n <= 6 ? 2 : 1);
}

// Relative time of a step of a lone body-per-lane tile (fb_split.h's figures).
inline double lone_step(int n, int map)
{
    return map == MAP_SPLIT4 ? 0.37 + 0.05 * n : map == MAP_SPLIT2 ? 0.12 + 0.095 * n : 0.15 * n;
}

// One body count of a fused launch: `count` systems, the most `steps` of which
// any takes, and the mapping of its body-per-lane tiles.
struct FusedGroup {
    int n;
    long long count;
    double steps;
    int map;
};

// With two lanes a body a lane holds the terms of up to 8 partners, which spill
// from a fused launch's 256 VGPRs beside the state of a run with rules: 60
// fixed steps with stop rules of 2000 systems, two lanes and one (rolled, three
// waves a SIMD), 11 bodies 208 and 302 us, 12 380 and 328, 14 509 and 379, 16 554
// and 422; adaptive (Eq. 5) 13 bodies 2.75 and 3.29 ms, 14 2.54 and 2.26, 16 2.91
// and 2.47.
inline int fused_two_most(bool adaptive, bool stops)
{
    return adaptive ? 13 : stops ? 11 : kMaxBodies;
}

// Mappings of the tiles of a fused launch with `waves` wavefronts resident: as
// long as all tiles have a wavefront each and no SIMD more than one, the group
// that takes longest gets two lanes a body, then four (kMinSplit bodies and
// more), since the launch lasts as long as its slowest tile.  24 requests to a
// server (3..10 bodies): 9.4 ms; one choice for all groups 10.4.  two_most is the
// most bodies that get two lanes (fused_two_most), larger ones four at once.
inline void fused_split(std::vector<FusedGroup> &groups, int num_cu, long long waves, int two_most)
{
    const long long most = std::min(4LL * num_cu, waves);
    long long tiles = 0;
    for (FusedGroup &g : groups) {
        g.map = MAP_BPL;
        tiles += split_tiles(g.n, g.count, MAP_BPL);
    }
    while (tiles <= most) {
        FusedGroup *slow = nullptr;
        for (FusedGroup &g : groups)
            if (g.count > 0 && (!slow || g.steps * lone_step(g.n, g.map) > slow->steps * lone_step(slow->n, slow->map)))
                slow = &g;
        if (!slow || slow->n < kMinSplit || slow->map == MAP_SPLIT4)
            break;
        const int next = slow->map == MAP_BPL && slow->n <= two_most ? MAP_SPLIT2 : MAP_SPLIT4;
        tiles += split_tiles(slow->n, slow->count, next) - split_tiles(slow->n, slow->count, slow->map);
        if (tiles <= most)
            slow->map = next;
    }
}

// Whether the group that takes longest cannot get more lanes a body.
inline bool fused_split_done(const std::vector<FusedGroup> &groups)
{
    const FusedGroup *slow = nullptr;
    for (const FusedGroup &g : groups)
        if (g.count > 0 && (!slow || g.steps * lone_step(g.n, g.map) > slow->steps * lone_step(slow->n, slow->map)))
            slow = &g;
    return !slow || slow->n < kMinSplit || slow->map == MAP_SPLIT4;
}

// Most steps of a launch of `count` n-body systems that is faster rolled than in
// the form `map` (several lanes a body, or unrolled).  The rolled kernels keep three
// wavefronts a SIMD and prepare nothing, so they load and store the systems in less
// time; every step then costs more.  Per cent of the rolled time, launches of 1, 2,
// 3, 4 and 6 steps, fixed:
//   4 rolled wavefronts a SIMD, unrolled: n = 5 134 122 116 114 107, 6 128 118
//     113 106 102, 8 136 120 111 110 105, 10 144 118 107 101 98, 16 124 107 100 100 92;
//   0.45, two lanes a body, nine SIMDs of ten taken: 5 132 132 124 118 108, 8 137
//     124 113 105 95, 16 126 108 95 86 76;
//   0.9, unrolled: 5 121 112 106 100 92, 8 110 99 92 86 80, 16 114 96 87 79 71;
//   0.1, four lanes a body: 5 97 100 95 90 83, 8 100 92 84 77 69, 16 87 71 62 56 49.
inline int short_steps(int n, long long count, int map, int num_cu)
{
    const long long simds = 4LL * num_cu, tiles = split_tiles(n, count, MAP_BPL);
    if (n < 4)
        return 0;
    if (tiles > simds)
        return n <= 6 ? 6 : n <= 8 ? 4 : n <= 10 ? 3 : 2;
    if (map == MAP_BPLU)
        return n <= 10 && 4 * tiles > 3 * simds ? 2 : 2 * tiles > simds ? 1 : 0;
    const long long split = split_tiles(n, count, map);
    if (8 * split > 7 * simds)
        return n <= 6 ? 5 : n <= 10 ? 3 : 2;
    if (2 * split > simds)
        return n <= 6 ? 3 : n <= 8 ? 2 : 1;
    return n <= 6 && 8 * split > 3 * simds ? 2 : 0;
}

// Form of a body-per-lane launch of at most `steps` steps over bucket B (n <=
// kMaxBodies): the several-lanes-a-body ones (fb_split.h, measured there) while
// no SIMD gets more than one of their wavefronts, or the unrolled kernels
// (fb_unrolled.hip, where both sides are measured) for 4..16
// bodies (4..10 with adaptive steps, 4..8 with stop rules in fixed steps); for
// other body counts while their wavefronts are no more than one per SIMD: 2 and 3
// bodies (the quad layout holds 16 systems a wavefront, the rolled one 32 and 21),
// and the larger ones with rules (their registers leave one wave).  60 steps with
// stop rules of 9 bodies, unrolled and rolled, 12000 systems 385 and 390 us, 16000
// 478 and 455, 50000 1130 and 1022; of 10 16000 570 and 516, 50000 1568 and
// 1378 (with adaptive steps, a longer chain to hide, one wave is faster there).
// Launches of a few steps are rolled (short_steps).
inline int bpl_mapping(const Bucket &B, bool adaptive, bool stops, int num_cu, long long steps)
{
    if (B.n > kMaxBodies)
        return MAP_BPL;
    const int most = adaptive ? kMaxUnrolledAdv : stops ? kMaxUnrolledStops : kMaxBodies;
    const bool always = B.n >= 4 && B.n <= most;
    int form = always || unrolled_tiles(B) <= 4LL * num_cu ? MAP_BPLU : MAP_BPL;
    if (B.n >= kMinSplit)
        for (int map : {MAP_SPLIT2, MAP_SPLIT4})
            if (split_tiles(B.n, B.count, map) <= 4LL * num_cu)
                form = map;
    return steps <= short_steps(B.n, B.count, form, num_cu) ? MAP_BPL : form;
}

// Lane mapping of a plain launch over bucket B: the plan's, or (auto)
// system-per-lane when n allows it and the bucket's 64-system tiles give
// every SIMD of the device a wavefront, else body-per-lane, whose n lanes
// per system spread a small bucket over more of the device.  `steps`: the most
// steps the launch takes.
inline int plain_mapping(const Plan &p, const Bucket &B, bool adaptive, bool stops, int num_cu,
                         long long steps)
{
    const int lim = adaptive || stops ? kMaxSplAdv : kMaxSplBodies;
    if (p.mapping == MAP_BPL || B.n > lim)
        return bpl_mapping(B, adaptive, stops, num_cu, steps);
    if (p.mapping == MAP_SPL)
        return MAP_SPL;
    return (B.count + 63) / 64 >= 4LL * num_cu ? MAP_SPL : bpl_mapping(B, adaptive, stops, num_cu, steps);
}

// Fused persistent kernel class for a launch over buckets of these body
// counts: the plan's choice, or (auto) for fixed steps the system-per-lane
// class when every bucket can run system-per-lane in it and its tiles (64
// systems each) give every SIMD of the device a wavefront; that class runs
// one wavefront per SIMD, so with fewer tiles the body-per-lane class, which
// spreads a system over n lanes, keeps more of the device busy.  With
// adaptive steps or stop rules (auto) always the body-per-lane class: a
// system-per-lane tile runs its 64 systems in lockstep, each to its own step
// count, and measured 1.7x slower than body-per-lane tiles (about 10
// systems each) on 65536 uneven-lifetime systems at full population.  Fixed
// steps with stop rules of kMinRolled bodies and more take the rolled form of
// that class (2) where their tiles give a SIMD more than two wavefronts and those
// of 10 bodies and more are half of them or more (k_persistent_rolled).
template <class BucketRange>
int persistent_class(const Plan &p0, const BucketRange &buckets, bool adaptive, bool stops, int num_cu)
{
    if (p0.mapping == MAP_SPL)
        return 1;
    if (stops && !adaptive) {
        long long tiles = 0, larger = 0;
        bool rolled = true;
        for (const Bucket &B : buckets) {
            rolled = rolled && B.n >= kMinRolled;
            tiles += B.count / (64 / B.n);
            larger += B.n > kMinRolled ? B.count / (64 / B.n) : 0;
        }
        return rolled && tiles > 8LL * num_cu && 2 * larger >= tiles ? 2 : 0;
    }
    if (p0.mapping == MAP_BPL || adaptive)
        return 0;
    const int lim = persistent_spl_limit(1, 0);
    long long tiles = 0;
    for (const Bucket &B : buckets) {
        if (B.n > lim)
            return 0;
        tiles += (B.count + 63) / 64;
    }
    return tiles >= 4LL * num_cu ? 1 : 0;
}

// Brackets the integration launches enqueued in its scope with HIP events on
// `s` when the kernel timer is enabled.
struct ProfScope {
    hipEvent_t a = nullptr, b = nullptr;
    hipStream_t s;
    explicit ProfScope(hipStream_t st);
    ~ProfScope();
};

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Byte offsets of one body-count bucket inside an ensemble workspace.
struct BucketLayout {
    int n, count, pitch;
    size_t st, t, t_end, dt, dtn, t0run, krun, nfull, steps, status, orig;
};

// Device workspace of one ensemble: buckets in descending body count, then
// the tables, staging and scheduling arrays.
struct Layout {
    std::vector<BucketLayout> b;
    int64_t n_bodies = 0;
    int max_tiles = 0;
    int list_total = 0;
    size_t buckets, orig_off, staging, diag, ints, tiles, lists0, lists1, list_base, counts0,
        counts1, order, mapping, total;
};

bool make_layout(int32_t n_sys, const int32_t *n_body, Layout &L);
std::vector<Bucket> bucket_views(char *base, const Layout &L);

// ---- transfers (fb_transfer.cpp) ------------------------------------------
// Pinned host memory of the current device: kHostPage bytes, or kHostBlock for
// more.  Whoever takes a block gives it back once nothing on the device uses
// it; a few of each size are kept for the next taker.
constexpr size_t kHostPage = 4096, kHostBlock = 1 << 20;
constexpr int kReadWorkers = 4;
struct HostBlock {
    char *p = nullptr;
    size_t bytes = 0;
    hipStream_t stream = nullptr;   // for transfers of its own, made by the first one
    int device = -1;
};
fb_status take_block(size_t bytes, HostBlock &out);
void give_block(HostBlock &b);
// Device ranges of one allocation on `device` -> host arrays (at most
// kMostParts; parts with a null `to` are left out), after the work on stream s;
// returns when they are there.  Throws nothing.
struct HostPart {
    void *to;
    const void *from;
    size_t bytes;
};
constexpr int kMostParts = 8;
fb_status read_to_host(const HostPart *parts, int n, hipStream_t s, int device);

}  // namespace rt
}  // namespace fb
