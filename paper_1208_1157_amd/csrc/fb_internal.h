// Internal types shared by the HIP kernels (fb_kernels.hip) and the host
// runtime (fb_runtime.cpp).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fb {

// Rows of a bucket's structure-of-arrays state; row r, body b, slot s lives
// at st[(r * n + b) * pitch + s] (slot fastest: lanes read consecutive
// doubles).  a0/j0 are the carried acceleration and jerk of the step's last
// evaluation.
enum Row { R_M = 0, R_X = 1, R_V = 4, R_A = 7, R_J = 10, R_COUNT = 13 };

enum SysStatus {
    ST_ACTIVE = 0, ST_DONE = 1, ST_ENCOUNTER = 2, ST_EJECTED = 3,
    ST_NONFINITE = 4, ST_STALLED = 5, ST_MAXSTEPS = 6, ST_UNBOUND = 7
};

// MAP_BPLU is body per lane with unrolled partner loops (fb_unrolled.hip);
// MAP_SPLIT2 and MAP_SPLIT4 give a body 2 or 4 lanes (fb_split.h); plans ask
// for any of these as MAP_BPL.
enum Mapping { MAP_SPL = 1, MAP_BPL = 2, MAP_BPLU = 3, MAP_SPLIT2 = 4, MAP_SPLIT4 = 5 };

constexpr int kMaxBodies = 16;         // kernels specialised per n exist for n <= 16
constexpr int kMaxLargeBodies = 512;   // larger systems run the runtime-n large-n kernels
constexpr int kMaxSplBodies = 10;      // plain system-per-lane instances exist for n <= 10
constexpr int kMaxSplAdv = 8;          // ... with adaptive steps / stop rules for n <= 8
constexpr int kMaxSplPersistent = 0;   // the body-per-lane fused class runs no system-per-lane tiles
constexpr int kMaxUnrolledAdv = 10;    // body per lane: 4 and more bodies always run unrolled, with
                                       // adaptive steps / stop rules 4..10
constexpr int kMaxUnrolledStops = 8;   // ... with stop rules in fixed steps 4..8
constexpr int kMinRolled = 9;          // fused class 2 (fixed steps with stop rules) runs 9..16 bodies
constexpr int kMaxRkckSpl = 6;         // fixed Cash-Karp steps system per lane exist for n <= 6
constexpr int kMaxMvsBodies = 8;       // MVS kernels (system per lane) exist for n <= 8

// Device view of one homogeneous body-count bucket.  Per-slot arrays have
// `pitch` entries; slots [0, count) hold systems.
struct Bucket {
    double *st;          // [R_COUNT][n][pitch]
    double *t;           // current time
    double *t_end;       // destination time of the current run
    double *dt;          // fixed step of the current run
    double *dtn;         // carried adaptive step (<= 0: not yet proposed)
    double *t0run;       // time at the start of the current run
    long long *krun;     // whole steps taken in the current run
    long long *nfull;    // whole steps the current run takes before t_end
    long long *steps;    // steps since creation
    int *status;         // SysStatus
    int *orig;           // caller's index of the system in each slot
    int n, pitch, count, pad;
};

// Several buckets that share one launch: bucket k's tiles are first[k] ..
// first[k + 1] - 1, body-per-lane tiles of floor(64 / n) systems each or
// what the kernel takes as a unit.  Passed to kernels by value.
struct BucketSet {
    static constexpr int kMost = kMaxBodies - 1;   // every n up to kMaxBodies
    Bucket b[kMost];
    int first[kMost + 1];
    int count;

    void clear() { count = first[0] = 0; }
    void add(const Bucket &B, int tiles)
    {
        b[count] = B;
        first[count + 1] = first[count] + tiles;
        ++count;
    }
    void add(const Bucket &B) { add(B, (B.count + 64 / B.n - 1) / (64 / B.n)); }
};

// The caller's arrays, system by system, and where its systems' bodies start
// (null: system o is slot o of the only bucket, its bodies from o n on).  The
// system of a slot is B.orig's, or `origins`[B.pad + slot], or (identity) the
// slot itself; the latter two are stored in B.orig, and identity also fills
// orig_off if it is not null.
struct CallerArrays {
    const double *mass = nullptr, *pos = nullptr, *vel = nullptr;
    const double *t0 = nullptr;              // null: all zero
    long long *orig_off = nullptr;
    const int *origins = nullptr;
    int identity = 0;
    int *bad = nullptr;                      // set to 1 by an invalid input, if not null
    int pad = 0;   // also initialise slots count..pitch-1 as inert padding (a
                   // whole bucket); 0 for a view of a bucket shared with others
};

// Read-back targets in the caller's order, each optional; orig_off as above.
struct StateOut {
    const long long *orig_off = nullptr;
    double *pos = nullptr, *vel = nullptr, *acc = nullptr, *jerk = nullptr, *t = nullptr;
    int *status = nullptr;
    long long *steps = nullptr;
    double *dtn = nullptr;
};

// How a run starts: exactly n_steps steps of dt (fixed_steps), or to t_end in
// steps of dt (adaptive 0), adaptive steps (1 pairwise rule, 2 Eq. 5; eta) or
// Cash-Karp steps from a first trial step dt (3).
struct RunStart {
    int on = 0;
    int fixed_steps = 0;
    int adaptive = 0;
    long long n_steps = 0;
    double t_end = 0.0, dt = 0.0, eta = 0.0;
};
inline RunStart start_steps(long long n_steps, double dt)
{
    RunStart r;
    r.on = r.fixed_steps = 1;
    r.n_steps = n_steps;
    r.dt = dt;
    return r;
}
inline RunStart start_to(double t_end, double dt, int adaptive, double eta)
{
    RunStart r;
    r.on = 1;
    r.t_end = t_end;
    r.dt = dt;
    r.adaptive = adaptive;
    r.eta = eta;
    return r;
}

// One unit of persistent-schedule work: `count` systems of bucket `bucket`
// starting at `first` (a slot, or an index into an active list).
struct Tile {
    int bucket, first, count, kind;   // kind = mapping * 32 + n
};

struct StepParams {
    int adaptive;        // 0 fixed step, 1 adaptive step rule
    int stop_rules;      // bit 0 close encounter, bit 1 ejection
    double eta;
    double r_eject;
    long long max_steps; // per-system cap (LLONG_MAX: none)
    int quantum;         // at most this many steps per system per launch
    int simds;           // fused launch in one-wavefront workgroups: the device's
                         // SIMDs, for the placing of a single round (else 0)
};

// Compaction bookkeeping for the persistent schedule (device memory).
struct ActiveLists {
    int *cur;            // [sum pitch] active slots of each bucket, by bucket base
    int *next;           // survivors written by the running quantum
    int *base;           // [n_buckets] offset of each bucket's list
    int *cur_count;      // [n_buckets]
    int *next_count;     // [n_buckets]
};

// Systems of a wavefront that gives each body G lanes.
constexpr int split_systems(int n, int G) { return 64 / (n * G); }
constexpr int kMinSplit = 5;   // fewer bodies: quads, or too few partners to share
// Systems of a tile.
constexpr int tile_systems(int mapping, int n)
{
    return mapping == MAP_SPL ? 64
                              : split_systems(n, mapping == MAP_SPLIT4 ? 4 : mapping == MAP_SPLIT2 ? 2 : 1);
}

// ---- set-up, start of a run, read-back (fb_setup.hip) ------------------
// Each takes any buckets and as few launches as their kinds need.
// Layout of the caller's arrays and the set-up evaluation, and (systems of at
// most kMaxBodies bodies) the start of a run, if run.on, without adaptive steps.
hipError_t launch_create(const Bucket *b, int nb, const CallerArrays &in, const RunStart &run,
                         hipStream_t s);
hipError_t launch_prepare(const Bucket *b, int nb, hipStream_t s);
// Tables of a fused launch over the small buckets: bucket views from entry
// first_bucket on with their order, mapping (map[k] of the k-th) and list
// offsets (from first_entry on), and, if lists is not
// null, the counts and the identity lists.
struct PersistentTables {
    Bucket *buckets;
    int *order, *mapping, *list_base, *counts, *lists;
    int first_bucket, first_entry;
    unsigned char map[BucketSet::kMost];
};
hipError_t launch_persistent_tables(const Bucket *small, int nb, const PersistentTables &t,
                                    hipStream_t s);
hipError_t launch_mvs_enter(const Bucket *b, int nb, hipStream_t s);
hipError_t launch_begin_run(const Bucket *b, int nb, const RunStart &run, hipStream_t s);
// mvs_form: converted to inertial form on the way; acc, jerk and dtn null.
hipError_t launch_read_back(const Bucket *b, int nb, const StateOut &out, bool mvs_form,
                            hipStream_t s);

// ---- launchers (fb_kernels.hip; steps of MVS and Cash-Karp in their own) --
hipError_t launch_prepare_large(const Bucket &B, hipStream_t s);
hipError_t launch_unpack_mvs_large(const Bucket &B, const StateOut &out, hipStream_t s);
// A run with adaptive steps of either rule, its first one proposed.
hipError_t launch_begin_adaptive(const Bucket &B, const RunStart &run, hipStream_t s);
hipError_t launch_plain(const Bucket &B, int mapping, int waves_per_group,
                        const StepParams &P, hipStream_t s);
// Wavefronts launch_unrolled starts for bucket B, and the launch (launch_plain with
// MAP_BPLU comes here).
int unrolled_tiles(const Bucket &B);
hipError_t launch_unrolled(const Bucket &B, const StepParams &P, hipStream_t s);
// A batch of n_sys equal systems in the caller's arrays, system after system,
// advanced in place by n_steps fixed steps of dt; status may be null.
struct SoloIO {
    const double *mass;
    double *pos, *vel;
    int *status;
    int n_sys;
    long long n_steps;
    double dt;
};
// Set-up, steps and results of such a batch in one launch, with the kernels of
// `mapping`: MAP_SPLIT2 and MAP_SPLIT4, and MAP_BPLU up to 4 bodies.
inline bool solo_in_one(int n, int mapping)
{
    return mapping == MAP_SPLIT2 || mapping == MAP_SPLIT4 || (mapping == MAP_BPLU && n <= 4);
}
hipError_t launch_solo_split(const SoloIO &io, int n, int G, const StepParams &P, hipStream_t s);
hipError_t launch_solo_quads(const SoloIO &io, int n, const StepParams &P, hipStream_t s);
// Steps with G (2 or 4) lanes a body, kMinSplit bodies and more
// (launch_plain with MAP_SPLIT2 and MAP_SPLIT4 comes here).
hipError_t launch_split(const Bucket &B, int G, const StepParams &P, hipStream_t s);
// cls: 0 = body-per-lane class fused kernel (256 VGPRs; system-per-lane tiles
// for n <= kMaxSplPersistent), 1 = system-per-lane class (full register file;
// system-per-lane tiles for n <= kMaxSplBodies, or kMaxSplAdv with adaptive
// steps / stop rules), 2 = rolled body-per-lane tiles of kMinRolled bodies and
// more with rules (168 VGPRs).
hipError_t launch_persistent(const Bucket *d_buckets, const Tile *d_tiles,
                             const int *d_ntiles, int *d_head, const int *d_lists,
                             const StepParams &P, int adv, int cls, int grid,
                             int waves_per_group, ActiveLists *compact,
                             hipStream_t s);
hipError_t launch_build_tiles(const Bucket *d_buckets, int n_buckets,
                              const int *d_order, const int *d_mapping,
                              ActiveLists L, Tile *d_tiles, int *d_ntiles,
                              int *d_head, hipStream_t s);
hipError_t launch_reset_counter(int *p, int n, hipStream_t s);
// Energy and angular momentum of every system of the buckets.
hipError_t launch_diag(const Bucket *b, int nb, double *energy, double *angmom, bool mvs_form,
                       hipStream_t s);
// Monitor record k of every system of B (kind 0 state, 1 star RV along the
// unit vector los, 2 energy and angular momentum) into a log buffer whose
// layout fb_log_bytes describes.
hipError_t launch_log(const Bucket &B, const long long *orig_off, int kind, const double *los,
                      int k, int max_records, double *out, hipStream_t s);
// Runge-Kutta Cash-Karp: fixed steps (eps == 0), or adaptive steps with error
// tolerance eps (P.adaptive nonzero); system per lane for fixed steps (n <=
// kMaxRkckSpl), one body per lane of a wavefront (every bucket of a set, n <=
// kMaxBodies, in one launch; same results), or of a workgroup (larger n).
hipError_t launch_rkck_spl(const Bucket &B, const StepParams &P, hipStream_t s);
hipError_t launch_rkck_bpl(const BucketSet &set, const StepParams &P, double eps, hipStream_t s);
hipError_t launch_rkck_large(const Bucket &B, const StepParams &P, double eps, hipStream_t s);
// Mixed-variable symplectic integrator (n <= kMaxMvsBodies, system per
// lane): conversion of a bucket to and from MVS form, fixed-step quanta.
hipError_t launch_mvs_enter_large(const Bucket &B, hipStream_t s);
hipError_t launch_mvs_leave(const Bucket &B, hipStream_t s);
// Three mappings that give identical results: system per lane (n <=
// kMaxMvsBodies), one body per lane of a wavefront (every bucket of a set, n
// <= kMaxBodies, in one launch) and one body per lane of a workgroup (any n).
hipError_t launch_plain_mvs(const Bucket &B, int waves_per_group, const StepParams &P,
                            hipStream_t s);
hipError_t launch_mvs_bpl(const BucketSet &set, const StepParams &P, hipStream_t s);
hipError_t launch_plain_mvs_large(const Bucket &B, const StepParams &P, hipStream_t s);
hipError_t launch_count_active(const Bucket &B, int *count, hipStream_t s);
// Workgroup shape of the large-n kernels with one body per lane (n >
// kMaxBodies; the Hermite steps choose theirs in fb_large.hip): T lanes, a
// multiple of 64 up to 512, holding S = floor(T / n) systems; the T that
// leaves the fewest lanes idle.  S = 0 if the system does not fit.
void large_shape(int n, int &T, int &S);
// Hermite steps of a bucket of more than kMaxBodies bodies (fb_large.hip).
hipError_t launch_large(const Bucket &B, const StepParams &P, int num_cu, hipStream_t s);
// FP64 FMA issue-ceiling probe: blocks x 256 lanes, iters x kFmaChains FMAs
// per lane (kFmaChains = 16); out holds blocks x 256 doubles.
hipError_t launch_fma_probe(double *out, int blocks, int iters, hipStream_t s);
// The pair evaluation's reciprocal square root, elementwise (accuracy check).
hipError_t launch_rsqrt(const double *in, double *out, long long n, hipStream_t s);
// Checkpoint restore of the carried (a0, j0), adaptive step, step count and
// status of every system of B from caller-order arrays.
hipError_t launch_restore(const Bucket &B, const long long *orig_off, const double *acc,
                          const double *jerk, const double *dtn, const long long *steps,
                          const int *status, hipStream_t s);
size_t persistent_lds_bytes(int cls, int waves_per_group);
int persistent_max_groups_per_cu(int adv, int cls, int waves_per_group);
// Largest n a persistent tile runs system-per-lane for, by kernel class.
inline int persistent_spl_limit(int cls, int adv)
{
    return cls == 1 ? (adv ? kMaxSplAdv : kMaxSplBodies) : kMaxSplPersistent;
}

}  // namespace fb
