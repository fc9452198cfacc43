// Host-side internals of the DSES library: device context, workspace, argument
// resolution and the registration driver shared by the plain, resident, batched
// and serving entry points.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <deque>
#include <cstdint>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include <rocprofiler-sdk-roctx/roctx.h>

#include "dses.h"
#include "internal.h"

namespace dses {

void set_error(const std::string &msg);

#define DSES_HIP(expr)                                                                      \
    do {                                                                                    \
        hipError_t _e = (expr);                                                             \
        if (_e != hipSuccess) {                                                             \
            ::dses::set_error(std::string(#expr) + ": " + hipGetErrorString(_e));           \
            return DSES_E_DEVICE;                                                           \
        }                                                                                   \
    } while (0)

// Every device and pinned-host allocation of the library goes through these,
// so that dses_debug_fail_allocs() can make chosen ones fail (tests of the
// error paths).  On failure *p is null.
hipError_t dev_alloc_raw(void **p, size_t bytes);
hipError_t host_alloc_raw(void **p, size_t bytes, unsigned int flags);
template <class T>
inline hipError_t dev_alloc(T **p, size_t bytes)
{
    void *v = nullptr;
    const hipError_t e = dev_alloc_raw(&v, bytes);
    *p = static_cast<T *>(v);
    return e;
}
template <class T>
inline hipError_t host_alloc(T **p, size_t bytes, unsigned int flags)
{
    void *v = nullptr;
    const hipError_t e = host_alloc_raw(&v, bytes, flags);
    *p = static_cast<T *>(v);
    return e;
}

// A roctx range on the calling thread (rocprofv3 --marker-trace records it)
// around a host-side phase of an entry point; end() closes it early.
struct TraceRange {
    bool open = true;
    explicit TraceRange(const char *name) { roctxRangePushA(name); }
    void end()
    {
        if (open) roctxRangePop();
        open = false;
    }
    ~TraceRange() { end(); }
    TraceRange(const TraceRange &) = delete;
    TraceRange &operator=(const TraceRange &) = delete;
};

// A device allocation that grows on demand (never shrinks while in use).
struct DevBuf {
    void *ptr = nullptr;
    size_t bytes = 0;
    dses_status ensure(size_t want);
    void release();
    ~DevBuf() { release(); }
};

// Pinned host buffer (hipHostMalloc), grown on demand.
struct PinnedBuf {
    void *ptr = nullptr;
    size_t bytes = 0;
    dses_status ensure(size_t want);
    void release();
    ~PinnedBuf() { release(); }
};

struct Context {
    int device = -1;
    int n_cu = 0;
    int lds_max = 0;
    std::string arch;
    hipStream_t stream = nullptr;
    std::mutex mu;                       // serialises the plain entry points
    // workspace of the plain path
    DevBuf in_src, in_tgt, in_rot, yq, yt, rec, scratch;
    DevBuf modes;                        // sweeps of few rotations: the mode of each part
    DevBuf upload;                       // status words, order by x, cell grid
    DevBuf topk_a, topk_b, topk_out;     // top-k passes and output staging
    DevBuf prune;                        // q-pruning: M* and the work cursor
    DevResult *host_res = nullptr;       // pinned
    PinnedBuf host_stage;                // the reference as read back, then the upload
    // timing
    bool timing_enabled = false;
    std::mutex stats_mu;
    dses_kstats stats{};
};

// Returns the initialised context or nullptr (error set).
Context *ctx();

// Resolved numeric parameters of one registration.
struct Params {
    float eps, delta, tau, r;
    int32_t klo[3], size[3];
    int metric;
    int scorer;
    float lp = 0.5f;         // exponent of DSES_TRUNC_LP
    int32_t df_lookup = DSES_DF_NEAREST;   // how the DF scorer reads the field
};

// Applies the plain-path options that resolve_params does not see (the Lp
// exponent; q has no meaning with DSES_VOTES; lane_group is 0, 16, 32 or 64;
// the distance-field lookup).
// Host-side check, no device use.
dses_status apply_metric_options(const dses_options &o, Params *p);

dses_status resolve_params(float eps, int metric, float delta_t, float tau, const float *t_min,
                           const float *t_max, int scorer, Params *p);
// Largest |coordinate| accepted for a registration with these parameters.
// Largest accepted |coordinate|: reference points must keep the fixed-point
// lattice values in range (ref_coord_limit); a source point of any magnitude up
// to kSrcCoordLimit is accepted (its lattice value saturates where it can no
// longer vote).
float ref_coord_limit(const Params &p);
constexpr float kSrcCoordLimit = 1.0e4f;

// Counter width of the vote: 32 bits when some bin could reach 2^16 votes (the
// proven bound), and also when every 32-bit slab would still carry at least
// 2^20 pairs, where the two VALU of the 16-bit increment cost more than the
// doubled per-slab work (4,096 x 16,384 points, box 101^3, 2.0M pairs per 32-bit
// slab: 3.4% faster; 717 x 1,024 points, box 69^3, 82K pairs: 25% slower).
int counter_bits_for(int64_t bound, int32_t n, int32_t m, const Params &p);
dses_status plan_geom(const Context *c, const Params &p, int32_t n, int32_t m, int counter_bits,
                      Geom *g);
// How a call votes.  gref: reference points per lane group of the windowed vote (32 or
// 64; 16 asked for is 32, or 16 in the general path), 0 where only the general path applies (sources not
// sorted, or x planes wider than 16-bit strides).  group: the general path's.  parts: a
// group's windows are split into (0: vote_parts_auto of the general path).  general: the
// general path's estimated time as a multiple of the windowed vote's.
struct VoteLayout {
    int gref, group, parts;
    double general;
};
// population: ref_block_population; asked: the caller's lane_group.  batched: the
// batched kernels hold groups of 32 or 64 points under 16-bit counters and of 64 under
// 32-bit ones.  The caller compares `general`: the plain path with the share that
// choose_parts leaves, the others with kBatchGeneral, because the general path takes a
// launch or a slice of its own there.
VoteLayout choose_layout(const Geom &g, bool sorted, float x_extent, int64_t population, int asked,
                         bool batched);
// Parts of a lane group's windows in the windowed vote, a power of two; asked: the
// caller's vote_parts if not 0.
int window_parts(const Geom &g, int gref, float x_extent, int asked);
constexpr double kBatchGeneral = 0.85;
// Reference points per lane group of the general path's vote with sorted sources: 16,
// 32 or 64 (`asked` if not 0); vote_parts as in SweepArgs.
int choose_group(const Geom &g, float x_extent, int asked, int vote_parts);
// Items a rotation's slabs are split into by the plain path (1: none); *share: the
// estimated time as a share of that of whole rotations.
int choose_parts(const Geom &g, int32_t k, float x_extent, int n_cu, double *share);
// Staging of a reference of g.m points for a vote of geometry g with lane groups of
// gref points (0: the general path), in bank order if `arrange`.
StageDesc stage_desc(const Geom &g, int gref, bool arrange, const float *tgt, const int32_t *perm,
                     int32_t *yq, float *yt);
// Whether k rotations, each split into `parts` items over n_cu workgroups, gain from bank
// order (k_arrange takes 20 us for groups of 32 points, 40 us for 64).  It shortens the
// LDS accesses of the votes that land in the box, about n m k times the product of
// size / (2 extent) over the axes for clouds of the reference's extent.  A round of items
// takes as long when it leaves workgroups idle, so k counts as whole rounds; a batch's
// problems share their rounds (n_cu 1).  Under 32-bit counters one workgroup holds a CU and
// waits for these accesses: from 0.4 10^9 votes every measured call gained (1,500 x 3,000
// points and 300 rotations, 0.52: 720 to 621; 2,600 x 8,200 and 60, 0.41: 635 to 607;
// 5,520 x 3,103 and 300, 2.0: 2,492 to 1,951) and up to 0.33 some lost (2,600 x 4,097 and
// 60, 0.20: 375 to 404 us).  Under 16-bit ones two share a CU and hide more of them: groups of
// 64 points still lost 3% at 1.1 (3,000 x 600 and 2,000), 1,203 x 3,001 points and 4,608
// rotations (6.0) gained 0.23 ms of 4.75, and groups of 32 (717 x 1,024) issue too many
// other instructions to gain.
inline bool worth_arranging(const Geom &g, int gref, float x_extent, int64_t k, int parts, int n_cu)
{
    if (gref == 0 || (gref == 32 && g.counter_bits == 16)) return false;
    const int64_t rounds = (k * parts + n_cu - 1) / n_cu;
    double votes = (double)g.n * g.m * (double)(rounds * n_cu) / parts;
    for (int a = 0; a < 3; ++a)
        votes *= std::min(1.0, g.size[a] / (2.0 * (double)x_extent));
    return votes >= (g.counter_bits == 32 ? 0.4e9 : 2.5e9);
}
// Upper bound on any bin's vote count (decides 16- vs 32-bit LDS counters):
// n x the largest reference population of a 2 x 2 x 2 block of cells of pitch
// slightly above delta (for a fixed source point, the pairs sharing a bin have
// their references in one delta-cube).
int64_t ref_block_population(const float *tgt_aos, int32_t m, const Params &p);
int64_t counter_bound(const float *tgt_aos, int32_t m, int32_t n, const Params &p);

// Fixed-point lattice scales (1/delta) 2^16 and (1/delta) 2^15, in double.
void lattice_scales(float delta, double *S16, double *S15);

// Reference order sorted by x; the staged fixed-point x coordinates (2^-16 bins,
// lattice offset folded in, the staging arithmetic) of the first and last point
// of that order (false if the sorted sweep cannot be used); the source bucket
// origin, shift and count of a box of size_x x-planes.
void sort_by_x(const float *tgt_aos, int32_t m, std::vector<int32_t> *perm);
bool ref_x_range(const float *tgt_aos, const std::vector<int32_t> &perm, float delta,
                 int32_t klo_x, int32_t *ylo, int32_t *yhi);
void source_buckets(int32_t ylo, int32_t yhi, int32_t size_x, int32_t *sb_lo, int32_t *sb_shift,
                    int32_t *sb_n);
// x extent in bins of the staged reference (lane-group choice).
inline float ref_x_extent(int32_t ylo, int32_t yhi)
{
    return (float)((double)(yhi - ylo) / 65536.0) + 1.0f;
}

// Exact cell grid for the GRID scorer, built on the host from reference points.
struct HostGrid {
    std::vector<float> pts;      // x y z and a pad per point (16 B), cell order
    std::vector<int32_t> start;  // ncell + 1
    float lo[3];
    float inv;
    int32_t dim[3];
};
dses_status build_grid(const float *tgt_aos, int32_t m, float r, HostGrid *out);

// Resident reference cloud.
struct TargetRes {
    int32_t m = 0;
    float *aos = nullptr;            // m x 3 device copy
    float *yt = nullptr;             // SoA device copy
    std::vector<float> host_aos;     // host copy (grid builds)
    float max_abs = 0.0f;            // largest |coordinate| (lattice range check)
    // distance field
    float *df = nullptr;
    int32_t df_res = 0;
    float df_r = 0.0f;
    float df_lo[3] = {0, 0, 0}, df_h[3] = {0, 0, 0}, df_inv[3] = {0, 0, 0};
    // Caches, guarded by grid_mu.  Entries are never freed before the target is
    // destroyed: kernels of the serving loop may still read an older entry.
    std::mutex grid_mu;
    std::vector<int32_t> perm_x;             // reference order sorted by x
    int32_t *d_perm = nullptr;
    struct Stage {                           // staged copy for one (delta, box)
        float delta;
        int32_t klo[3];
        int32_t zbits, gref;                 // the layout it is staged for
        int32_t px, py;                      // the strides its bank order is made for
        int32_t *yq;                         // fixed-point copy (stage_words(m) int32)
        float *yt;
    };
    std::deque<Stage> stages;                // deque: references survive push_back
    struct Population {                      // ref_block_population for (delta, box)
        float delta;
        int32_t klo[3], size[3];
        int64_t pop;
    };
    std::vector<Population> pops;
    struct Grid {                            // cell grid for one radius
        float r;
        float *pts;
        int32_t *start;
        HostGrid meta;
    };
    std::deque<Grid> grids;
};

struct RotRes {
    int64_t k = 0;
    float *rot = nullptr;            // k x 9 device copy
};

// Everything the driver needs about one registration, with device pointers.
struct Job {
    const float *src = nullptr;      // n x 3, device
    int32_t n = 0;
    const float *tgt = nullptr;      // m x 3, device (AoS)
    int32_t m = 0;
    const float *rot = nullptr;      // k x 9, device
    int32_t k = 0;
    Params p{};
    const TargetRes *target = nullptr;   // resident reference (grid / field source)
    const float *host_tgt = nullptr;     // host AoS copy of the reference, if known
    bool exhaustive = false;             // Alg. 1: every lattice translation per rotation
};

// The option struct a caller passed, checked against its declared size (0: the
// full current size) and copied; missing trailing fields stay 0 (defaults).
dses_status copy_options(const dses_options *opt, dses_options *o);

// Device memory handed out from a fixed region instead of allocated: takes of
// 256-byte-aligned blocks from [base, base + cap); null when the region is spent.
struct Arena {
    char *base = nullptr;
    size_t cap = 0, used = 0;
    void *take(size_t bytes)
    {
        const size_t at = (used + 255) & ~size_t(255);
        if (at > cap || bytes > cap - at) return nullptr;
        used = at + bytes;
        return base + at;
    }
};

// Run one registration on `stream` using the context workspace (caller holds c->mu).
// With an arena every device buffer of the call comes from it and nothing is
// allocated (no timing events, no pinned staging, no top-k or pruning buffers).
dses_status run_plain(Context *c, const Job &job, hipStream_t stream, bool check_inputs,
                      dses_result *out, const dses_options &o, Arena *arena = nullptr);

void add_stats(Context *c, double vote_ms, double score_ms, double select_ms, double stage_ms,
               int64_t launches, int64_t pairs_voted, int64_t pairs_scored, int64_t cands);

// ref_block_population of a resident target, cached per (delta, box).
int64_t target_block_population(TargetRes *tm, const Params &p);
// x range of a resident target's staged fixed-point coordinates at pitch p.delta and
// box p.klo (sorting the reference on first use); false if the sorted vote cannot
// be used.
bool target_x_range(TargetRes *tm, const Params &p, int32_t *ylo, int32_t *yhi);
// Stage a resident target for geometry g and lane groups of gref points (cached by
// pitch, box origin and layout, with bank orders for a few strides; holds tm->grid_mu
// while building; synchronous on `stream`).
dses_status ensure_target_stage(TargetRes *tm, const Params &p, const Geom &g, int gref,
                                hipStream_t stream, const TargetRes::Stage **out);
// Build (or reuse) the resident target's cell grid for radius r; fills cg.
dses_status ensure_target_grid(TargetRes *tm, float r, CellGrid *cg);

// Distance field build (device), defined in field.hip.
hipError_t launch_df_build(const float *pts_soa, const int32_t *start, const HostGrid &grid,
                           int32_t res, const float *lo, const float *h, float r, float *out,
                           hipStream_t stream);

}  // namespace dses

struct dses_target {
    dses::TargetRes res;
};

struct dses_rotset {
    dses::RotRes res;
};
