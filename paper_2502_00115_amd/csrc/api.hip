// DSES C ABI: context, argument checking and the plain registration driver.
#include <hip/hip_runtime.h>

#include <cstddef>
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <string>
#include <unordered_map>
#include <vector>

#include "host.h"

namespace dses {

static thread_local std::string g_err;

void set_error(const std::string &msg) { g_err = msg; }

namespace {
std::mutex g_fault_mu;
int64_t g_fault_skip = 0, g_fault_count = 0;   // dses_debug_fail_allocs

// true if this allocation is one the injection makes fail
bool injected_failure()
{
    std::lock_guard<std::mutex> lk(g_fault_mu);
    if (g_fault_count <= 0) return false;
    if (g_fault_skip > 0) {
        --g_fault_skip;
        return false;
    }
    --g_fault_count;
    return true;
}
}  // namespace

hipError_t dev_alloc_raw(void **p, size_t bytes)
{
    *p = nullptr;
    if (injected_failure()) return hipErrorOutOfMemory;
    const hipError_t e = hipMalloc(p, bytes);
    if (e != hipSuccess) *p = nullptr;
    return e;
}

hipError_t host_alloc_raw(void **p, size_t bytes, unsigned int flags)
{
    *p = nullptr;
    if (injected_failure()) return hipErrorOutOfMemory;
    const hipError_t e = hipHostMalloc(p, bytes, flags);
    if (e != hipSuccess) *p = nullptr;
    return e;
}

dses_status DevBuf::ensure(size_t want)
{
    if (want <= bytes && ptr) return DSES_OK;
    release();
    size_t b = std::max<size_t>(want, 256);
    b = (b + 4095) & ~size_t(4095);
    if (dev_alloc(&ptr, b) != hipSuccess) {
        ptr = nullptr;
        bytes = 0;
        (void)hipGetLastError();
        set_error("device allocation of " + std::to_string(b) + " bytes failed");
        return DSES_E_NOMEM;
    }
    bytes = b;
    return DSES_OK;
}

void DevBuf::release()
{
    if (ptr) (void)hipFree(ptr);
    ptr = nullptr;
    bytes = 0;
}

dses_status PinnedBuf::ensure(size_t want)
{
    if (want <= bytes && ptr) return DSES_OK;
    release();
    const size_t b = (std::max<size_t>(want, 4096) + 4095) & ~size_t(4095);
    if (host_alloc(&ptr, b, hipHostMallocDefault) != hipSuccess) {
        ptr = nullptr;
        bytes = 0;
        (void)hipGetLastError();
        set_error("pinned host allocation of " + std::to_string(b) + " bytes failed");
        return DSES_E_NOMEM;
    }
    bytes = b;
    return DSES_OK;
}

void PinnedBuf::release()
{
    if (ptr) (void)hipHostFree(ptr);
    ptr = nullptr;
    bytes = 0;
}

static std::mutex g_init_mu;
static Context *g_ctx = nullptr;

static dses_status init_device(int device)
{
    std::lock_guard<std::mutex> lk(g_init_mu);
    if (g_ctx) {
        if (device >= 0 && device != g_ctx->device) {
            set_error("library already initialised on another device");
            return DSES_E_STATE;
        }
        return DSES_OK;
    }
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess || count <= 0) {
        (void)hipGetLastError();
        set_error("no HIP device available");
        return DSES_E_DEVICE;
    }
    if (device < 0) device = 0;
    if (device >= count) {
        set_error("device index out of range");
        return DSES_E_DEVICE;
    }
    hipDeviceProp_t prop;
    DSES_HIP(hipGetDeviceProperties(&prop, device));
    std::string arch = prop.gcnArchName;
    if (arch.rfind("gfx950", 0) != 0) {
        set_error("unsupported GPU architecture " + arch + " (gfx950 required)");
        return DSES_E_DEVICE;
    }
    DSES_HIP(hipSetDevice(device));
    auto *c = new Context();
    c->device = device;
    c->arch = arch;
    c->n_cu = prop.multiProcessorCount;
    int lds = 0;
    DSES_HIP(hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, device));
    c->lds_max = std::min(lds, 160 * 1024);
    void *hr = nullptr;
    hipError_t e = hipStreamCreateWithFlags(&c->stream, hipStreamNonBlocking);
    if (e == hipSuccess) e = host_alloc(&hr, sizeof(DevResult), hipHostMallocDefault);
    if (e != hipSuccess) {
        if (c->stream) (void)hipStreamDestroy(c->stream);
        delete c;
        DSES_HIP(e);
    }
    c->host_res = static_cast<DevResult *>(hr);
    g_ctx = c;
    return DSES_OK;
}

Context *ctx()
{
    if (!g_ctx && init_device(-1) != DSES_OK) return nullptr;
    if (g_ctx) (void)hipSetDevice(g_ctx->device);
    return g_ctx;
}

dses_status resolve_params(float eps, int metric, float delta_t, float tau, const float *t_min,
                           const float *t_max, int scorer, Params *p)
{
    if (!(eps > 0.0f) || !std::isfinite(eps)) {
        set_error("eps must be positive and finite");
        return DSES_E_INVAL;
    }
    if (metric < DSES_TRUNC_L2 || metric > DSES_VOTES) {
        set_error("unknown metric");
        return DSES_E_INVAL;
    }
    if (scorer < DSES_SCORER_AUTO || scorer > DSES_SCORER_DF) {
        set_error("unknown scorer");
        return DSES_E_INVAL;
    }
    p->eps = eps;
    p->delta = delta_t == 0.0f ? eps : delta_t;
    p->tau = tau == 0.0f ? eps : tau;
    if (!(p->delta > 0.0f) || !std::isfinite(p->delta) || !(p->tau > 0.0f) ||
        !std::isfinite(p->tau)) {
        set_error("delta_t and tau must be positive and finite");
        return DSES_E_INVAL;
    }
    p->r = std::max(p->eps, p->tau);
    p->metric = metric;
    p->scorer = scorer;
    float lo[3] = {-1.0f, -1.0f, -1.0f}, hi[3] = {1.0f, 1.0f, 1.0f};
    bool zero = true;
    if (t_min && t_max)
        for (int a = 0; a < 3; ++a) zero = zero && t_min[a] == 0.0f && t_max[a] == 0.0f;
    if (!zero)
        for (int a = 0; a < 3; ++a) { lo[a] = t_min[a]; hi[a] = t_max[a]; }
    for (int a = 0; a < 3; ++a) {
        if (!std::isfinite(lo[a]) || !std::isfinite(hi[a])) {
            set_error("translation box must be finite");
            return DSES_E_INVAL;
        }
        const double kl = std::ceil((double)lo[a] / (double)p->delta - 1e-4);
        const double kh = std::floor((double)hi[a] / (double)p->delta + 1e-4);
        if (!(kh >= kl) || kh - kl + 1 > 4096 || std::fabs(kl) > 1e6 || std::fabs(kh) > 1e6) {
            set_error("translation box is empty or has more than 4096 bins per axis");
            return DSES_E_INVAL;
        }
        p->klo[a] = (int32_t)kl;
        p->size[a] = (int32_t)(kh - kl + 1);
    }
    return DSES_OK;
}

int counter_bits_for(int64_t bound, int32_t n, int32_t m, const Params &p)
{
    if (bound > 65535) return 32;
    const int64_t plane_words = (int64_t)p.size[1] * p.size[2];
    const int64_t pps = std::max<int64_t>(1, std::min<int64_t>((kHistWordsMax & ~3) / plane_words,
                                                               p.size[0]));
    const int64_t nslabs32 = (p.size[0] + pps - 1) / pps;
    return (int64_t)n * m >= (int64_t)nslabs32 << 20 ? 32 : 16;
}

dses_status plan_geom(const Context *c, const Params &p, int32_t n, int32_t m, int counter_bits,
                      Geom *g)
{
    (void)c;
    g->n = n;
    g->m = m;
    g->delta = p.delta;
    lattice_scales(p.delta, &g->S16, &g->S15);
    g->eps = p.eps;
    g->tau = p.tau;
    g->r = p.r;
    g->metric = p.metric;
    g->lp = p.lp;
    for (int a = 0; a < 3; ++a) { g->klo[a] = p.klo[a]; g->size[a] = p.size[a]; }
    g->zbits = counter_bits == 16 ? 15 : 16;
    g->counter_bits = counter_bits;
    g->row_words = counter_bits == 16 ? (p.size[2] + 1) / 2 : p.size[2];
    const int64_t plane_words = (int64_t)p.size[1] * g->row_words;
    const int64_t avail = kHistWordsMax & ~int64_t(3);
    int64_t pps = avail / plane_words;
    if (pps < 1) {
        set_error("translation box plane (size_y * size_z bins) does not fit in LDS");
        return DSES_E_INVAL;
    }
    pps = std::min<int64_t>(pps, p.size[0]);
    const int64_t nslabs = (p.size[0] + pps - 1) / pps;
    pps = (p.size[0] + nslabs - 1) / nslabs;
    g->pps = (int32_t)pps;
    g->nslabs = (int32_t)nslabs;
    g->slab_words = (int32_t)(pps * plane_words);
    g->wide = 4 * plane_words > 0xFFFF ? 1 : 0;
    return DSES_OK;
}

// Parts of a lane group's windows in the windowed vote, a power of two: `asked` rounded
// down, or at most 96 units per slab for the 16 waves (128 of at least 128 sources on
// average, because 49 to 64 units leave a part of the waves without a last one: 5,520 x
// 1,540 points at 0.03 2.27 / 2.09 us a rotation, 5,520 x 3,103 at 0.052 3.48 / 3.21) and at
// most 8, with no part shorter than a block of 16 but for two units a wave.  Halving the
// parts of shorter ones took 0.78 to 0.93 of the time (100 x 3,000 points at 0.0118 2.37 /
// 1.86 us a rotation, 400 x 1,000 2.13 / 1.88), of parts of 20 to 300 sources 1.0 to 1.18
// (1,500 x 2,000 at 0.015 4.07 / 4.36, 4,000 x 1,000 2.41 / 2.74).
int window_parts(const Geom &g, int gref, float x_extent, int asked)
{
    int parts = 1;
    if (asked > 0) {
        while (parts < 16 && 2 * parts <= asked) parts *= 2;
        return parts;
    }
    const int groups = (g.m + gref - 1) / gref;
    const double window = (g.pps + (double)gref * x_extent / g.m) * g.n / (x_extent + g.size[0]);
    while (parts < 8) {
        const int units = groups * 2 * parts;
        const double part = window / (2 * parts);
        if (units > 128 || part < (units > 96 ? 128 : (units > 32 ? 16 : 0))) break;
        parts *= 2;
    }
    return parts;
}

// Costs per slab, in pairs of a 32-point group.  A group's windows cover its own x extent
// besides the slab's planes, so larger groups stream more sources, but they are fewer
// and need half the loads per pair; a unit's set-up is worth kUnit pairs.  64 points are
// taken only where every wave gets a group (1,500 x 300 points 0.25 / 0.28 us).  The
// general path pays more for a pair, a unit and a rotation, but it has groups of 16 points, which
// matter where even 32 span more than a slab, and whose pairs meet less often in one
// counter where a few lattice cells hold much of the reference.  The share of the pairs
// that lie in the box in x is that of two clouds of the reference's extent about its
// middle.  Constants fitted to 450 sizes and lattices; us a rotation, groups of 32 / 64 /
// general path: 2,000 x 8,192 at 0.03 3.66 / 3.48 / 5.00; 717 x 1,024 0.30 / 0.31 / 0.32;
// 200 x 17,555 at 0.0118 9.6 / 6.9 / 6.5; 12,000 x 100 8.1 / 14.5 / 5.7; 4,000 x 1,000 4.5 /
// 6.4 / 4.0; 5,298 x 853 at 0.046, a third of them in one cell, 2.7 / 2.7 / 2.0.
VoteLayout choose_layout(const Geom &g, bool sorted, float x_extent, int64_t population, int asked,
                         bool batched)
{
    constexpr double kUnit = 300.0, kLarge = 0.95;
    constexpr double kGeneralUnit = 600.0, kGeneral = 1.13, kGeneralRotation = 12000.0;
    VoteLayout l{0, 64, 0, 0.0};
    if (!sorted) return l;
    l.group = choose_group(g, x_extent, asked, 0);
    if (g.wide) return l;
    const double m = g.m, X = x_extent;
    const double u = std::min(1.0, g.size[0] / (2.0 * X));
    const double pairs = (double)g.n * m * u * (2.0 - u) / g.nslabs;
    auto reach = [&](int group) { return 1.0 + group * X / (m * g.pps); };
    // the part of the reference in the fullest block of cells, beyond what a surface has
    // there and one set of lanes
    const double full = std::max(0.0, (double)(population - 16) / m - 8.0 / (X * X));
    double cost[2];
    for (int i = 0; i < 2; ++i) {
        const int gref = 32 << i, groups = (g.m + gref - 1) / gref;
        cost[i] = kUnit * groups * window_parts(g, gref, x_extent, 0) +
                  (i ? kLarge : 1.0) * pairs * (groups * gref / m) * reach(gref) *
                      (1.0 + 5.0 * full);
    }
    const bool large = asked ? asked > 32 : (batched && g.counter_bits == 32) ||
                                              (g.m > 15 * 64 && cost[1] < cost[0]);
    l.gref = large ? 64 : 32;
    l.parts = window_parts(g, l.gref, x_extent, 0);
    l.general = HUGE_VAL;
    if (asked > 16) return l;
    const int groups = (g.m + 15) / 16;
    const double general = kGeneralRotation / g.nslabs +
                           kGeneralUnit * groups * vote_parts_auto(groups) +
                           kGeneral * pairs * (groups * 16 / m) * reach(16) * (1.0 + 2.2 * full);
    l.group = 16;
    l.general = general / cost[large];
    // windows of a few sources over many groups: the general path's units are cheaper
    if (large && g.m > 64 * 64 && (g.pps + 64 * X / m) * g.n / (X + g.size[0]) < 4.0) {
        l.group = 64;
        l.general = std::min(l.general, 0.94);
    }
    return l;
}

// Smaller groups span less x, so their windows carry less slack (about group * X
// source-bins per slab over all groups, X the reference's x extent in bins), but there
// are more work units, each costing about kUnitSteps wave steps of set-up, padding and
// slab-end imbalance (fitted); rho = n / (X + size_x) sources per bin turns a step into
// 64 / rho source-bins.  The size with the least modelled cost wins (ties: the larger).
// Box +-1 at a pitch of 0.01, ms a call with 16 / 32 / 64 points: 717 x
// 1,024 points, 2,048 rotations 7.2 / 7.8 / 8.8; 2,000 x 4,096, 1,024 rotations 15.5 /
// 13.4 / 13.9.
int choose_group(const Geom &g, float x_extent, int asked, int vote_parts)
{
    constexpr float kUnitSteps = 4.9f;
    if (asked) return asked;
    const float per_unit = kUnitSteps * 64.0f * (x_extent + (float)g.size[0]) / (float)g.n;
    int best = 0;
    float least = 0.0f;
    for (int group = 64; group >= 16; group >>= 1) {
        const int groups = (g.m + group - 1) / group;
        const int parts = vote_parts > 0 ? vote_parts : vote_parts_auto(groups);
        const float cost = (float)group * x_extent + per_unit * (float)(groups * parts);
        if (!best || cost < least) {
            least = cost;
            best = group;
        }
    }
    return best;
}

// A workgroup holds a compute unit, so k rotations run in ceil(k / CUs) rounds and the
// last may be nearly empty.  Items of fewer slabs fill it; each repeats the sort of the
// sources, and the scores move to a launch of their own.  The estimate is the largest
// sum of a workgroup's items, in cycles: a compute unit votes about 8.5 pairs per cycle,
// a slab's clear, waits and scan take about 8,000, a sort 8,000 and 3 per source, the
// second launch 24,000.  The votes are spread over the slabs as the differences of two
// clouds of the reference's x extent (a triangle; the middle slabs hold most), about the
// box's middle or a quarter of the box to either side: where the clouds lie is not known
// here, and two slabs of which one holds most votes lose by being two items.
// Measured (ms, whole / in parts): 2,000 x 8,192 points at 0.03, 100 rotations 1.32 /
// 0.82, 300 rotations 2.33 / 1.63, 576 rotations 3.15 / 2.50; 4,096 x 16,384 points 4.21 / 2.23,
// 7.55 / 4.88, 10.77 / 8.23; 1,000 x 8,192 points at 0.05 (two slabs), 576 rotations 1.83 /
// 1.98, so the rule leaves it whole.  The estimate itself takes 9 us at 15 slabs and 13 at
// 84 (34 and 68 with a division per part, place and probe).
int choose_parts(const Geom &g, int32_t k, float x_extent, int n_cu, double *share)
{
    *share = 1.0;
    constexpr int kMostParts = 16, kProbes = 16;
    const int slabs = (g.size[0] + g.pps - 1) / g.pps;
    if (slabs < 2 || k > 8 * n_cu) return 1;       // at most one round of nine to gain
    const double width = std::max(1.0, (double)x_extent);
    auto below = [&](double x) {                   // share of the differences below x bins
        const double u = std::min(1.0, std::max(-1.0, x / width));
        return u < 0 ? 0.5 * (1 + u) * (1 + u) : 1 - 0.5 * (1 - u) * (1 - u);
    };
    const double pairs = (double)g.n * g.m / 8.5, sort = 8000.0 + 3.0 * g.n;
    std::vector<double> weight[3];                 // of the slabs, by the clouds' place
    for (int side = 0; side < 3; ++side)
        for (int s = 0; s < slabs; ++s) {
            const double x0 = s * g.pps - 0.5 * g.size[0] + 0.25 * (side - 1) * g.size[0];
            weight[side].push_back(8000.0 + pairs * (below(x0 + g.pps) - below(x0)));
        }
    // time[side]: the largest sum of a workgroup's items
    auto estimate = [&](int parts, double *time) {
        double item[3][kMostParts];
        for (int side = 0; side < 3; ++side) {
            time[side] = 0;
            for (int p = 0; p < parts; ++p) {
                item[side][p] = sort;
                for (int s = p; s < slabs; s += parts) item[side][p] += weight[side][s];
            }
        }
        for (int q = 0; q < kProbes; ++q) {        // workgroups q n_cu / 16
            const int b = q * n_cu / kProbes;
            if (b >= k * parts) break;
            double sum[3] = {0, 0, 0};
            uint32_t before = 0;                   // its items b, b + n_cu, ... of earlier parts
            for (int p = 0; p < parts; ++p) {
                const int e = (p + 1) * k;
                const uint32_t upto = e > b ? (uint32_t)(e - b + n_cu - 1) / (uint32_t)n_cu : 0;
                for (int side = 0; side < 3; ++side)
                    sum[side] += item[side][p] * (double)(upto - before);
                before = upto;
            }
            for (int side = 0; side < 3; ++side) time[side] = std::max(time[side], sum[side]);
        }
    };
    double whole[3], split[3];
    estimate(1, whole);
    double least = 0.92;
    int best = 1;
    for (int parts = 2; parts <= std::min(slabs, kMostParts); ++parts) {
        estimate(parts, split);
        double time = 0;                           // as a share of the time in one piece
        for (int side = 0; side < 3; ++side)
            time = std::max(time, (split[side] + 24000.0) / whole[side]);
        if (time < least) {
            *share = least = time;
            best = parts;
        }
    }
    return best;
}

StageDesc stage_desc(const Geom &g, int gref, bool arrange, const float *tgt, const int32_t *perm,
                     int32_t *yq, float *yt)
{
    return StageDesc{tgt,     perm, g.m,  g.S16, g.S15, {g.klo[0], g.klo[1], g.klo[2]},
                     g.zbits, gref ? gref : 64, arrange ? 1 : 0,
                     g.row_words * g.size[1], g.row_words, yq, yt};
}

// Largest vote count any bin can reach: for a fixed source point the pairs that
// share a bin have reference points inside one cube of side delta (widened by the
// float rounding of the bin decision), and such a cube meets at most 2 cells per
// axis of a grid of pitch slightly above delta.  So every count is at most
// n * (largest reference population of a 2x2x2 block of cells).
int64_t ref_block_population(const float *tgt, int32_t m, const Params &p)
{
    double maxabs = 0.0;
    for (int64_t e = 0; e < 3 * (int64_t)m; ++e) maxabs = std::max(maxabs, (double)std::fabs(tgt[e]));
    int32_t kmax = 0;
    for (int a = 0; a < 3; ++a) kmax = std::max(kmax, std::abs(p.klo[a]) + p.size[a]);
    const double s = 1.0 / (double)p.delta;
    const double slack = 16.0 * 5.97e-8 * (4.0 * maxabs * s + kmax + 2.0);   // bin units
    const double h = (double)p.delta * (1.0 + std::max(1e-3, 4.0 * slack));
    auto key = [](int64_t x, int64_t y, int64_t z) {
        return ((x + (1 << 20)) << 42) | ((y + (1 << 20)) << 21) | (z + (1 << 20));
    };
    // points per cell of pitch h; the bound is the largest total of a block of
    // 2 x 2 x 2 cells.  When the cells span a modest box, counts go to a dense
    // array with a one-cell margin, and the 8 blocks of each occupied cell are summed
    // there, first along z (8,192 points: 266 us with each point's 8 blocks of 8 cells,
    // 168 so); otherwise a hash map of cells and blocks gives the same number.
    std::vector<int64_t> ci(3 * (size_t)m);
    int64_t lo[3] = {INT64_MAX, INT64_MAX, INT64_MAX}, hi[3] = {INT64_MIN, INT64_MIN, INT64_MIN};
    for (int32_t j = 0; j < m; ++j)
        for (int a = 0; a < 3; ++a) {
            const double v = (double)tgt[3 * (size_t)j + a] / h;
            int64_t c = (int64_t)v;                          // toward zero
            c -= v < (double)c;                              // floor
            ci[3 * (size_t)j + a] = c;
            lo[a] = std::min(lo[a], c);
            hi[a] = std::max(hi[a], c);
        }
    if (m > 0 && hi[0] - lo[0] < (1 << 12) && hi[1] - lo[1] < (1 << 12) &&
        hi[2] - lo[2] < (1 << 12)) {
        const int64_t D1 = hi[1] - lo[1] + 3, D2 = hi[2] - lo[2] + 3;
        const int64_t cells = (hi[0] - lo[0] + 3) * D1 * D2;
        if (cells <= ((int64_t)1 << 21)) {
            thread_local std::vector<int32_t> cnt;       // all zero between calls
            if ((int64_t)cnt.size() < cells) cnt.assign((size_t)cells, 0);
            auto at = [&](int32_t j) {
                return ((ci[3 * (size_t)j] - lo[0] + 1) * D1 + (ci[3 * (size_t)j + 1] - lo[1] + 1)) * D2 +
                       (ci[3 * (size_t)j + 2] - lo[2] + 1);
            };
            std::vector<int32_t> occupied;
            occupied.reserve((size_t)m);
            for (int32_t j = 0; j < m; ++j) {
                const int64_t c = at(j);
                if (cnt[(size_t)c]++ == 0) occupied.push_back((int32_t)c);
            }
            int64_t best = 0;
            for (const int32_t c : occupied) {
                int32_t z[3][3][2];              // pairs along z of the 27 cells around c
                for (int x = 0; x < 3; ++x)
                    for (int y = 0; y < 3; ++y) {
                        const int32_t *row = cnt.data() + (c + ((x - 1) * D1 + (y - 1)) * D2);
                        z[x][y][0] = row[-1] + row[0];
                        z[x][y][1] = row[0] + row[1];
                    }
                for (int x = 0; x < 2; ++x)
                    for (int y = 0; y < 2; ++y)
                        for (int b = 0; b < 2; ++b)
                            best = std::max<int64_t>(best, (int64_t)z[x][y][b] + z[x + 1][y][b] +
                                                               z[x][y + 1][b] + z[x + 1][y + 1][b]);
            }
            for (const int32_t c : occupied) cnt[(size_t)c] = 0;
            return best;
        }
    }
    std::unordered_map<int64_t, int32_t> cell;
    cell.reserve((size_t)m * 2);
    for (int32_t j = 0; j < m; ++j)
        cell[key(ci[3 * (size_t)j], ci[3 * (size_t)j + 1], ci[3 * (size_t)j + 2])] += 1;
    std::unordered_map<int64_t, int64_t> block;
    block.reserve(cell.size() * 16);
    for (const auto &kv : cell) {
        const int64_t z = (kv.first & ((1 << 21) - 1)) - (1 << 20);
        const int64_t y = ((kv.first >> 21) & ((1 << 21) - 1)) - (1 << 20);
        const int64_t x = (kv.first >> 42) - (1 << 20);
        for (int ox = -1; ox <= 0; ++ox)
            for (int oy = -1; oy <= 0; ++oy)
                for (int oz = -1; oz <= 0; ++oz) block[key(x + ox, y + oy, z + oz)] += kv.second;
    }
    int64_t best = 0;
    for (const auto &kv : block) best = std::max(best, kv.second);
    return best;
}

int64_t counter_bound(const float *tgt, int32_t m, int32_t n, const Params &p)
{
    return ref_block_population(tgt, m, p) * (int64_t)n;
}

// ---------------------------------------------------------------------------
// exact cell grid (host build)
// ---------------------------------------------------------------------------
dses_status build_grid(const float *tgt, int32_t m, float r, HostGrid *out)
{
    // Cell pitch slightly above r so that, despite float rounding of the cell
    // index, every reference point within r of a query is in the 27 cells around
    // the query's cell.
    const float h = r * 1.001f;
    out->inv = 1.0f / h;
    float mn[3] = {tgt[0], tgt[1], tgt[2]}, mx[3] = {tgt[0], tgt[1], tgt[2]};
    for (int32_t j = 1; j < m; ++j)
        for (int a = 0; a < 3; ++a) {
            mn[a] = std::min(mn[a], tgt[3 * j + a]);
            mx[a] = std::max(mx[a], tgt[3 * j + a]);
        }
    int64_t ncell = 1;
    for (int a = 0; a < 3; ++a) {
        out->lo[a] = mn[a];
        const double span = ((double)mx[a] - (double)mn[a]) * (double)out->inv;
        out->dim[a] = (int32_t)std::floor(span) + 2;
        ncell *= out->dim[a];
    }
    if (ncell > (int64_t)64 << 20) {
        set_error("reference extent too large for the cell grid at this eps/tau");
        return DSES_E_INVAL;
    }
    std::vector<int32_t> cell(m);
    out->start.assign((size_t)ncell + 1, 0);
    for (int32_t j = 0; j < m; ++j) {
        int32_t id[3];
        for (int a = 0; a < 3; ++a) {
            const float u = (tgt[3 * j + a] - out->lo[a]) * out->inv;
            id[a] = std::min(std::max((int32_t)std::floor(u), 0), out->dim[a] - 1);
        }
        cell[j] = (id[0] * out->dim[1] + id[1]) * out->dim[2] + id[2];
        out->start[cell[j] + 1]++;
    }
    for (int64_t q = 0; q < ncell; ++q) out->start[q + 1] += out->start[q];
    std::vector<int32_t> cur(out->start.begin(), out->start.end() - 1);
    out->pts.assign((size_t)4 * m, 0.0f);
    for (int32_t j = 0; j < m; ++j) {
        const int32_t at = cur[cell[j]]++;
        for (int a = 0; a < 3; ++a) out->pts[(size_t)4 * at + a] = tgt[3 * j + a];
    }
    return DSES_OK;
}

// ---------------------------------------------------------------------------
// host-side input checks
// ---------------------------------------------------------------------------
// The fixed-point vote needs every staged reference value |y s + 1/2 - k_lo|
// below 2^13 bins, so that every pair difference and the padding values stay
// apart in 32 bits (a rotated source value is saturated at 2^14 bins instead:
// beyond it no pair with such a reference can land in the box).
float ref_coord_limit(const Params &p)
{
    int32_t kmax = 0;
    for (int a = 0; a < 3; ++a)
        kmax = std::max(kmax, std::max(std::abs(p.klo[a]), std::abs(p.klo[a] + p.size[a])));
    const double lim = ((double)(1 << 13) - kmax - 8.0) * (double)p.delta;
    return (float)std::min(std::max(lim, 0.0), 1.0e4);
}

static dses_status check_host_inputs(const float *src, int64_t n, const float *tgt, int64_t m,
                                     const float *rot, int64_t k, float limit)
{
    for (int64_t e = 0; e < 3 * n; ++e)
        if (!(std::fabs(src[e]) <= kSrcCoordLimit)) {
            set_error("source coordinate is non-finite or too large for the lattice");
            return DSES_E_INVAL;
        }
    if (tgt)
        for (int64_t e = 0; e < 3 * m; ++e)
            if (!(std::fabs(tgt[e]) <= limit)) {
                set_error("reference coordinate is non-finite or too large for the lattice");
                return DSES_E_INVAL;
            }
    if (rot)
        for (int64_t q = 0; q < k; ++q) {
            const float *R = rot + 9 * q;
            for (int i = 0; i < 3; ++i)
                for (int j = 0; j < 3; ++j) {
                    float d = R[i] * R[j] + R[3 + i] * R[3 + j] + R[6 + i] * R[6 + j];
                    d -= (i == j) ? 1.0f : 0.0f;
                    if (!(std::fabs(d) <= 1e-4f)) {
                        set_error("rotation " + std::to_string(q) +
                                  " is not orthonormal (|R^T R - I| > 1e-4) or not finite");
                        return DSES_E_INVAL;
                    }
                }
        }
    return DSES_OK;
}

void add_stats(Context *c, double vote_ms, double score_ms, double select_ms, double stage_ms,
               int64_t launches, int64_t pairs_voted, int64_t pairs_scored, int64_t cands)
{
    std::lock_guard<std::mutex> lk(c->stats_mu);
    c->stats.vote_score_ms += vote_ms;
    c->stats.score_ms += score_ms;
    c->stats.select_ms += select_ms;
    c->stats.stage_ms += stage_ms;
    c->stats.vote_score_launches += launches;
    c->stats.pairs_voted += pairs_voted;
    c->stats.pairs_scored += pairs_scored;
    c->stats.candidates += cands;
}

// Order by ascending x, equal x in index order (-0 equals 0).  From 512 points on by
// three counting passes over 11 bits of the key each, below by comparison (us, comparison
// / counting: 512 points 6.2 / 5.5, 2,048 points 84 / 15, 8,192 points 538 / 72).
void sort_by_x(const float *tgt, int32_t m, std::vector<int32_t> *perm)
{
    perm->resize(m);
    if (m < 512) {
        std::vector<std::pair<float, int32_t>> kv((size_t)m);
        for (int32_t j = 0; j < m; ++j) kv[j] = {tgt[3 * (size_t)j], j};
        std::sort(kv.begin(), kv.end());
        for (int32_t j = 0; j < m; ++j) (*perm)[j] = kv[j].second;
        return;
    }
    std::vector<uint64_t> kv((size_t)m), to((size_t)m);      // key, index
    uint32_t first[3][2048] = {};
    for (int32_t j = 0; j < m; ++j) {
        uint32_t u;
        std::memcpy(&u, &tgt[3 * (size_t)j], sizeof(u));
        if (u == 0x80000000u) u = 0;
        u ^= (u >> 31) ? 0xFFFFFFFFu : 0x80000000u;          // ascending as unsigned
        kv[j] = (uint64_t)u << 32 | (uint32_t)j;
        for (int d = 0; d < 3; ++d) first[d][(u >> (11 * d)) & 2047]++;
    }
    for (int d = 0; d < 3; ++d) {
        uint32_t at = 0;
        for (uint32_t &f : first[d]) {
            const uint32_t c = f;
            f = at;
            at += c;
        }
        for (int32_t j = 0; j < m; ++j)
            to[first[d][(kv[j] >> (32 + 11 * d)) & 2047]++] = kv[j];
        kv.swap(to);
    }
    for (int32_t j = 0; j < m; ++j) (*perm)[j] = (int32_t)(uint32_t)kv[j];
}

void lattice_scales(float delta, double *S16, double *S15)
{
    const double s = 1.0 / (double)delta;
    *S16 = s * 65536.0;
    *S15 = s * 32768.0;
}

// The staging arithmetic of one reference x coordinate (two rounded double
// operations, then to the nearest integer, halves to even).
static int32_t stage_x(float y, double S16, int32_t klo_x)
{
    double v = (double)y * S16;
    v = v + (0.5 - (double)klo_x) * 65536.0;
    return (int32_t)std::nearbyint(v);
}

bool ref_x_range(const float *tgt, const std::vector<int32_t> &perm, float delta, int32_t klo_x,
                 int32_t *ylo, int32_t *yhi)
{
    if (perm.empty()) return false;
    double S16, S15;
    lattice_scales(delta, &S16, &S15);
    *ylo = stage_x(tgt[3 * (size_t)perm.front()], S16, klo_x);
    *yhi = stage_x(tgt[3 * (size_t)perm.back()], S16, klo_x);
    return *yhi >= *ylo;
}

void source_buckets(int32_t ylo, int32_t yhi, int32_t size_x, int32_t *sb_lo, int32_t *sb_shift,
                    int32_t *sb_n)
{
    // a source votes only if some Y - P lies in [0, size_x 2^16): P in
    // (ylo - size_x 2^16, yhi]
    const int64_t lo = (int64_t)ylo - ((int64_t)size_x << 16) + 1;
    const int64_t range = (int64_t)yhi - lo + 1;
    // 16 buckets per bin when the range fits: window ends are rounded to a bucket,
    // and finer buckets measured faster up to 16 (4,096-point sources against
    // 16,384 points: 2.4% against 4 per bin; 717 against 1,024: 0.3%; 32 per bin
    // no better, 64 slower)
    int shift = 12;
    while ((range >> shift) + 1 > kSrcBuckets && shift < 31) ++shift;
    *sb_lo = (int32_t)lo;
    *sb_shift = shift;
    // only as many buckets as the range needs (the sort clears and scans them all)
    const int64_t need = (range >> shift) + 2;
    *sb_n = (int32_t)std::min<int64_t>(kSrcBuckets, (need + kBlock - 1) / kBlock * kBlock);
}

dses_status apply_metric_options(const dses_options &o, Params *p)
{
    if (!(o.p >= 0.0f && o.p <= 1.0f)) {
        set_error("the Lp exponent p must be in (0, 1] (0: default 0.5)");
        return DSES_E_INVAL;
    }
    p->lp = o.p > 0.0f ? o.p : 0.5f;
    if (p->metric == DSES_VOTES && o.q > 0.0f) {
        set_error("q-pruning has no effect with DSES_VOTES");
        return DSES_E_INVAL;
    }
    if (o.lane_group != 0 && o.lane_group != 16 && o.lane_group != 32 && o.lane_group != 64) {
        set_error("lane_group must be 0 (automatic), 16, 32 or 64");
        return DSES_E_INVAL;
    }
    if (o.df_lookup != DSES_DF_NEAREST && o.df_lookup != DSES_DF_TRILINEAR) {
        set_error("df_lookup must be DSES_DF_NEAREST or DSES_DF_TRILINEAR");
        return DSES_E_INVAL;
    }
    p->df_lookup = o.df_lookup;
    return DSES_OK;
}

dses_status copy_options(const dses_options *opt, dses_options *o)
{
    *o = dses_options{};
    if (!opt) return DSES_OK;
    const size_t given = opt->struct_size ? opt->struct_size : sizeof(dses_options);
    // the first field that existed in every version ends at lane_group
    if (given < offsetof(dses_options, df_lookup) || given > sizeof(dses_options)) {
        set_error("dses_options.struct_size is not a size of this structure");
        return DSES_E_INVAL;
    }
    std::memcpy(o, opt, given);
    return DSES_OK;
}

static int effective_scorer(const Job &job)
{
    if (job.p.metric == DSES_VOTES) return kScoreVotes;
    int s = job.p.scorer;
    if (s == DSES_SCORER_AUTO)
        s = (job.target && job.target->df && job.target->df_r == job.p.r &&
             job.p.metric != DSES_TRUNC_L1)
                ? DSES_SCORER_DF
                : DSES_SCORER_GRID;
    return s;
}

// ---------------------------------------------------------------------------
// the plain driver
// ---------------------------------------------------------------------------
dses_status run_plain(Context *c, const Job &job, hipStream_t stream, bool check_inputs,
                      dses_result *out, const dses_options &o, Arena *arena)
{
    TraceRange whole("dses.registration");
    TraceRange prepare("dses.prepare");        // host work and staging before the launches
    // a device buffer of the call: from the arena when given, else the context's
    auto dbuf = [&](DevBuf &b, size_t bytes, void **ptr) -> dses_status {
        if (arena) {
            *ptr = arena->take(bytes);
            if (*ptr) return DSES_OK;
            set_error("the call needs more than the " + std::to_string(arena->cap >> 20) +
                      " MiB scratch array of the no-allocation entry point");
            return DSES_E_NOMEM;
        }
        const dses_status s = b.ensure(bytes);
        *ptr = b.ptr;
        return s;
    };
    if (arena && (o.q > 0.0f || o.top_k > 0 || c->timing_enabled || job.exhaustive)) {
        set_error("the no-allocation path takes no pruning, top-k, timing or Alg. 1");
        return DSES_E_INVAL;
    }
    const Params &p = job.p;
    void *records = o.records;
    const bool on_device = (o.flags & DSES_DEVICE_PTRS) != 0;
    if (o.top_k < 0 || o.top_k > DSES_TOPK_MAX || (o.top_k > 0 && !o.topk) ||
        !(o.q >= 0.0f && o.q <= 1.0f)) {
        set_error("top_k must be in 0..DSES_TOPK_MAX with a topk buffer, q in [0, 1]");
        return DSES_E_INVAL;
    }
    const int scorer = effective_scorer(job);
    if (scorer == DSES_SCORER_DF) {
        if (!job.target || !job.target->df) {
            set_error("DF scorer needs a resident target created with a distance field");
            return DSES_E_INVAL;
        }
        if (job.target->df_r != p.r) {
            set_error("distance field truncation must equal max(eps, tau)");
            return DSES_E_INVAL;
        }
        if (p.metric == DSES_TRUNC_L1) {
            set_error("the DF scorer does not support DSES_TRUNC_L1");
            return DSES_E_INVAL;
        }
    }
    const size_t m = (size_t)job.m;
    dses_status st;
    // host copy of the reference: needed for the counter bound and the cell grid
    std::vector<float> host_copy;
    const float *ht = job.target ? job.target->host_aos.data() : job.host_tgt;
    if (!ht) {
        host_copy.resize(3 * m);
        const size_t tb = 3 * m * sizeof(float);
        void *to = host_copy.data();
        if (!arena) {                          // through pinned memory: one copy, one wait
            if ((st = c->host_stage.ensure(tb)) != DSES_OK) return st;
            to = c->host_stage.ptr;
        }
        DSES_HIP(hipMemcpyAsync(to, job.tgt, tb, hipMemcpyDeviceToHost, stream));
        DSES_HIP(hipStreamSynchronize(stream));
        if (!arena) std::memcpy(host_copy.data(), to, tb);
        for (float v : host_copy)
            if (!(std::fabs(v) <= ref_coord_limit(p))) {
                set_error("reference coordinate is non-finite or too large for the lattice");
                return DSES_E_INVAL;
            }
        ht = host_copy.data();
    }
    const int64_t population = job.target
                                   ? target_block_population(const_cast<TargetRes *>(job.target), p)
                                   : ref_block_population(ht, job.m, p);
    const int counter_bits = counter_bits_for(population * job.n, job.n, job.m, p);
    Geom g;
    if ((st = plan_geom(c, p, job.n, job.m, counter_bits, &g)) != DSES_OK) return st;

    // Reference sorted by x, and the range of its staged fixed-point x coordinate
    // (the same arithmetic as the staging kernel) for the source buckets, so each
    // wave can restrict its vote loop to reachable points.
    std::vector<int32_t> perm_local;
    const std::vector<int32_t> *perm = nullptr;
    if (job.target) {
        auto *tm = const_cast<TargetRes *>(job.target);
        std::lock_guard<std::mutex> lk(tm->grid_mu);
        if (tm->perm_x.empty()) sort_by_x(ht, job.m, &tm->perm_x);
        perm = &tm->perm_x;
    } else {
        sort_by_x(ht, job.m, &perm_local);
        perm = &perm_local;
    }
    int32_t ylo = 0, yhi = 0;
    const bool sorted = job.n <= kSortMax && ref_x_range(ht, *perm, p.delta, p.klo[0], &ylo, &yhi);
    const float x_extent = ref_x_extent(ylo, yhi);
    VoteLayout lay{};                          // Alg. 1 takes no votes
    if (!job.exhaustive)
        lay = choose_layout(g, sorted, x_extent, population, o.lane_group, false);
    double share = 1.0;                        // of its time that a split leaves the windowed vote
    int parts = lay.gref && !arena && !(o.q > 0.0f)
                    ? choose_parts(g, job.k, x_extent, c->n_cu, &share)
                    : 1;
    if (lay.general < share) {
        lay.gref = 0;
        lay.parts = 0;
        parts = 1;
    }
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((int64_t)job.k * parts, c->n_cu));
    void *d_perm = nullptr, *d_scratch = nullptr, *d_yq = nullptr, *d_yt = nullptr;
    void *d_rec = nullptr, *d_status = nullptr;
    if (sorted && (st = dbuf(c->scratch, (size_t)grid * slot_words(job.n) * sizeof(int32_t),
                             &d_scratch)) != DSES_OK)
        return st;

    if (parts > 1 &&
        (st = c->modes.ensure((size_t)job.k * parts * 2 * sizeof(uint32_t))) != DSES_OK)
        return st;
    if (o.q > 0.0f && (st = c->prune.ensure(64)) != DSES_OK) return st;
    if ((st = dbuf(c->yq, stage_words(m) * sizeof(int32_t), &d_yq)) != DSES_OK) return st;
    if ((st = dbuf(c->yt, 3 * m * sizeof(float), &d_yt)) != DSES_OK) return st;
    // with an arena the records go straight to the caller's buffer when it gives one
    if (arena && records)
        d_rec = records;
    else if ((st = dbuf(c->rec, (size_t)job.k * sizeof(dses_record), &d_rec)) != DSES_OK)
        return st;

    SweepArgs a{};
    a.src = job.src;
    a.rot = job.rot;
    a.yq = static_cast<int32_t *>(d_yq);
    a.yt = static_cast<float *>(d_yt);
    a.rec = static_cast<dses_record *>(d_rec);
    a.k = job.k;
    a.g = g;
    a.scratch = sorted ? static_cast<int32_t *>(d_scratch) : nullptr;
    a.scratch_stride = job.n;
    source_buckets(ylo, yhi, g.size[0], &a.sb_lo, &a.sb_shift, &a.sb_n);
    a.gref = lay.gref;
    a.group = lay.group;
    a.vote_parts = lay.parts;

    HostGrid hg;                               // of a reference that is not resident
    if (scorer == DSES_SCORER_GRID) {
        const TargetRes *t = job.target;
        if (t) {
            if ((st = ensure_target_grid(const_cast<TargetRes *>(t), p.r, &a.grid)) != DSES_OK)
                return st;
        } else {
            if ((st = build_grid(ht, job.m, p.r, &hg)) != DSES_OK) return st;
        }
    } else if (scorer == DSES_SCORER_DF) {
        const TargetRes *t = job.target;
        a.field.val = t->df;
        a.field.res = t->df_res;
        a.field.r = t->df_r;
        a.field.lookup = job.p.df_lookup;
        for (int q = 0; q < 3; ++q) { a.field.lo[q] = t->df_lo[q]; a.field.inv[q] = t->df_inv[q]; }
    }

    const bool timing = c->timing_enabled;     // never with an arena
    hipEvent_t ev[4] = {};
    auto rec_ev = [&](int i) { if (timing) (void)hipEventRecord(ev[i], stream); };

    // What the host prepared, on the device: the status words (zero), the order by x and
    // the cell grid.  Small calls are bound by launches, copies and waits, so without an
    // arena these are one block and one asynchronous copy from pinned memory, which the
    // next call reuses only after this one's final synchronisation; the check shares a
    // launch with the staging, the result comes back by the selection's own stores, and
    // records on the device need no second wait: 64 x 256 points, 577 rotations 184 ->
    // 131 us; Alg. 1 over the same sizes and 21^3 translations 534 -> 478 us; 501 x 1,531
    // host points, 9,973 rotations 3.46 -> 3.32 ms.
    const size_t pb = hg.pts.size() * sizeof(float), sb = hg.start.size() * sizeof(int32_t);
    void *d_pts = nullptr, *d_start = nullptr;
    if (arena) {
        // no pinned staging: the copies read the host vectors, which live until the
        // synchronisation
        if ((st = dbuf(c->upload, 64, &d_status)) != DSES_OK) return st;
        if ((st = dbuf(c->upload, m * sizeof(int32_t), &d_perm)) != DSES_OK) return st;
        if (pb && (st = dbuf(c->upload, pb, &d_pts)) != DSES_OK) return st;
        if (sb && (st = dbuf(c->upload, sb, &d_start)) != DSES_OK) return st;
        DSES_HIP(launch_clear(static_cast<uint32_t *>(d_status), 16, stream));
        DSES_HIP(hipMemcpyAsync(d_perm, perm->data(), m * sizeof(int32_t), hipMemcpyHostToDevice,
                                stream));
        if (pb)
            DSES_HIP(hipMemcpyAsync(d_pts, hg.pts.data(), pb, hipMemcpyHostToDevice, stream));
        if (sb)
            DSES_HIP(hipMemcpyAsync(d_start, hg.start.data(), sb, hipMemcpyHostToDevice, stream));
        if (pb) DSES_HIP(hipStreamSynchronize(stream));
    } else {
        auto up = [](size_t v) { return (v + 255) & ~(size_t)255; };
        const size_t o_perm = 256, o_pts = o_perm + up(m * sizeof(int32_t)),
                     o_start = o_pts + up(pb), total = o_start + sb;
        if ((st = c->upload.ensure(total)) != DSES_OK) return st;
        if ((st = c->host_stage.ensure(total)) != DSES_OK) return st;
        // all that may fail on the host comes before the copy: a call that ends early would
        // leave it in flight behind its stream's work, to overwrite the status words of a
        // later call on another stream
        if (timing)
            for (auto &e : ev) DSES_HIP(hipEventCreate(&e));
        char *hs = static_cast<char *>(c->host_stage.ptr), *ds = static_cast<char *>(c->upload.ptr);
        std::memset(hs, 0, o_perm);
        std::memcpy(hs + o_perm, perm->data(), m * sizeof(int32_t));
        if (pb) std::memcpy(hs + o_pts, hg.pts.data(), pb);
        if (sb) std::memcpy(hs + o_start, hg.start.data(), sb);
        DSES_HIP(hipMemcpyAsync(ds, hs, total, hipMemcpyHostToDevice, stream));
        d_status = ds;
        d_perm = ds + o_perm;
        d_pts = ds + o_pts;
        d_start = ds + o_start;
    }
    uint32_t *bad = static_cast<uint32_t *>(d_status);
    if (scorer == DSES_SCORER_GRID && !job.target) {
        a.grid.pts = static_cast<float *>(d_pts);
        a.grid.start = static_cast<int32_t *>(d_start);
        for (int q = 0; q < 3; ++q) { a.grid.lo[q] = hg.lo[q]; a.grid.dim[q] = hg.dim[q]; }
        a.grid.inv = hg.inv;
    }

    prepare.end();
    TraceRange device("dses.sweep_select");    // launches to the result on the host
    rec_ev(0);
    const bool arrange = worth_arranging(g, a.gref, x_extent, job.k, parts, c->n_cu);
    const CheckArgs ca{job.src,  job.n, job.tgt, job.m, job.rot, job.k, kSrcCoordLimit,
                       ref_coord_limit(p), bad};
    DSES_HIP(launch_prepare(check_inputs ? &ca : nullptr,
                            stage_desc(g, a.gref, arrange, job.tgt, static_cast<int32_t *>(d_perm),
                                       static_cast<int32_t *>(d_yq), static_cast<float *>(d_yt)),
                            stream));
    rec_ev(1);
    if (job.exhaustive) {
        DSES_HIP(launch_exhaustive(a, scorer, grid, stream));
    } else if (o.q > 0.0f) {
        uint32_t *pw = static_cast<uint32_t *>(c->prune.ptr);
        DSES_HIP(launch_sweep(a, kScoreNone, grid, stream));
        DSES_HIP(launch_score_pruned(a, scorer, o.q, pw, pw + 1, grid, stream));
    } else if (parts > 1) {
        DSES_HIP(launch_sweep_parts(a, scorer, grid, c->modes.ptr, parts, stream));
    } else {
        DSES_HIP(launch_sweep(a, scorer, grid, stream));
    }
    rec_ev(2);
    // the result goes to pinned host memory by the kernel's own stores
    DSES_HIP(launch_select(a.rec, job.k, job.rot, p.delta, c->host_res, bad, stream));
    rec_ev(3);
    // Records for a buffer of this device are copied by a kernel that looks at the
    // selection's outcome, so that they need no second wait; other buffers by the runtime,
    // once the outcome is known.
    bool publish = false;
    if (records && on_device && records != (void *)a.rec &&
        reinterpret_cast<uintptr_t>(records) % alignof(dses_record) == 0) {
        hipPointerAttribute_t at{};
        publish = hipPointerGetAttributes(&at, records) == hipSuccess &&
                  at.type == hipMemoryTypeDevice && at.device == c->device;
        if (!publish) (void)hipGetLastError();
    }
    if (publish) DSES_HIP(launch_publish(a.rec, records, job.k, bad, stream));
    // given back while the device works (a grid of 4 million cells: 7.18 / 6.90 ms a call)
    hg.pts = std::vector<float>();
    hg.start = std::vector<int32_t>();
    DSES_HIP(hipStreamSynchronize(stream));
    device.end();
    const DevResult r = *c->host_res;
    if (timing) {
        float t01 = 0, t12 = 0, t23 = 0;
        (void)hipEventElapsedTime(&t01, ev[0], ev[1]);
        (void)hipEventElapsedTime(&t12, ev[1], ev[2]);
        (void)hipEventElapsedTime(&t23, ev[2], ev[3]);
        for (auto &e : ev) (void)hipEventDestroy(e);
        const int64_t pairs = (int64_t)job.n * job.m * job.k;
        add_stats(c, t12, 0.0, t23, t01, 1, pairs, scorer == DSES_SCORER_BRUTE ? pairs : 0, job.k);
    }
    if (r.bad_input) {
        set_error("non-finite or out-of-range coordinate, or non-orthonormal rotation");
        return DSES_E_INVAL;
    }
    if (r.rot_index < 0) {
        set_error("no rotation received a vote inside the translation box");
        return DSES_E_NOCANDIDATE;
    }
    const bool copy_records = records && records != (void *)a.rec && !publish;
    if (copy_records) {
        DSES_HIP(hipMemcpyAsync(records, a.rec, (size_t)job.k * sizeof(dses_record),
                                on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost,
                                stream));
    }
    if (o.top_k > 0) {
        const size_t sb = topk_scratch_bytes(job.k, o.top_k);
        if ((st = c->topk_a.ensure(sb)) != DSES_OK) return st;
        if ((st = c->topk_b.ensure(sb)) != DSES_OK) return st;
        if ((st = c->topk_out.ensure(DSES_TOPK_MAX * sizeof(dses_candidate))) != DSES_OK) return st;
        auto *dst = on_device ? static_cast<dses_candidate *>(o.topk)
                              : static_cast<dses_candidate *>(c->topk_out.ptr);
        DSES_HIP(launch_topk(a.rec, job.k, o.top_k, p.delta, c->topk_a.ptr, c->topk_b.ptr, dst,
                             stream));
        if (!on_device)
            DSES_HIP(hipMemcpyAsync(o.topk, dst, (size_t)o.top_k * sizeof(dses_candidate),
                                    hipMemcpyDeviceToHost, stream));
    }
    if (copy_records || o.top_k > 0) DSES_HIP(hipStreamSynchronize(stream));
    if (out) {
        std::memcpy(out->R, r.R, sizeof(out->R));
        std::memcpy(out->t, r.t, sizeof(out->t));
        out->rot_index = r.rot_index;
        out->inliers = r.inliers;
        out->error = r.error;
        out->votes = r.votes;
        out->n_valid = r.n_valid;
    }
    return DSES_OK;
}

}  // namespace dses

using namespace dses;

extern "C" {

const char *dses_last_error(void) { return g_err.c_str(); }

const char *dses_version(void) { return "dses-mi355x 0.1"; }

dses_status dses_init(int32_t device) { return init_device(device); }

dses_status dses_debug_fail_allocs(int32_t skip, int32_t count)
{
    if (skip < 0 || count < 0) {
        set_error("dses_debug_fail_allocs: negative argument");
        return DSES_E_INVAL;
    }
    std::lock_guard<std::mutex> lk(g_fault_mu);
    g_fault_skip = count > 0 ? skip : 0;
    g_fault_count = count;
    return DSES_OK;
}

dses_status dses_kernel_stats(dses_kstats *out, int32_t reset)
{
    Context *c = ctx();
    if (!c) return DSES_E_DEVICE;
    std::lock_guard<std::mutex> lk(c->stats_mu);
    if (out) *out = c->stats;
    if (reset) c->stats = dses_kstats{};
    return DSES_OK;
}

dses_status dses_register(const float *src, int64_t n, const float *tgt, int64_t m,
                          const float *rotations, int64_t k, float eps, dses_metric metric,
                          const dses_options *opt, dses_result *out)
{
    set_error("");
    if (!src || !tgt || !rotations || !out) {
        set_error("NULL pointer argument");
        return DSES_E_INVAL;
    }
    if (n <= 0 || m <= 0 || k <= 0 || k > INT32_MAX || n * m >= ((int64_t)1 << 31)) {
        set_error("n, m, k must be positive with n*m < 2^31 and k < 2^31");
        return DSES_E_INVAL;
    }
    dses_options o;
    if (copy_options(opt, &o) != DSES_OK) return DSES_E_INVAL;
    if (o.top_k < 0 || o.top_k > DSES_TOPK_MAX || (o.top_k > 0 && !o.topk) ||
        !(o.q >= 0.0f && o.q <= 1.0f)) {
        set_error("top_k must be in 0..DSES_TOPK_MAX with a topk buffer, q in [0, 1]");
        return DSES_E_INVAL;
    }
    Params p;
    dses_status st = resolve_params(eps, metric, o.delta_t, o.tau, o.t_min, o.t_max, o.scorer, &p);
    if (st != DSES_OK) return st;
    if ((st = apply_metric_options(o, &p)) != DSES_OK) return st;
    if (p.scorer == DSES_SCORER_DF && p.metric != DSES_VOTES) {
        set_error("the DF scorer needs a resident target (dses_register_resident)");
        return DSES_E_INVAL;
    }
    const bool dev = (o.flags & DSES_DEVICE_PTRS) != 0;
    if (!dev) {
        st = check_host_inputs(src, n, tgt, m, rotations, k, ref_coord_limit(p));
        if (st != DSES_OK) return st;
    }
    Context *c = ctx();
    if (!c) return DSES_E_DEVICE;
    std::lock_guard<std::mutex> lk(c->mu);
    c->timing_enabled = (o.flags & DSES_TIMING) != 0;
    hipStream_t stream = o.stream ? static_cast<hipStream_t>(o.stream) : c->stream;
    Job job;
    job.n = (int32_t)n;
    job.m = (int32_t)m;
    job.k = (int32_t)k;
    job.p = p;
    if (dev) {
        job.src = src;
        job.tgt = tgt;
        job.rot = rotations;
    } else {
        if ((st = c->in_src.ensure(3 * n * sizeof(float))) != DSES_OK) return st;
        if ((st = c->in_tgt.ensure(3 * m * sizeof(float))) != DSES_OK) return st;
        if ((st = c->in_rot.ensure(9 * k * sizeof(float))) != DSES_OK) return st;
        DSES_HIP(hipMemcpyAsync(c->in_src.ptr, src, 3 * n * sizeof(float), hipMemcpyHostToDevice,
                                stream));
        DSES_HIP(hipMemcpyAsync(c->in_tgt.ptr, tgt, 3 * m * sizeof(float), hipMemcpyHostToDevice,
                                stream));
        DSES_HIP(hipMemcpyAsync(c->in_rot.ptr, rotations, 9 * k * sizeof(float),
                                hipMemcpyHostToDevice, stream));
        job.src = static_cast<float *>(c->in_src.ptr);
        job.tgt = static_cast<float *>(c->in_tgt.ptr);
        job.rot = static_cast<float *>(c->in_rot.ptr);
        job.host_tgt = tgt;
    }
    return run_plain(c, job, stream, dev, out, o);
}

dses_status dses_register_exhaustive(const float *src, int64_t n, const float *tgt, int64_t m,
                                     const float *rotations, int64_t k, float eps,
                                     dses_metric metric, const dses_options *opt,
                                     dses_result *out)
{
    set_error("");
    if (!src || !tgt || !rotations || !out) {
        set_error("NULL pointer argument");
        return DSES_E_INVAL;
    }
    if (n <= 0 || m <= 0 || k <= 0 || k > INT32_MAX || n * m >= ((int64_t)1 << 31) ||
        n > kExhaustiveMaxSrc) {
        set_error("n, m, k must be positive with n*m < 2^31 and n <= 12288");
        return DSES_E_INVAL;
    }
    dses_options o;
    if (copy_options(opt, &o) != DSES_OK) return DSES_E_INVAL;
    if (o.top_k != 0 || o.q != 0.0f) {
        set_error("top_k and q are not options of the exhaustive search");
        return DSES_E_INVAL;
    }
    Params p;
    dses_status st = resolve_params(eps, metric, o.delta_t, o.tau, o.t_min, o.t_max, o.scorer, &p);
    if (st != DSES_OK) return st;
    if ((st = apply_metric_options(o, &p)) != DSES_OK) return st;
    if (p.metric == DSES_VOTES || p.scorer == DSES_SCORER_DF) {
        set_error("the exhaustive search scores with BRUTE or GRID and a robust metric");
        return DSES_E_INVAL;
    }
    if ((int64_t)p.size[0] * p.size[1] * p.size[2] > INT32_MAX) {
        set_error("the exhaustive search takes at most 2^31 - 1 translations per rotation");
        return DSES_E_INVAL;
    }
    const bool dev = (o.flags & DSES_DEVICE_PTRS) != 0;
    if (!dev) {
        st = check_host_inputs(src, n, tgt, m, rotations, k, ref_coord_limit(p));
        if (st != DSES_OK) return st;
    }
    Context *c = ctx();
    if (!c) return DSES_E_DEVICE;
    std::lock_guard<std::mutex> lk(c->mu);
    c->timing_enabled = (o.flags & DSES_TIMING) != 0;
    hipStream_t stream = o.stream ? static_cast<hipStream_t>(o.stream) : c->stream;
    Job job;
    job.n = (int32_t)n;
    job.m = (int32_t)m;
    job.k = (int32_t)k;
    job.p = p;
    job.exhaustive = true;
    if (dev) {
        job.src = src;
        job.tgt = tgt;
        job.rot = rotations;
    } else {
        if ((st = c->in_src.ensure(3 * n * sizeof(float))) != DSES_OK) return st;
        if ((st = c->in_tgt.ensure(3 * m * sizeof(float))) != DSES_OK) return st;
        if ((st = c->in_rot.ensure(9 * k * sizeof(float))) != DSES_OK) return st;
        DSES_HIP(hipMemcpyAsync(c->in_src.ptr, src, 3 * n * sizeof(float), hipMemcpyHostToDevice,
                                stream));
        DSES_HIP(hipMemcpyAsync(c->in_tgt.ptr, tgt, 3 * m * sizeof(float), hipMemcpyHostToDevice,
                                stream));
        DSES_HIP(hipMemcpyAsync(c->in_rot.ptr, rotations, 9 * k * sizeof(float),
                                hipMemcpyHostToDevice, stream));
        job.src = static_cast<float *>(c->in_src.ptr);
        job.tgt = static_cast<float *>(c->in_tgt.ptr);
        job.rot = static_cast<float *>(c->in_rot.ptr);
        job.host_tgt = tgt;
    }
    return run_plain(c, job, stream, dev, out, o);
}

}  // extern "C"
