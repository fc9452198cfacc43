// Which layout the library picks for a plain call or a batch of one problem: its own
// host rules, called directly.
#include "host.h"

#include <chrono>

using namespace dses;

// box: translations in [-box, box]^3; out: counter bits, wide, nslabs, pps, sorted, gref,
// group, windows, arrange, parts.
extern "C" int route(const float *tgt, int m, int n, int k, float eps, float box, int lane_group,
                     int batched, int32_t *out)
{
    Params p;
    const float lo[3] = {-box, -box, -box}, hi[3] = {box, box, box};
    dses_status st = resolve_params(eps, DSES_TRUNC_L2, 0.0f, 0.0f, lo, hi, DSES_SCORER_AUTO, &p);
    if (st != DSES_OK) return st;
    Geom g;
    const int64_t population = ref_block_population(tgt, m, p);
    const int bits = counter_bits_for(population * n, n, m, p);
    if ((st = plan_geom(nullptr, p, n, m, bits, &g)) != DSES_OK) return st;
    std::vector<int32_t> perm;
    sort_by_x(tgt, m, &perm);
    int32_t ylo = 0, yhi = 0;
    const bool sorted = n <= kSortMax && ref_x_range(tgt, perm, p.delta, p.klo[0], &ylo, &yhi);
    const float x = ref_x_extent(ylo, yhi);
    VoteLayout l = choose_layout(g, sorted, x, population, lane_group, batched);
    double share = 1.0;
    int parts = l.gref && !batched ? choose_parts(g, k, x, 256, &share) : 1;
    if (l.general < (batched ? kBatchGeneral : share)) {
        l.gref = l.parts = 0;
        parts = 1;
    }
    const int32_t v[10] = {bits, g.wide, g.nslabs, g.pps, sorted, l.gref,
                           l.gref || !sorted ? 0 : l.group, l.parts,
                           worth_arranging(g, l.gref, x, k, parts, batched ? 1 : 256), parts};
    for (int i = 0; i < 10; ++i) out[i] = v[i];
    return DSES_OK;
}

// Least time in us, of many tries, of choose_parts over `slabs` slabs of three planes and of
// the order by x of an m-point reference.
extern "C" void parts_and_sort_us(const float *tgt, int m, int slabs, int k, double *parts,
                                  double *sort)
{
    Geom g{};
    g.n = 64;
    g.m = 256;
    g.pps = 3;
    g.size[0] = 3 * slabs;
    auto least = [](auto f) {
        double best = 1e30;
        for (int i = 0; i < 200; ++i) {
            const auto t = std::chrono::steady_clock::now();
            f();
            const std::chrono::duration<double, std::micro> d = std::chrono::steady_clock::now() - t;
            best = std::min(best, d.count());
        }
        return best;
    };
    int sum = 0;
    std::vector<int32_t> perm;
    double share;
    *parts = least([&] { sum += choose_parts(g, k, 100.0f, 256, &share); });
    *sort = least([&] { sort_by_x(tgt, m, &perm); });
}
