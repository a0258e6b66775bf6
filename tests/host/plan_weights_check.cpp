// The weights that candidate plans are compared by are those of their fused ops (1
// for one that mixes, a quarter for a diagonal one) as the plan that is kept builds
// them, among them gates that cancel or leave a phase.  Prints "ok" and returns 0.
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "qsv_internal.hpp"

using namespace qsv;

int main() {
    std::mt19937_64 g(3);
    int compared = 0, whole = 0;
    for (int trial = 0; trial < 30; ++trial) {
        const int n = 13 + trial % 8, m = 12 - trial % 2;
        std::vector<Op> ops;
        auto add = [&](std::vector<cd> u, std::vector<int> t, uint64_t ctrl = 0) {
            Gate ga;
            ga.k = (int)t.size();
            for (int j = 0; j < ga.k; ++j) ga.t[j] = t[j];
            ga.ctrl = ctrl;
            ga.U = std::move(u);
            Op o;
            if (canonicalize(ga, o)) ops.push_back(o);
        };
        const double r = std::sqrt(0.5);
        const std::vector<cd> h = {r, r, r, -r}, x = {0, 1, 1, 0}, s = {1, 0, 0, cd(0, 1)},
                              ry = {0.8, -0.6, 0.6, 0.8};
        for (int i = 0; i < 150; ++i) {
            const int a = (int)(g() % n), b = (int)((a + 1 + g() % (n - 1)) % n), c = (int)(g() % n);
            switch (g() % (trial % 3 == 0 ? 4 : 6)) {
            case 0: add(x, {b}, 1ull << a); break;
            case 1: add(s, {a}); break;
            case 2:     // cancels, or leaves a phase, once the gates between have moved
                add(x, {b}, 1ull << a);
                if (c != a && c != b) add(s, {c});
                if (g() % 2) add(s, {b});
                add(x, {b}, 1ull << a);
                break;
            case 3: add(h, {a}); break;
            case 4: add(ry, {a}); break;
            default: add(s, {b}, 1ull << a); break;
            }
        }
        for (int k_max : {1, 2, 3})
            for (int setting = 0; setting < 8; ++setting) {
                auto plan = [&](std::vector<double> *weights) {
                    static const int caps[] = {2, 4, 8}, op_caps[] = {1 << 30, 32};
                    return setting == 0 ? plan_passes(ops, n, m, 3, k_max, kMaxK, weights)
                           : setting == 7
                               ? plan_passes_relabel(ops, n, m, 3, k_max, kMaxK, 17, 8, 40, weights)
                               : plan_passes_relabel(ops, n, m, 3, k_max, kMaxK, 9, caps[setting % 3],
                                                     op_caps[setting % 2], weights);
                };
                std::vector<double> weights;
                const std::vector<Pass> light = plan(&weights), full = plan(nullptr);
                if (light.size() != full.size() || weights.size() != full.size()) {
                    std::fprintf(stderr, "trial %d: %zu, %zu, %zu passes\n", trial, light.size(), full.size(),
                                 weights.size());
                    return 1;
                }
                for (size_t p = 0; p < full.size(); ++p) {
                    double w = 0.0;
                    for (const Op &o : full[p].ops) w += o.mixing() ? 1.0 : 0.25;
                    ++compared;
                    if (light[p].tile != full[p].tile || std::fabs(w - weights[p]) > 1e-9) {
                        std::fprintf(stderr, "trial %d k_max %d setting %d pass %zu: %g, not %g\n", trial, k_max,
                                     setting, p, weights[p], w);
                        return 1;
                    }
                    whole += !full[p].ops.empty();
                }
            }
    }
    std::printf("ok (%d passes, %d with ops)\n", compared, whole);
    return 0;
}
