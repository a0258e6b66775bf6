// The host model of the register kernel refuses table groups that the kernel, which
// ORs the parts of a table's offset, would read elsewhere: a table off its multiple,
// a part on the place of another.  The programs of a QFT as lowered pass.  Prints
// "ok" and returns 0.
#include <cmath>
#include <cstdio>
#include <string>
#include <vector>

#include "qsv_internal.hpp"
#include "tileprog.hpp"

using namespace qsv;

int main() {
    const int n = 18, m = 12, rb = 4;
    std::vector<Op> ops;
    auto add = [&](std::vector<cd> u, int t, uint64_t ctrl) {
        Gate g;
        g.k = 1;
        g.t[0] = t;
        g.ctrl = ctrl;
        g.U = std::move(u);
        Op o;
        if (canonicalize(g, o)) ops.push_back(o);
    };
    const double r = std::sqrt(0.5);
    for (int j = n - 1; j >= 0; --j) {
        add({r, r, r, -r}, j, 0);
        for (int k = j - 1; k >= 0; --k) add({1, 0, 0, std::polar(1.0, 3.14159 / (1 << (j - k)))}, j, 1ull << k);
    }
    int groups = 0, refused = 0;
    for (int elem : {16, 8})
        for (const Pass &ps : plan_tiled(ops, n, m, 2, 17, true)) {
            std::vector<double> mats;
            TileProgram pg;
            compile_pass(ps, rb, mats, pg, elem);
            auto model = [&](const TileProgram &p) {
                std::vector<cd> psi(1ull << n, cd(1, 0));
                return emulate_reg_pass(p, rb, mats, elem, n, psi);
            };
            const std::string err = model(pg);
            if (!err.empty()) {
                std::fprintf(stderr, "%s\n", err.c_str());
                return 1;
            }
            for (size_t i = 0; i < pg.rops.size(); ++i) {
                if (pg.rops[i].kind != dev::ROP_DGRP) continue;
                for (int k = 0; k < pg.rops[i].a; ++k) {
                    ++groups;
                    int at[6], parts = 0, free_lane = -1;
                    const uint32_t lane = pg.rops[i].dt[k].lane;
                    for (int t = 0; t < 6; ++t) {
                        if (((lane >> (4 * t)) & 15u) != 15u) at[parts++] = t;
                        else free_lane = t;
                    }
                    if (parts == 0) continue;
                    for (int plant = 0; plant < 2; ++plant) {
                        TileProgram bad = pg;
                        dev::DiagTab &d = bad.rops[i].dt[k];
                        const uint32_t first = (lane >> (4 * at[0])) & 15u;
                        if (plant == 0) {
                            d.off += (uint32_t)elem;
                        } else {
                            if (free_lane < 0) continue;
                            d.lane &= ~((15u ^ first) << (4 * free_lane));
                        }
                        if (model(bad).empty()) {
                            std::fprintf(stderr, "mistake %d in a table passed\n", plant);
                            return 1;
                        }
                        ++refused;
                    }
                }
            }
        }
    if (groups == 0 || refused == 0) {
        std::fprintf(stderr, "no table groups\n");
        return 1;
    }
    std::printf("ok (%d tables, %d mistakes refused)\n", groups, refused);
    return 0;
}
