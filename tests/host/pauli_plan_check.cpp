// The plan of a Pauli sum, evaluated on the host as the kernels do it and compared
// with the strings themselves on a random state; and the time that a plan takes,
// which has to grow with the number of strings, not with its square.  Prints "ok"
// and returns 0.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <complex>
#include <cstdio>
#include <random>
#include <vector>

#include "pauli.hpp"

using namespace qsv::dev;
using cd = std::complex<double>;

static double sign(uint64_t v) { return __builtin_popcountll(v) & 1 ? -1.0 : 1.0; }

static double direct(const std::vector<cd> &psi, uint64_t x, uint64_t z) {
    static const cd f[4] = {cd(1, 0), cd(0, 1), cd(-1, 0), cd(0, -1)};
    cd v = 0;
    for (uint64_t j = 0; j < psi.size(); ++j) v += std::conj(psi[j ^ x]) * psi[j] * sign(j & z);
    return (v * f[__builtin_popcountll(x & z) & 3]).real();
}

static double planned(const std::vector<cd> &psi, int nq, const PauliPlan &p) {
    double sum = 0.0;
    auto share = [](cd a, cd b, bool odd) { return odd ? (std::conj(b) * a).imag() : (std::conj(b) * a).real(); };
    for (const PauliSet &s : p.sets) {
        uint64_t tile = 0;
        for (int l = 0; l < kPauliTileBits; ++l)
            if (s.tpos[l] < 64) tile |= 1ull << s.tpos[l];
        auto place = [&](uint32_t l) {
            uint64_t v = 0;
            for (int b = 0; b < kPauliTileBits; ++b)
                if ((l >> b) & 1) v |= 1ull << s.tpos[b];
            return v;
        };
        const uint32_t pad = s.pad_thr | s.pad_reg << kPauliThreadBits;
        for (uint64_t base = 0; base < psi.size(); ++base) {
            if (base & tile) continue;
            for (int gi = s.group0; gi < s.group0 + s.groups; ++gi) {
                const PauliXGroup &g = p.groups[gi];
                const uint32_t xl = g.xthr | g.xreg << kPauliThreadBits;
                const int hb = g.xreg ? 31 - __builtin_clz(g.xreg) : -1;
                for (uint32_t l = 0; l < (1u << kPauliTileBits); ++l) {
                    const uint32_t thr = l & ((1u << kPauliThreadBits) - 1), reg = l >> kPauliThreadBits;
                    if ((l & pad) || (hb >= 0 && ((reg >> hb) & 1))) continue;
                    const double q = share(psi[base | place(l)], psi[base | place(l ^ xl)], g.odd);
                    for (int t = -1; t < g.terms; ++t) {
                        const PauliTerm &pt = t < 0 ? g.first : p.terms[g.term0 + t];
                        sum += q * pt.c * sign(base & pt.zo) * sign(thr & pt.zthr) * ((pt.sreg >> reg) & 1 ? -1.0 : 1.0);
                    }
                }
            }
        }
    }
    for (const PauliWideGroup &w : p.wide)
        for (uint64_t j = 0; j < psi.size(); ++j) {
            if ((j >> w.hbit) & 1) continue;
            for (int t = 0; t < w.nt; ++t)
                sum += w.c[t] * sign(j & w.z[t]) * share(psi[j], psi[j ^ w.x], w.odd);
        }
    (void)nq;
    return sum;
}

static double plan_ms(int nq, int terms, std::mt19937_64 &g) {
    std::vector<uint64_t> x(terms), z(terms);
    std::vector<double> c(terms, 1.0);
    for (auto &v : x) v = g() & ((1ull << nq) - 1);
    for (auto &v : z) v = g() & ((1ull << nq) - 1);
    double best = 1e30;
    for (int r = 0; r < 3; ++r) {
        PauliPlan p;
        const auto a = std::chrono::steady_clock::now();
        pauli_plan(nq, terms, x.data(), z.data(), c.data(), p);
        best = std::min(best, std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - a).count());
        size_t n = p.terms.size() + p.groups.size();
        for (const PauliWideGroup &w : p.wide) n += w.nt;
        if (n != (size_t)terms) {
            std::fprintf(stderr, "%zu of %d strings planned\n", n, terms);
            std::exit(1);
        }
    }
    return best;
}

int main() {
    std::mt19937_64 g(5);
    std::normal_distribution<double> N;
    for (int nq : {0, 1, 3, 9, 12, 13, 14})
        for (int terms : {1, 2, 40, 300})
            for (int kind = 0; kind < 4; ++kind) {
                if (nq == 14 && terms == 300 && kind == 1) continue;    // quick enough without
                const uint64_t full = (1ull << nq) - 1;
                std::vector<cd> psi(1ull << nq);
                double norm = 0;
                for (auto &v : psi) {
                    v = cd(N(g), N(g));
                    norm += std::norm(v);
                }
                for (auto &v : psi) v /= std::sqrt(norm);
                std::vector<uint64_t> x(terms), z(terms);
                std::vector<double> c(terms);
                double want = 0.0, scale = 0.0;
                for (int t = 0; t < terms; ++t) {
                    x[t] = kind == 0 ? g() & g() & full : kind == 1 ? g() & full : kind == 2 ? g() & 3 & full : full >> (g() % 4);
                    z[t] = g() & full;
                    c[t] = N(g);
                    want += c[t] * direct(psi, x[t], z[t]);
                    scale += std::fabs(c[t]);
                }
                PauliPlan p;
                pauli_plan(nq, terms, x.data(), z.data(), c.data(), p);
                const double got = planned(psi, nq, p);
                if (!(std::fabs(got - want) <= 1e-12 * scale)) {
                    std::fprintf(stderr, "%d qubits, %d strings, kind %d: %.15g, not %.15g\n", nq, terms, kind, got, want);
                    return 1;
                }
            }
    // four times the strings: 16 times as long if every tile looks at every mask
    const double small = plan_ms(24, 20000, g), large = plan_ms(24, 80000, g);
    if (large > 8.0 * small) {
        std::fprintf(stderr, "20000 strings %.1f ms, 80000 strings %.1f ms\n", small, large);
        return 1;
    }
    std::printf("ok (20000 strings %.1f ms, 80000 strings %.1f ms; 60000 on 20 qubits %.1f ms)\n", small, large,
                plan_ms(20, 60000, g));
    return 0;
}
