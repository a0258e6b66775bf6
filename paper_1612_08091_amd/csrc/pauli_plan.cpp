// Host plan of a Pauli sum: which strings one tile shape serves.
#include <algorithm>
#include <cstring>
#include <map>

#include "pauli.hpp"

namespace qsv {
namespace dev {

namespace {
inline int pc(uint64_t v) { return __builtin_popcountll(v); }
constexpr int kLow = 3;             // the lowest positions are in every tile: whole 128-byte lines
constexpr size_t kScored = 2048;    // masks that a choice of positions looks at, at most
constexpr unsigned kResident = 512; // workgroups the chip holds (two per CU, by LDS)
}  // namespace

void pauli_plan(int nq, int nterms, const uint64_t *x, const uint64_t *z,
                const double *c, PauliPlan &p) {
    p = PauliPlan{};
    constexpr int rb = kPauliRegBits, m = kPauliTileBits, nr = 1 << rb;
    // strings by X mask and parity of n_Y
    std::map<std::pair<uint64_t, int>, std::vector<int>> by;
    for (int t = 0; t < nterms; ++t) by[{x[t], pc(x[t] & z[t]) & 1}].push_back(t);
    std::vector<std::pair<uint64_t, int>> left;
    const uint64_t low = (1ull << std::min(kLow, nq)) - 1;
    auto coef = [&](int t, bool pairs) {
        // i^{n_Y} times the pair's 2 Re (n_Y even) or 2 i Im (odd)
        static const double f[4] = {1.0, -1.0, -1.0, 1.0};
        return c[t] * f[pc(x[t] & z[t]) & 3] * (pairs ? 2.0 : 1.0);
    };
    for (const auto &g : by) {
        if (pc(g.first.first | low) <= m) {
            left.push_back(g.first);
            continue;
        }
        for (size_t f = 0; f < g.second.size(); f += kPauliWide) {
            PauliWideGroup w{};
            w.x = g.first.first;
            w.hbit = 63 - __builtin_clzll(w.x);
            w.odd = g.first.second;
            w.nt = (int32_t)std::min<size_t>(kPauliWide, g.second.size() - f);
            for (int k = 0; k < w.nt; ++k) {
                w.z[k] = z[g.second[f + k]];
                w.c[k] = coef(g.second[f + k], true);
            }
            p.wide.push_back(w);
        }
    }
    // Tile shapes, greedily: from the widest X mask left, add the position that
    // brings most of the other masks nearest to fitting (a mask that lacks k
    // positions counts 8^-k for each), until the tile is full.  Random strings
    // of weight <= 4 on 25 qubits, 111 distinct masks: 8 shapes of 12 bits, as
    // many as a search over pairs of masks finds.
    while (!left.empty()) {
        uint64_t tile = low, seed = 0;
        for (const auto &g : left)
            if (pc(g.first | low) > pc(seed | low)) seed = g.first;
        tile |= seed;
        while (pc(tile) < std::min(m, nq)) {
            double score[64] = {0.0};
            int best = -1;
            for (size_t i = 0; i < left.size(); i += 1 + left.size() / kScored) {
                const uint64_t miss = left[i].first & ~tile;
                const int k = pc(miss);
                if (k == 0 || k > m - pc(tile)) continue;
                double w = 1.0;
                for (int j = 0; j < k; ++j) w *= 0.125;
                for (uint64_t b = miss; b; b &= b - 1) score[__builtin_ctzll(b)] += w;
            }
            for (int q = 0; q < nq; ++q)
                if (score[q] > 0.0 && (best < 0 || score[q] > score[best])) best = q;
            if (best < 0) break;
            tile |= 1ull << best;
        }
        for (int q = 0; q < nq && pc(tile) < m; ++q) tile |= 1ull << q;
        // register bits: the positions above the lowest that most of the masks
        // served hold (a mask with a register bit needs half the pairs)
        std::vector<std::pair<uint64_t, int>> in, out;
        int freq[64] = {0};
        for (const auto &g : left) {
            if (g.first & ~tile) {
                out.push_back(g);
                continue;
            }
            in.push_back(g);
            for (int q = 0; q < nq; ++q) freq[q] += (int)((g.first >> q) & 1);
        }
        uint64_t regs = 0;
        for (int r = 0; r < rb; ++r) {
            int best = -1;
            for (int q = nq - 1; q >= 0; --q)
                if (((tile & ~low & ~regs) >> q) & 1)
                    if (best < 0 || freq[q] > freq[best]) best = q;
            if (best >= 0) regs |= 1ull << best;
        }
        PauliSet s{};
        int loc[64], nt = 0, nrg = 0;
        std::fill(loc, loc + 64, -1);
        std::fill(s.tpos, s.tpos + 16, kPauliNoPos);
        for (int q = 0; q < nq; ++q) {
            if (!((tile >> q) & 1)) continue;
            const bool reg = ((regs >> q) & 1) || nt == kPauliThreadBits;
            loc[q] = reg ? kPauliThreadBits + nrg++ : nt++;
            s.tpos[loc[q]] = (uint32_t)q;
            s.ins[s.n_ins++] = (uint32_t)q;
        }
        for (int b = nt; b < kPauliThreadBits; ++b) s.pad_thr |= 1u << b;
        for (int b = nrg; b < rb; ++b) s.pad_reg |= 1u << b;
        auto local = [&](uint64_t v) {
            uint32_t l = 0;
            for (uint64_t b = v & tile; b; b &= b - 1) l |= 1u << loc[__builtin_ctzll(b)];
            return l;
        };
        s.group0 = (int32_t)p.groups.size();
        s.groups = (int32_t)in.size();
        const uint32_t tmask = (1u << kPauliThreadBits) - 1;
        for (const auto &key : in) {
            PauliXGroup g{};
            const uint32_t xl = local(key.first);
            g.xthr = xl & tmask;
            g.xreg = xl >> kPauliThreadBits;
            g.odd = key.second;
            g.term0 = (int32_t)p.terms.size();
            const std::vector<int> &ts = by[key];
            g.terms = (int32_t)ts.size() - 1;
            for (int t : ts) {
                PauliTerm q{};
                const uint32_t zl = local(z[t]);
                q.c = coef(t, g.xreg != 0);
                q.zo = z[t] & ~tile;
                q.zthr = zl & tmask;
                for (int i = 0; i < nr; ++i)
                    if (__builtin_popcount((uint32_t)i & (zl >> kPauliThreadBits)) & 1) q.sreg |= 1u << i;
                if (t == ts.front()) g.first = q;
                else p.terms.push_back(q);
            }
            p.groups.push_back(g);
        }
        p.sets.push_back(s);
        left.swap(out);
    }
    // A small state has few tiles: its groups are shared out over more rows,
    // each reading the tiles again from the cache.  A large one has a few
    // workgroups per CU and set, each with many tiles.
    const uint64_t ntiles = nq > m ? 1ull << (nq - m) : 1;
    if (!p.sets.empty()) {
        const uint64_t share = kResident / ntiles / p.sets.size();
        if (share > 1) {
            std::vector<PauliSet> rows;
            for (const PauliSet &s : p.sets) {
                const int64_t parts = (int64_t)std::min<uint64_t>(share, (uint64_t)s.groups);
                for (int64_t k = 0; k < parts; ++k) {
                    PauliSet r = s;
                    r.group0 = s.group0 + (int)(s.groups * k / parts);
                    r.groups = s.group0 + (int)(s.groups * (k + 1) / parts) - r.group0;
                    rows.push_back(r);
                }
            }
            p.sets.swap(rows);
        }
        p.grid_x = (unsigned)std::min<uint64_t>(ntiles, std::max<uint64_t>(64, 4 * kResident / p.sets.size()));
    }
    if (!p.wide.empty()) {
        const uint64_t work = ((1ull << nq) / 2 + 255) / 256;
        p.wide_x = (unsigned)std::min<uint64_t>(work, std::max<uint64_t>(64, std::min<uint64_t>(512, 8192 / p.wide.size())));
    }
}

size_t pauli_blob_bytes(const PauliPlan &p) {
    return p.sets.size() * sizeof(PauliSet) + p.groups.size() * sizeof(PauliXGroup) +
           p.terms.size() * sizeof(PauliTerm) + p.wide.size() * sizeof(PauliWideGroup);
}

void pauli_blob(const PauliPlan &p, unsigned char *out) {
    auto put = [&](const void *d, size_t n) {
        if (n) std::memcpy(out, d, n);
        out += n;
    };
    put(p.groups.data(), p.groups.size() * sizeof(PauliXGroup));    // on their lines
    put(p.wide.data(), p.wide.size() * sizeof(PauliWideGroup));
    put(p.sets.data(), p.sets.size() * sizeof(PauliSet));
    put(p.terms.data(), p.terms.size() * sizeof(PauliTerm));
}

}  // namespace dev
}  // namespace qsv
