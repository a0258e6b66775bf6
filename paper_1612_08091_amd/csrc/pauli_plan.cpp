// Host plan of a Pauli sum: which strings one tile shape serves.
#include <algorithm>
#include <cstring>

#include "pauli.hpp"

namespace qsv {
namespace dev {

namespace {
inline int pc(uint64_t v) { return __builtin_popcountll(v); }
constexpr int kLow = 3;             // the lowest positions are in every tile: whole 128-byte lines
constexpr size_t kScored = 2048;    // masks that a choice of positions looks at, at most
constexpr unsigned kResident = 512; // workgroups the chip holds (two per CU, by LDS)

// Strings with one X mask and one parity of n_Y: order[first..first + count).
struct Strings {
    uint64_t x;
    int odd, first, count;
};

// Groups ascending by mask, then parity; the strings of each in their own order.
// (A table of the masks seen and a sort of the groups: most sums have many strings
// on few masks.)
std::vector<Strings> group_strings(int nterms, const uint64_t *x, const uint64_t *z,
                                   std::vector<int> &order) {
    int bits = 4;
    while ((2 << bits) < 4 * nterms && bits < 30) ++bits;
    std::vector<int> slot((size_t)2 << bits, -1), of(nterms);
    std::vector<Strings> found;
    for (int t = 0; t < nterms; ++t) {
        const int odd = pc(x[t] & z[t]) & 1;
        size_t at = (size_t)((x[t] + 1) * 0x9e3779b97f4a7c15ull >> (64 - bits)) * 2 + (size_t)odd;
        while (slot[at] >= 0 && found[slot[at]].x != x[t]) at = (at + 2) & (slot.size() - 1);
        if (slot[at] < 0) {
            slot[at] = (int)found.size();
            found.push_back({x[t], odd, 0, 0});
        }
        of[t] = slot[at];
        ++found[of[t]].count;
    }
    std::vector<int> by(found.size());
    for (size_t g = 0; g < by.size(); ++g) by[g] = (int)g;
    std::sort(by.begin(), by.end(), [&](int a, int b) {
        return found[a].x != found[b].x ? found[a].x < found[b].x : found[a].odd < found[b].odd;
    });
    std::vector<Strings> groups;
    std::vector<int> next(found.size());
    int first = 0;
    for (int g : by) {
        next[g] = found[g].first = first;
        first += found[g].count;
        groups.push_back(found[g]);
    }
    for (int t = 0; t < nterms; ++t) order[next[of[t]]++] = t;
    return groups;
}

// The groups that no tile serves yet, ascending by X mask.  Those taken stay in
// place until they are half of all, so that a tile's own are found by a walk that
// leaves out what a mask outside the tile begins with, and a sum of many masks is
// planned in little more than the time to sort it (60000 random strings on 20
// qubits: 60 ms, 1200 when every tile looked at every mask left).
struct Waiting {
    std::vector<int> at;            // group numbers
    std::vector<char> taken;        // by group number
    size_t alive = 0;
    const std::vector<Strings> &groups;

    explicit Waiting(const std::vector<Strings> &g) : taken(g.size(), 0), groups(g) {}
    void add(int g) {
        at.push_back(g);
        ++alive;
    }
    // the waiting groups of at[lo..hi) whose masks lie within `tile`; they agree on
    // the bits above `bit`, which lie in it
    void collect(size_t lo, size_t hi, int bit, uint64_t tile, std::vector<int> &out) const {
        while (bit >= 0 && hi - lo > 16) {
            // the masks with the bit clear come first
            const auto mid = std::partition_point(at.begin() + lo, at.begin() + hi, [&](int g) {
                return !((groups[g].x >> bit) & 1);
            }) - at.begin();
            if ((tile >> bit) & 1) {
                collect(lo, (size_t)mid, bit - 1, tile, out);
                lo = (size_t)mid;
            } else {
                hi = (size_t)mid;
            }
            --bit;
        }
        for (size_t i = lo; i < hi; ++i)
            if (!taken[at[i]] && !(groups[at[i]].x & ~tile)) out.push_back(at[i]);
    }
    void take(const std::vector<int> &in) {
        for (int g : in) taken[g] = 1;
        alive -= in.size();
        if (2 * alive > at.size()) return;
        at.erase(std::remove_if(at.begin(), at.end(), [&](int g) { return taken[g] != 0; }), at.end());
    }
};
}  // namespace

void pauli_plan(int nq, int nterms, const uint64_t *x, const uint64_t *z,
                const double *c, PauliPlan &p) {
    p = PauliPlan{};
    constexpr int rb = kPauliRegBits, m = kPauliTileBits, nr = 1 << rb;
    // strings by X mask and parity of n_Y
    std::vector<int> order(nterms);
    const std::vector<Strings> groups = group_strings(nterms, x, z, order);
    Waiting left(groups);
    const uint64_t low = (1ull << std::min(kLow, nq)) - 1;
    auto coef = [&](int t, bool pairs) {
        // i^{n_Y} times the pair's 2 Re (n_Y even) or 2 i Im (odd)
        static const double f[4] = {1.0, -1.0, -1.0, 1.0};
        return c[t] * f[pc(x[t] & z[t]) & 3] * (pairs ? 2.0 : 1.0);
    };
    for (size_t k = 0; k < groups.size(); ++k) {
        const Strings &g = groups[k];
        if (pc(g.x | low) <= m) {
            left.add((int)k);
            continue;
        }
        for (int f = 0; f < g.count; f += kPauliWide) {
            PauliWideGroup w{};
            w.x = g.x;
            w.hbit = 63 - __builtin_clzll(w.x);
            w.odd = g.odd;
            w.nt = std::min(kPauliWide, g.count - f);
            for (int j = 0; j < w.nt; ++j) {
                w.z[j] = z[order[g.first + f + j]];
                w.c[j] = coef(order[g.first + f + j], true);
            }
            p.wide.push_back(w);
        }
    }
    // Tile shapes, greedily: from the widest X mask left, add the position that
    // brings most of the other masks nearest to fitting (a mask that lacks k
    // positions counts 8^-k for each), until the tile is full.  Random strings
    // of weight <= 4 on 25 qubits, 111 distinct masks: 8 shapes of 12 bits, as
    // many as a search over pairs of masks finds.
    std::vector<int> widest = left.at, in;
    std::stable_sort(widest.begin(), widest.end(),
                     [&](int a, int b) { return pc(groups[a].x | low) > pc(groups[b].x | low); });
    for (int seed : widest) {
        if (left.taken[seed]) continue;
        uint64_t tile = low | groups[seed].x;
        while (pc(tile) < std::min(m, nq)) {
            double score[64] = {0.0};
            int best = -1;
            for (size_t i = 0; i < left.at.size(); i += 1 + left.at.size() / kScored) {
                if (left.taken[left.at[i]]) continue;
                const uint64_t miss = groups[left.at[i]].x & ~tile;
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
        in.clear();
        left.collect(0, left.at.size(), nq - 1, tile, in);
        left.take(in);
        int freq[64] = {0};
        for (int g : in)
            for (uint64_t b = groups[g].x; b; b &= b - 1) ++freq[__builtin_ctzll(b)];
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
        for (int k : in) {
            PauliXGroup g{};
            const uint32_t xl = local(groups[k].x);
            g.xthr = xl & tmask;
            g.xreg = xl >> kPauliThreadBits;
            g.odd = groups[k].odd;
            g.term0 = (int32_t)p.terms.size();
            g.terms = groups[k].count - 1;
            for (int j = 0; j < groups[k].count; ++j) {
                const int t = order[groups[k].first + j];
                PauliTerm q{};
                const uint32_t zl = local(z[t]);
                q.c = coef(t, g.xreg != 0);
                q.zo = z[t] & ~tile;
                q.zthr = zl & tmask;
                for (int i = 0; i < nr; ++i)
                    if (__builtin_popcount((uint32_t)i & (zl >> kPauliThreadBits)) & 1) q.sreg |= 1u << i;
                if (j == 0) g.first = q;
                else p.terms.push_back(q);
            }
            p.groups.push_back(g);
        }
        p.sets.push_back(s);
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
