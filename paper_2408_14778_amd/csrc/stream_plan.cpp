// The stream of an out-of-core iteration: see stream_plan.hpp.
#include "stream_plan.hpp"

#include <algorithm>
#include <cstring>

namespace cfr {

namespace {

// The first level in cut .. D whose largest subtree has at most kStreamMax nodes.
int32_t second_cut(const Layout& L, int32_t cut) {
    std::vector<int32_t> size(L.N, 1);
    for (int64_t v = L.N - 1; v >= L.level_offset[cut + 1]; --v) size[L.parent[v]] += size[v];
    int32_t l = cut;
    for (; l < L.D; ++l) {
        const auto a = size.begin() + L.level_offset[l], b = size.begin() + L.level_offset[l + 1];
        if (*std::max_element(a, b) <= kStreamMax) break;
    }
    return l;
}

// Partition p's nodes by local id (level-cut nodes have their canonical ids).
struct Window {
    const Layout& L;
    const PartPlan& P;
    int32_t p;
    int64_t at(int64_t v) const { return P.off[p] + (v - P.base); }
    bool cut(int64_t v) const { return v < P.base; }
    int32_t player(int64_t v) const { return cut(v) ? L.node_player[v] : P.player[at(v)]; }
    // first child of node v (or of the end of a range) of level l
    int32_t child(int64_t v, int32_t l) const {
        return l == P.cut ? P.patch[P.patch_off[p] + (v - P.a[p])] : P.child_begin[at(v) + p];
    }
    int32_t code(int64_t v) const {
        const int32_t who = player(v), h = cut(v) ? L.node_infoset[v] : P.infoset[at(v)];
        return who < 0 ? -1 : who > 0 ? h : static_cast<int32_t>(L.Hp) + h;
    }
    double payoff(int64_t v) const {
        if (!cut(v)) return P.value0[at(v)];
        if (L.node_player[v] >= 0) return 0.0;
        return L.payoff64.empty() ? static_cast<double>(L.payoff[v]) : L.payoff64[v];
    }
    // nodes of level l: [first(l), first(l) + count(l))
    int32_t first(int32_t l) const {
        return l == P.cut ? P.a[p] : P.lo[static_cast<size_t>(p) * (P.D - P.cut + 1) + (l - P.cut - 1)];
    }
    int32_t count(int32_t l) const {
        if (l == P.cut) return P.b[p] - P.a[p];
        const size_t i = static_cast<size_t>(p) * (P.D - P.cut + 1) + (l - P.cut - 1);
        return P.lo[i + 1] - P.lo[i];
    }
};

template <class W, class F>
W word_of(F pay) {
    W w;
    static_assert(sizeof(W) == sizeof(F));
    std::memcpy(&w, &pay, sizeof w);
    return w;
}

int64_t pad_part(int64_t n) { return (n + kStreamPart - 1) / kStreamPart * kStreamPart; }

// Words of W bytes that the bits of n nodes take.
int64_t bit_words(int64_t n, int64_t W) { return pad_part(((n + 31) / 32 * 4 + W - 1) / W); }

// Appends a run: its bits and records, breadth first from the roots [x, y) of level l.
template <class W, class F>
void append_unit(const Window& V, int64_t x, int64_t y, int32_t l, std::vector<W>& out,
                 const StreamUnit& u) {
    const int64_t head = bit_words(u.n, sizeof(W));
    out.resize(u.at + head + pad_part(u.n), W{0});
    std::vector<uint32_t> bits((u.n + 31) / 32, 0);
    W* rec = out.data() + u.at + head;
    int64_t i = 0;
    while (x < y) {
        for (int64_t v = x; v < y; ++v, ++i) {
            const int32_t code = V.code(v);
            if (code >= 0) {
                bits[i / 32] |= 1u << (i % 32);
                rec[i] = static_cast<W>(code);
            } else {
                rec[i] = word_of<W, F>(static_cast<F>(V.payoff(v)));
            }
        }
        const int64_t cx = V.child(x, l), cy = V.child(y, l);
        x = cx;
        y = cy;
        ++l;
    }
    std::memcpy(out.data() + u.at, bits.data(), bits.size() * sizeof(uint32_t));
}

}  // namespace

void plan_stream(const Layout& L, const PartPlan& P, bool f64, StreamPlan& S, bool sizes_only) {
    S = StreamPlan{};
    S.cut = P.cut;
    S.base = P.base;
    S.split = second_cut(L, P.cut);
    const int32_t cut = P.cut, split = S.split, nl = split - cut + 1;
    S.unit0.push_back(0);
    for (int32_t p0 = 0; p0 < P.parts;) {
        // consecutive partitions while their nodes between the cuts fit one window
        std::vector<int64_t> n(nl, 0);
        int64_t mid = 0;
        int32_t p1 = p0;
        for (; p1 < P.parts; ++p1) {
            const Window V{L, P, p1};
            int64_t more = 0;
            for (int32_t l = cut + 1; l <= split; ++l) more += V.count(l);
            if (p1 > p0 && mid + more > P.window) break;
            mid += more;
            for (int32_t l = cut; l <= split; ++l) n[l - cut] += V.count(l);
        }
        S.window = std::max(S.window, mid);
        std::vector<int64_t> first(nl);
        int64_t id = P.base, rec = S.mid;
        for (int32_t l = cut; l <= split; ++l) {
            first[l - cut] = l == cut ? P.a[p0] : id;
            if (l > cut) id += n[l - cut];
            S.id.push_back(static_cast<int32_t>(first[l - cut]));
            S.count.push_back(static_cast<int32_t>(n[l - cut]));
            S.rec.push_back(rec);
            if (l < split) rec += n[l - cut];
        }
        S.mid = rec;
        for (int32_t l = cut; l < split && !sizes_only; ++l) {
            int64_t before = first[l + 1 - cut];  // local id of the partition's first node a level down
            for (int32_t p = p0; p < p1; ++p) {
                const Window V{L, P, p};
                const int64_t x = V.first(l), y = x + V.count(l);
                for (int64_t v = x; v < y; ++v) {
                    S.mid_code.push_back(V.code(v));
                    S.mid_child.push_back(static_cast<int32_t>(before + (V.child(v, l) - V.first(l + 1))));
                    S.mid_pay.push_back(V.payoff(v));
                }
                before += V.count(l + 1);
            }
        }
        // runs of consecutive subtrees of the second cut
        int64_t local = first[split - cut];
        for (int32_t p = p0; p < p1; ++p) {
            const Window V{L, P, p};
            const int64_t end = V.first(split) + int64_t{V.count(split)};
            StreamUnit u;
            int64_t from = V.first(split);
            auto close = [&](int64_t to) {
                if (u.n == 0) return;
                u.roots = static_cast<int32_t>(to - from);
                u.id0 = static_cast<int32_t>(local);
                local += u.roots;
                S.max_unit = std::max(S.max_unit, u.n);
                u.at = S.words;
                S.words += bit_words(u.n, f64 ? 8 : 4) + pad_part(u.n);
                ++S.units_n;
                if (sizes_only) {
                    // (the counts are all that is asked for)
                } else if (f64) {
                    append_unit<uint64_t, double>(V, from, to, split, S.stream64, u);
                } else {
                    append_unit<uint32_t, float>(V, from, to, split, S.stream32, u);
                }
                if (!sizes_only) S.units.push_back(u);
                u = StreamUnit{};
                from = to;
            };
            for (int64_t v = from; v < end; ++v) {
                int32_t size = 0;
                int32_t l = split;
                for (int64_t x = v, y = v + 1; x < y; ++l) {
                    size += static_cast<int32_t>(y - x);
                    const int64_t cx = V.child(x, l), cy = V.child(y, l);
                    x = cx;
                    y = cy;
                }
                if (u.n > 0 && u.n + size > kStreamRun) close(v);
                u.n += size;
            }
            close(end);
        }
        S.unit0.push_back(static_cast<int32_t>(S.units_n));
        ++S.groups;
        p0 = p1;
    }
}

}  // namespace cfr
