// regrid.cpp -- host side of a regrid: the refine / coarsen decision from the
// device error estimate and the data source of every new leaf (the "AMR
// Coarsen Refine" node of the flow charts, Fig. 1 and Fig. 2, which the paper
// keeps on the host with the tree).
#include <algorithm>
#include <utility>

#include "block_table.hpp"
#include "mesh.hpp"

namespace agile {

namespace {

// periodic neighbour index: c in [-1, n]
inline int64_t wrapc(int64_t c, int64_t n) { return c < 0 ? c + n : (c >= n ? c - n : c); }

} // namespace

int regrid_decide(const PlanInput &in, int64_t n, const agile_block_desc *blocks, const double *err, int max_level,
                  double refine, double coarsen, std::vector<agile_block_desc> &out, std::vector<RegridSource> &src,
                  int64_t &refined, int64_t &coarsened, std::string &error) {
    out.clear();
    src.clear();
    refined = coarsened = 0;
    if (max_level < 1 || max_level > in.max_level) {
        error = "regrid: maximum level outside [1, the mesh's maximum level]";
        return AGILE_EINVAL;
    }
    auto dims = [&](int l, int d) { return int64_t(in.base[d]) << (l - 1); };
    BlockTable leaf{size_t(n)};
    for (int64_t q = 0; q < n; ++q)
        leaf.insert(block_key(blocks[q].level, blocks[q].idx[0], blocks[q].idx[1], blocks[q].idx[2]), int(q));
    // old leaf covering level-l block c, or -1 when finer leaves cover it
    auto covering = [&](int l, const int64_t c[3]) -> int {
        for (int L = l; L >= 1; --L) {
            const int q = leaf.find(block_key(L, c[0] >> (l - L), c[1] >> (l - L), c[2] >> (l - L)));
            if (q >= 0) return q;
        }
        return -1;
    };

    // refinement and its propagation to coarser face neighbours
    std::vector<char> R(size_t(n), 0);
    std::vector<int> work;
    for (int64_t q = 0; q < n; ++q)
        if (err[q] > refine && blocks[q].level < max_level) {
            R[q] = 1;
            work.push_back(int(q));
        }
    while (!work.empty()) {
        const int q = work.back();
        work.pop_back();
        const int l = blocks[q].level;
        for (int d = 0; d < 3; ++d)
            for (int s = -1; s <= 1; s += 2) {
                int64_t c[3] = {blocks[q].idx[0], blocks[q].idx[1], blocks[q].idx[2]};
                c[d] = wrapc(c[d] + s, dims(l, d));
                const int h = covering(l, c);
                if (h >= 0 && blocks[h].level < l && !R[h]) {
                    R[h] = 1;
                    work.push_back(h);
                }
            }
    }

    // coarsening candidates: complete octets of low-error leaves, none refined
    auto low = [&](int k) { return k >= 0 && err[k] < coarsen && !R[k]; };
    struct Octet {
        int child[8];
    };
    std::vector<Octet> P;
    std::vector<char> gone(size_t(n), 0);   // leaves of the octets that are coarsened
    for (int64_t q = 0; q < n; ++q) {
        const agile_block_desc &b = blocks[q];
        if (b.level < 2 || ((b.idx[0] | b.idx[1] | b.idx[2]) & 1) || !low(int(q))) continue;
        Octet o;
        bool ok = true;
        for (int c = 0; c < 8 && ok; ++c) {
            o.child[c] = leaf.find(block_key(b.level, b.idx[0] + (c & 1), b.idx[1] + ((c >> 1) & 1), b.idx[2] + (c >> 2)));
            ok = low(o.child[c]);
        }
        if (!ok) continue;
        for (int k : o.child) gone[k] = 1;
        P.push_back(o);
    }

    // whether level-l block c is a leaf of the new mesh, for the current choice
    // of coarsened octets: an old leaf that stays, the parent of a coarsened
    // octet or a child of a refined leaf
    auto new_leaf = [&](int l, const int64_t c[3]) -> bool {
        const int q = leaf.find(block_key(l, c[0], c[1], c[2]));
        if (q >= 0) return !gone[q] && !R[q];
        if (l < in.max_level) {
            const int k = leaf.find(block_key(l + 1, 2 * c[0], 2 * c[1], 2 * c[2]));
            if (k >= 0 && gone[k]) return true;
        }
        if (l == 1) return false;
        const int p = leaf.find(block_key(l - 1, c[0] >> 1, c[1] >> 1, c[2] >> 1));
        return p >= 0 && R[p];
    };
    // coarsening balance: withdraw octets whose parent would touch a leaf two
    // levels finer, until none does (withdrawing only refines neighbourhoods)
    for (bool changed = !P.empty(); changed;) {
        std::vector<Octet> keep, withdrawn;
        for (const Octet &p : P) {
            const agile_block_desc &b = blocks[p.child[0]];
            const int lp = b.level - 1;
            bool bad = false;
            for (int d = 0; d < 3 && !bad; ++d)
                for (int s = -1; s <= 1 && !bad; s += 2) {
                    int64_t c[3] = {b.idx[0] >> 1, b.idx[1] >> 1, b.idx[2] >> 1};
                    c[d] = wrapc(c[d] + s, dims(lp, d));
                    bool covered = false;
                    for (int L = lp; L >= 1 && !covered; --L) {
                        const int64_t up[3] = {c[0] >> (lp - L), c[1] >> (lp - L), c[2] >> (lp - L)};
                        covered = new_leaf(L, up);
                    }
                    if (covered) continue;
                    // subdivided: its children facing the parent must be leaves
                    for (int o = 0; o < 8 && !bad; ++o) {
                        const int64_t ch[3] = {2 * c[0] + (o & 1), 2 * c[1] + ((o >> 1) & 1), 2 * c[2] + (o >> 2)};
                        if ((ch[d] & 1) != (s < 0 ? 1 : 0)) continue;
                        if (!new_leaf(lp + 1, ch)) bad = true;
                    }
                }
            (bad ? withdrawn : keep).push_back(p);
        }
        for (const Octet &p : withdrawn)
            for (int k : p.child) gone[k] = 0;
        P.swap(keep);
        changed = !withdrawn.empty();
    }

    // the new leaves with their sources, sorted
    std::vector<std::pair<uint64_t, RegridSource>> nl;
    nl.reserve(size_t(n));
    for (int64_t q = 0; q < n; ++q) {
        const agile_block_desc &b = blocks[q];
        RegridSource S;
        S.src[0] = int(q);
        if (R[q]) {
            S.kind = 1;
            for (int o = 0; o < 8; ++o) {
                S.octant = o;
                nl.emplace_back(block_key(b.level + 1, 2 * int64_t(b.idx[0]) + (o & 1),
                                          2 * int64_t(b.idx[1]) + ((o >> 1) & 1), 2 * int64_t(b.idx[2]) + (o >> 2)), S);
            }
        } else if (!gone[q]) {
            nl.emplace_back(block_key(b.level, b.idx[0], b.idx[1], b.idx[2]), S);
        }
    }
    for (const Octet &p : P) {
        const agile_block_desc &b = blocks[p.child[0]];
        RegridSource S;
        S.kind = 2;
        for (int o = 0; o < 8; ++o) S.src[o] = p.child[o];
        nl.emplace_back(block_key(b.level - 1, b.idx[0] >> 1, b.idx[1] >> 1, b.idx[2] >> 1), S);
    }
    std::vector<std::pair<uint64_t, int>> at(nl.size());
    for (size_t i = 0; i < nl.size(); ++i) at[i] = {nl[i].first, int(i)};
    std::sort(at.begin(), at.end(), [](const auto &a, const auto &b) { return a.first < b.first; });
    out.resize(nl.size());
    src.resize(nl.size());
    for (size_t i = 0; i < at.size(); ++i) {
        const uint64_t k = at[i].first;
        out[i].level = int(k >> 60);
        out[i].idx[0] = int((k >> 40) & 0xfffff);
        out[i].idx[1] = int((k >> 20) & 0xfffff);
        out[i].idx[2] = int(k & 0xfffff);
        src[i] = nl[size_t(at[i].second)].second;
    }
    for (char r : R) refined += r;
    coarsened = int64_t(P.size());
    return AGILE_OK;
}

// Data sources of the blocks `nw` of a regridded mesh from the blocks `old`
// of the same domain, by position: a block that exists in both is copied, one
// whose parent block is old is that parent's child, one whose 8 children are
// old is their mean.  (The tiles of a regrid of larger blocks, where the
// decision was taken per block.)
int regrid_sources(const std::vector<agile_block_desc> &old, const std::vector<agile_block_desc> &nw,
                   std::vector<RegridSource> &src, std::string &error) {
    BlockTable at{old.size()};
    for (size_t q = 0; q < old.size(); ++q)
        at.insert(block_key(old[q].level, old[q].idx[0], old[q].idx[1], old[q].idx[2]), int(q));
    src.assign(nw.size(), RegridSource{});
    for (size_t q = 0; q < nw.size(); ++q) {
        const agile_block_desc &b = nw[q];
        RegridSource &r = src[q];
        int k = at.find(block_key(b.level, b.idx[0], b.idx[1], b.idx[2]));
        if (k >= 0) {
            r.kind = 0;
            r.src[0] = k;
            continue;
        }
        if (b.level > 1) {
            k = at.find(block_key(b.level - 1, b.idx[0] >> 1, b.idx[1] >> 1, b.idx[2] >> 1));
            if (k >= 0) {
                r.kind = 1;
                r.octant = int((b.idx[0] & 1) + 2 * (b.idx[1] & 1) + 4 * (b.idx[2] & 1));
                r.src[0] = k;
                continue;
            }
        }
        r.kind = 2;
        for (int o = 0; o < 8; ++o) {
            k = at.find(block_key(b.level + 1, 2 * int64_t(b.idx[0]) + (o & 1), 2 * int64_t(b.idx[1]) + ((o >> 1) & 1),
                                  2 * int64_t(b.idx[2]) + (o >> 2)));
            if (k < 0) {
                error = "regrid: a new block has no source in the old mesh";
                return AGILE_EINVAL;
            }
            r.src[o] = k;
        }
    }
    return AGILE_OK;
}

} // namespace agile
