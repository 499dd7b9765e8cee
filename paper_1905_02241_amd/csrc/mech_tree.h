// mech_tree.h -- host side of the cable solve: the cut of cell trees into
// units and the order in which a unit's rows are eliminated.  Plain C++, no
// device code (the CPU tests build it by itself).
#pragma once

#include <stdint.h>

#include <algorithm>
#include <string>
#include <vector>

namespace mech {

// A unit is a whole cell or a forest of them (FULL), a forest of subtrees
// whose roots hang off a larger cell's trunk (PIECE), or that trunk (TOP)
// with the piece roots as ghost rows.  Rows of the solve live at positions:
// every node has one, and every piece root has a second one as a ghost in
// its trunk's unit.
enum { kUnitFull = 0, kUnitPiece = 1, kUnitTop = 2 };

// LDS of a unit solved there: per position the four doubles of its row, its
// children (4 B), an elimination record (8 B), two fold records (8 B each; a row
// that is eliminated changes at most two others), a list entry (2 B; where it
// takes a second one, it changes one row less) and a bit; and the round
// boundaries and padding.
constexpr int kCableLdsBytesPerNode = 64;
constexpr int kCableLdsFixed = 1024;
// Records of a unit in LDS hold 12-bit rows; its children entries take 0xfff
// for no row, its other records the row after its last.  A round of e rows has at
// most 2e fold records and one for each row left, so at most two thirds of a
// unit's rows: two for each of 1024 threads.
constexpr int kCableLdsUnitMax = 3071;
constexpr int kNoRow = 0xfff;
// An elimination round of at most this many records is run by one wave, which
// needs no workgroup barrier.
constexpr int kTreeWave = 64;
// Rounds that any unit may take (log of 2^31 rows to the base 4/3 is 75).
constexpr int kTreeRounds = 80;

struct CableHost {
    std::vector<int32_t> parent, pos_node, pos_par, pos_src, elim_n, elim_p, elim_ptr, unit_pos, unit_elim,
        unit_mode, list_up, list_top, list_top_g, list_down, pos_pnode;
    std::vector<int32_t> cell_of;   // per unit: a PIECE's or TOP's cell, -1 for FULL
};

// Validates Hines order and contiguous cells, then cuts the trees into units
// of at most `cap` positions (a trunk may exceed it).  `heights`: also writes
// each unit's edge records bucketed by the child's height, the elimination
// order by heights that mech_cable_plan reports (the launches follow
// build_schedule's order instead).  Returns "" on success.
inline std::string build_cable(int64_t N, const int32_t *parent, int cap, CableHost &h, bool heights) {
    h = CableHost();
    if (cap < 1) cap = 1;
    std::vector<int32_t> first;
    for (int64_t n = 0; n < N; ++n) {
        const int32_t p = parent[n];
        if (p < -1 || p >= n) return "parent[n] must be -1 or a node index below n (Hines order)";
        if (p < 0) first.push_back((int32_t)n);
        else if (first.empty() || p < first.back())
            return "every cell must be a contiguous node range starting at its root";
    }
    if (N > 0 && (first.empty() || first[0] != 0)) return "node 0 must be a root";
    const int n_cells = (int)first.size();
    first.push_back((int32_t)N);
    h.parent.assign(parent, parent + N);
    std::vector<int32_t> sub(N, 1), ht(N, 0);
    for (int64_t n = N - 1; n >= 0; --n)
        if (parent[n] >= 0) {
            sub[parent[n]] += sub[n];
            ht[parent[n]] = std::max(ht[parent[n]], ht[n] + 1);
        }
    std::vector<int32_t> pos(N, -1), th(N, 0), levels;
    h.unit_pos.push_back(0);
    if (heights) h.elim_ptr.push_back(0);
    struct Rec { int32_t h, n, p; };
    // closes the unit whose positions were placed last; recs are (height,
    // child position, parent position), a root paired with itself
    auto add_unit = [&](int mode, std::vector<Rec> &recs, int nlev, int cell) {
        const int u = (int)h.unit_mode.size();
        h.unit_mode.push_back(mode);
        h.cell_of.push_back(cell);
        h.unit_pos.push_back((int32_t)h.pos_node.size());
        if (heights) {
            h.unit_elim.push_back((int32_t)h.elim_ptr.size() - 1);
            // by height, and within a height by parent
            std::stable_sort(recs.begin(), recs.end(),
                             [](const Rec &x, const Rec &y) { return x.h != y.h ? x.h < y.h : x.p < y.p; });
            size_t k = 0;
            for (int L = 0; L < nlev; ++L) {
                for (; k < recs.size() && recs[k].h == L; ++k) {
                    h.elim_n.push_back(recs[k].n);
                    h.elim_p.push_back(recs[k].p);
                }
                h.elim_ptr.push_back((int32_t)h.elim_n.size());
            }
        }
        levels.push_back(nlev);
        const int size = h.unit_pos[u + 1] - h.unit_pos[u];
        if (mode == kUnitFull || mode == kUnitPiece) h.list_up.push_back(u);
        if (mode == kUnitFull || mode == kUnitPiece) h.list_down.push_back(u);
        if (mode == kUnitTop) (size <= cap ? h.list_top : h.list_top_g).push_back(u);
    };
    auto place = [&](int32_t n, int32_t par_pos, int32_t src) {
        const int32_t i = (int32_t)h.pos_node.size();
        h.pos_node.push_back(n);
        h.pos_pnode.push_back(parent[n]);
        h.pos_par.push_back(par_pos);
        h.pos_src.push_back(src);
        return i;
    };

    // whole cells that fit, packed into forests of up to `pack` nodes so that
    // many small cells do not each take a workgroup
    int64_t fit_nodes = 0;
    for (int c = 0; c < n_cells; ++c)
        if (first[c + 1] - first[c] <= cap) fit_nodes += first[c + 1] - first[c];
    const int pack = (int)std::min<int64_t>(cap, std::max<int64_t>(1024, (fit_nodes + 511) / 512));
    std::vector<Rec> recs;
    int nlev = 0, cur = 0;
    auto close_full = [&]() {
        // every root's own record goes to the unit's top height
        for (Rec &r : recs)
            if (r.h < 0) r.h = nlev - 1;
        if (cur > 0) add_unit(kUnitFull, recs, nlev, -1);
        recs.clear();
        nlev = 0;
        cur = 0;
    };
    for (int c = 0; c < n_cells; ++c) {
        const int32_t a = first[c], b = first[c + 1];
        if (b - a > cap) continue;
        if (cur + (b - a) > pack) close_full();
        for (int32_t n = a; n < b; ++n) {
            const int32_t p = parent[n];
            pos[n] = place(n, p >= 0 ? pos[p] : -1, -1);
            if (heights) recs.push_back({p >= 0 ? ht[n] : -1, pos[n], p >= 0 ? pos[p] : pos[n]});
        }
        nlev = std::max(nlev, ht[a] + 1);
        cur += b - a;
    }
    close_full();

    // cells too large: maximal subtrees that fit become pieces, packed into
    // forests; the trunk (subtree larger than cap) is one unit
    for (int c = 0; c < n_cells; ++c) {
        const int32_t a = first[c], b = first[c + 1];
        if (b - a <= cap) continue;
        std::vector<int32_t> pid(b - a, -1), roots, unit_of;
        for (int32_t n = a; n < b; ++n) {
            if (sub[n] > cap) continue;
            const int32_t p = parent[n];
            if (sub[p] > cap) {
                pid[n - a] = (int32_t)roots.size();
                roots.push_back(n);
            } else {
                pid[n - a] = pid[p - a];
            }
        }
        // greedy packing in root order
        int units = 0, fill = 0;
        for (int32_t r : roots) {
            if (units == 0 || fill + sub[r] > cap) {
                ++units;
                fill = 0;
            }
            fill += sub[r];
            unit_of.push_back(units - 1);
        }
        std::vector<std::vector<int32_t>> members(units);
        for (int32_t n = a; n < b; ++n)
            if (pid[n - a] >= 0) members[unit_of[pid[n - a]]].push_back(n);
        for (int k = 0; k < units; ++k) {
            recs.clear();
            int nl = 0;
            for (int32_t n : members[k]) {
                const int32_t p = parent[n];
                const bool root = sub[p] > cap;
                pos[n] = place(n, root ? -1 : pos[p], -1);
                if (root) nl = std::max(nl, ht[n]);
                else if (heights) recs.push_back({ht[n], pos[n], pos[p]});
            }
            add_unit(kUnitPiece, recs, nl, c);
        }
        // the trunk with the piece roots as ghost leaves; heights counted
        // within the unit (a ghost is a leaf)
        std::vector<int32_t> tn;
        for (int32_t n = a; n < b; ++n)
            if (sub[n] > cap || (parent[n] >= 0 && sub[parent[n]] > cap)) tn.push_back(n);
        for (auto it = tn.rbegin(); it != tn.rend(); ++it) th[*it] = 0;
        for (auto it = tn.rbegin(); it != tn.rend(); ++it)
            if (parent[*it] >= 0) th[parent[*it]] = std::max(th[parent[*it]], th[*it] + 1);
        recs.clear();
        for (size_t k = 0; k < tn.size(); ++k) {
            const int32_t n = tn[k], p = parent[n];
            const bool ghost = sub[n] <= cap;
            const int32_t i = place(n, p >= 0 ? pos[p] : -1, ghost ? pos[n] : -1);
            if (!ghost) pos[n] = i;   // trunk nodes: their only position
            if (heights) recs.push_back({th[n], i, p >= 0 ? pos[p] : i});
        }
        add_unit(kUnitTop, recs, th[a] + 1, c);
    }
    if (heights) h.unit_elim.push_back((int32_t)h.elim_ptr.size() - 1);
    // tallest units first so that the longest chains of barriers start first
    auto by_height = [&](std::vector<int32_t> &l) {
        std::stable_sort(l.begin(), l.end(), [&](int32_t x, int32_t y) { return levels[x] > levels[y]; });
    };
    by_height(h.list_up);
    by_height(h.list_top);
    by_height(h.list_top_g);
    by_height(h.list_down);
    return "";
}

// The order of elimination within the units.  Hines elimination folds a row
// into its parent once its children are done, so a tree takes as many
// dependent steps as it is tall.  Here a round eliminates every leaf and
// every second node of each unbranched run at once: a row with at most one
// child left can be eliminated whatever its depth, and leaves its child
// hanging off its parent with a new coupling.  Each round removes about half
// of the rows, so a unit takes about log2 of its size (branched cells cut at
// 1024 nodes: at most 11 rounds where the tallest unit has 82 heights).
//
// A round's rows are pairwise not adjacent, so they are final when it starts.
// Each surviving neighbour of one of them has a fold record, and one thread
// folds all of that row's eliminated neighbours in the record's order: no
// row is written by two threads and the result does not depend on
// scheduling.  The roots of a unit are never eliminated.
//
// Rows are numbered within their unit.  `fold` records hold (row, its
// eliminated parent or kNoRow, its first eliminated child or kNoRow, index of
// further children in `more` or -1), `elim` records (row, parent, child or
// the row itself); `more` entries hold a row and, in the top bit, whether the
// list ends.
// `kid` marks the rows that have a child left when they are eliminated: in a
// unit's rows in LDS the coupling to it takes the place of the pivot then, and the
// others' pivots stay there.
struct FoldRec { int32_t t, parent, child, more; };
struct ElimRec { int32_t i, p, c; };
// On the device a unit's tables are one block of memory (tree_tables below).
// A unit solved in LDS packs a record in a 64-bit word, 12 bits a row; a
// missing neighbour is the row after the unit's last (S = 1, the rest 0), so
// that a thread can read all neighbours at once; two children are in the word,
// and 16 bits are the index of a list of more.  A trunk with its rows in
// global memory (list_top_g) takes four ints.
constexpr uint32_t kMoreNone = 0xffffu;      // the index field of a packed record without a list
constexpr uint32_t kChildNone = 0xfffffu;    // the same in a packed children entry
constexpr uint32_t kMoreLast = 0x80000000u;
inline uint64_t pack_fold(const FoldRec &r, const uint32_t *more, int n) {
    int second = -1, m = r.more;
    if (m >= 0) {
        second = (int)(more[m] & ~kMoreLast);
        m = (more[m] & kMoreLast) ? -1 : m + 1;
    }
    auto row = [&](int x) { return (uint64_t)(x < 0 ? n : x); };
    return (uint64_t)r.t | row(r.parent) << 12 | row(r.child) << 24 | row(second) << 36 |
           (uint64_t)(m < 0 ? kMoreNone : (uint32_t)m) << 48;
}
inline uint64_t pack_elim(const ElimRec &r, int n) {
    return (uint64_t)r.i | (uint64_t)r.p << 12 | (uint64_t)(r.c == r.i ? n : r.c) << 24;
}
inline uint32_t pack_child(int child, int more) {
    return (uint32_t)(child < 0 ? kNoRow : child) | (more < 0 ? kChildNone : (uint32_t)more) << 12;
}

struct TreeSchedule {
    std::vector<int32_t> unit_rnd;          // [units + 1] into rnd_fold / rnd_elim (rounds + 1 entries each)
    std::vector<int32_t> rnd_fold, rnd_elim;   // record boundaries, counted over all units
    std::vector<int32_t> unit_more;         // [units + 1] into more
    std::vector<FoldRec> fold;
    std::vector<ElimRec> elim;
    std::vector<uint32_t> more;
    // per position: its first child in the unit (or -1) and the further
    // children's index in more (unit-relative, or -1), for the axial currents
    std::vector<int32_t> child, child_more;
    std::vector<char> kid;   // per position
};

inline void build_schedule(const CableHost &h, TreeSchedule &s) {
    s = TreeSchedule();
    const int U = (int)h.unit_mode.size();
    const size_t P = h.pos_node.size();
    s.child.assign(P, -1);
    s.child_more.assign(P, -1);
    s.kid.assign(P, 0);
    s.fold.reserve(P + P / 8);
    s.elim.reserve(P);
    s.unit_rnd.push_back(0);
    s.unit_more.push_back(0);
    std::vector<int32_t> cp, nch, alive, next, mark, first, link, lastc, sel, touched;
    for (int u = 0; u < U; ++u) {
        const int p0 = h.unit_pos[u], n = h.unit_pos[u + 1] - p0;
        const size_t m0 = s.more.size();
        // cp: parent among the rows left; nch: children left; xr: the xor of
        // the children's rows, the only child's row when one is left
        cp.resize(n);
        nch.assign(n, 0);
        std::vector<int32_t> xr(n, 0);
        alive.resize(n);
        first.assign(n, -1);
        link.assign(n, -1);
        lastc.assign(n, -1);
        for (int i = 0; i < n; ++i) {
            cp[i] = h.pos_par[p0 + i] >= 0 ? h.pos_par[p0 + i] - p0 : -1;
            alive[i] = i;
            if (cp[i] >= 0) {
                ++nch[cp[i]];
                xr[cp[i]] ^= i;
            }
        }
        // a list of rows linked per owner, in the order of insertion; its
        // tail goes to `more`
        auto append = [&](int owner, int row) {
            link[row] = -1;
            if (first[owner] < 0) first[owner] = row;
            else link[lastc[owner]] = row;
            lastc[owner] = row;
        };
        auto flush = [&](int owner, int32_t &head, int32_t &more) {
            head = first[owner];
            more = -1;
            if (head >= 0 && link[head] >= 0) {
                more = (int32_t)(s.more.size() - m0);
                for (int r = link[head]; r >= 0; r = link[r])
                    s.more.push_back((uint32_t)r | (link[r] < 0 ? kMoreLast : 0u));
            }
            first[owner] = lastc[owner] = -1;
        };
        for (int i = 0; i < n; ++i)
            if (cp[i] >= 0) append(cp[i], i);
        for (int i = 0; i < n; ++i) flush(i, s.child[p0 + i], s.child_more[p0 + i]);

        mark.assign(n, -1);
        s.rnd_fold.push_back((int32_t)s.fold.size());
        s.rnd_elim.push_back((int32_t)s.elim.size());
        for (int round = 0;; ++round) {
            // Deepest rows first: a leaf, then every second row above it.  mark
            // is `round` on a taken row's neighbours, -round - 2 on a taken row
            // and n + round on a neighbour that is listed.  An eligible row is
            // passed over only for a taken child, and a tree has fewer branch
            // rows than leaves, so a round takes at least a quarter of the rows
            // and kTreeRounds rounds are enough.
            const int taken = -round - 2;
            sel.clear();
            for (size_t k = alive.size(); k-- > 0;) {
                const int i = alive[k];
                if (cp[i] < 0 || nch[i] > 1 || mark[i] == round) continue;
                sel.push_back(i);
                mark[cp[i]] = round;
                if (nch[i] == 1) mark[xr[i]] = round;
                mark[i] = taken;
            }
            if (sel.empty()) break;
            touched.clear();
            // ascending rows, so that a parent's eliminated children are folded in row order
            std::reverse(sel.begin(), sel.end());
            for (int i : sel) {
                const int p = cp[i], c = nch[i] == 1 ? xr[i] : -1;
                s.elim.push_back({i, p, c >= 0 ? c : i});
                s.kid[p0 + i] = c >= 0;
                if (mark[p] == round) {
                    mark[p] = n + round;
                    touched.push_back(p);
                }
                append(p, i);
                if (c >= 0 && mark[c] == round) {
                    mark[c] = n + round;
                    touched.push_back(c);
                }
            }
            for (int t : touched) {
                FoldRec r{t, -1, -1, -1};
                if (cp[t] >= 0 && mark[cp[t]] == taken) r.parent = cp[t];
                flush(t, r.child, r.more);
                s.fold.push_back(r);
            }
            // the rows that are left: a child of an eliminated row hangs off that row's parent
            for (int i : sel) {
                const int p = cp[i];
                xr[p] ^= i;
                if (nch[i] == 1) {
                    cp[xr[i]] = p;
                    xr[p] ^= xr[i];
                } else {
                    --nch[p];
                }
            }
            next.clear();
            for (int i : alive)
                if (mark[i] != taken) next.push_back(i);
            alive.swap(next);
            s.rnd_fold.push_back((int32_t)s.fold.size());
            s.rnd_elim.push_back((int32_t)s.elim.size());
        }
        s.unit_rnd.push_back((int32_t)s.rnd_fold.size());
        s.unit_more.push_back((int32_t)s.more.size());
    }
}

// A unit as a workgroup finds it: one 64-byte read.  Its block holds, each at
// a multiple of 16 bytes: the children of every row (o_more bytes), the lists
// (up to o_kid), a bit a row, in 32-bit words, for the rows marked in `kid` (up
// to o_fold; none in a trunk with rows in global memory), the fold records (up to
// o_rf), the round boundaries of the fold (up to o_re) and of the elimination
// records (up to o_elim), the elimination records (up to bytes).
struct TreeUnit {
    int32_t p0, np, mode, nr;
    int32_t block;   // in units of 16 bytes
    int32_t o_more, o_fold, o_rf, o_re, o_elim, bytes;
    int32_t solves_trunk;   // piece: solves its cell's trunk itself
    int32_t wide;           // rows in global memory
    int32_t o_kid;
    int32_t unused[2];
};
struct TreeTables {
    std::vector<TreeUnit> unit;
    std::vector<char> block;
    std::vector<char> wide;       // per unit
};
inline std::vector<char> wide_units(const CableHost &h) {
    std::vector<char> w(h.unit_mode.size(), 0);
    for (int32_t u : h.list_top_g) w[u] = 1;
    return w;
}
// Bytes that a unit's block takes at most.
inline size_t table_bound(size_t rows, bool wide) {
    const size_t rounds = std::min<size_t>(rows, kTreeRounds + 1);
    return rows * (wide ? 8 + 8 + 32 + 16 : 4 + 2 + 16 + 8) + (rows / 32 + 1) * 4 + 8 * rounds + 8 * 16;
}
inline void tree_tables(const CableHost &h, const TreeSchedule &s, TreeTables &d) {
    d = TreeTables();
    const int U = (int)h.unit_mode.size();
    d.wide = wide_units(h);
    d.unit.resize(U);
    for (int u = 0; u < U; ++u) {
        TreeUnit &t = d.unit[u];
        t = TreeUnit();
        t.p0 = h.unit_pos[u];
        t.np = h.unit_pos[u + 1] - t.p0;
        t.mode = h.unit_mode[u];
        const int a = s.unit_rnd[u], b = s.unit_rnd[u + 1] - 1;
        t.nr = b - a;
        t.block = (int32_t)(d.block.size() / 16);
        const size_t start = d.block.size();
        auto put = [&](const void *p, size_t n) {
            const char *c = (const char *)p;
            d.block.insert(d.block.end(), c, c + n);
        };
        auto close = [&]() {
            d.block.resize((d.block.size() + 15) & ~(size_t)15);
            return (int32_t)(d.block.size() - start);
        };
        const bool w = d.wide[u];
        t.wide = w;
        for (int i = t.p0; i < t.p0 + t.np; ++i) {
            const int32_t both[2] = {s.child[i], s.child_more[i]};
            const uint32_t one = pack_child(s.child[i], s.child_more[i]);
            if (w) put(both, 8);
            else put(&one, 4);
        }
        t.o_more = close();
        for (int m = s.unit_more[u]; m < s.unit_more[u + 1]; ++m) {
            const uint32_t x = s.more[m];
            const uint16_t y = (uint16_t)((x & 0xfffu) | ((x & kMoreLast) ? 0x8000u : 0u));
            if (w) put(&x, 4);
            else put(&y, 2);
        }
        const uint32_t past = 0;   // read, not used, behind the last entry
        put(&past, w ? 4 : 2);
        t.o_kid = close();
        for (int i = 0; !w && i < t.np; i += 32) {
            uint32_t x = 0;
            for (int k = i; k < std::min(i + 32, t.np); ++k) x |= (uint32_t)s.kid[t.p0 + k] << (k - i);
            put(&x, 4);
        }
        t.o_fold = close();
        for (int q = s.rnd_fold[a]; q < s.rnd_fold[b]; ++q) {
            const uint64_t x = pack_fold(s.fold[q], s.more.data() + s.unit_more[u], t.np);
            if (w) put(&s.fold[q], 16);
            else put(&x, 8);
        }
        t.o_rf = close();
        for (int j = a; j <= b; ++j) {
            const int32_t x = s.rnd_fold[j] - s.rnd_fold[a];
            put(&x, 4);
        }
        t.o_re = close();
        for (int j = a; j <= b; ++j) {
            const int32_t x = s.rnd_elim[j] - s.rnd_elim[a];
            put(&x, 4);
        }
        t.o_elim = close();
        for (int q = s.rnd_elim[a]; q < s.rnd_elim[b]; ++q) {
            const ElimRec &e = s.elim[q];
            const int32_t four[4] = {e.i, e.p, e.c, 0};
            const uint64_t x = pack_elim(e, t.np);
            if (w) put(four, 16);
            else put(&x, 8);
        }
        t.bytes = close();
    }
}

// LDS bytes of a unit's rows (L, T, U, S each): its own and the one that stands
// for a missing neighbour.
constexpr int tree_row_bytes(int np) { return 32 * (np + 1); }
// Bytes of a unit's block that the first launch copies to LDS: whole cells need
// all of it, pieces what leads to their roots, trunks the children alone (the
// last launch takes a piece's block from o_re on).  By value: a reference to the
// unit kept it in memory on the device, 68 bytes of scratch a lane and 12 % of a
// solve.
constexpr int tree_up_bytes(int mode, int bytes, int o_re, int o_kid) {
    return mode == kUnitFull ? bytes : mode == kUnitPiece ? o_re : o_kid;
}

// What the launches of a solve run, a unit (in `b` a pair) a workgroup, and their
// sizes.  Trunks that every piece of the cell has room for beside its own rows
// are solved by the pieces; the others take a launch of their own.
struct TreeLaunches {
    std::vector<int32_t> pos;   // four per position (CableDev::pos)
    std::vector<TreeUnit> a, top, top_g, b;
    size_t lds_a = 0, lds_top = 0, lds_b = 0;   // dynamic LDS
    size_t rows_a = 0, rows_b = 0;              // rows of the largest unit
};
inline void tree_launches(const CableHost &h, TreeTables &t, size_t lds_bytes, TreeLaunches &l) {
    l = TreeLaunches();
    const int U = (int)t.unit.size();
    auto alone = [](const TreeUnit &u) { return (size_t)tree_row_bytes(u.np) + u.bytes; };
    auto down = [](const TreeUnit &u) { return (size_t)tree_row_bytes(u.np) + u.bytes - u.o_re; };
    auto grow = [](size_t &x, size_t y) { x = std::max(x, y); };
    std::vector<int> trunk_of;
    std::vector<size_t> piece_max;
    for (int u = 0; u < U; ++u) {
        if (h.cell_of[u] < 0) continue;
        const size_t cell = (size_t)h.cell_of[u];
        if (trunk_of.size() <= cell) {
            trunk_of.resize(cell + 1, -1);
            piece_max.resize(cell + 1, 0);
        }
        if (t.unit[u].mode == kUnitTop) trunk_of[cell] = u;
        else grow(piece_max[cell], down(t.unit[u]));
    }
    std::vector<char> shared(U, 0);
    for (int32_t u : h.list_top) shared[u] = alone(t.unit[u]) + piece_max[h.cell_of[u]] <= lds_bytes;
    auto first = [&](const TreeUnit &x) {
        l.a.push_back(x);
        grow(l.lds_a, (size_t)tree_row_bytes(x.np) + tree_up_bytes(x.mode, x.bytes, x.o_re, x.o_kid));
        grow(l.rows_a, (size_t)x.np);
    };
    auto last = [&](const TreeUnit &x, const TreeUnit &trunk, size_t bytes) {
        l.b.push_back(x);
        l.b.push_back(trunk);
        grow(l.lds_b, bytes);
        grow(l.rows_b, (size_t)x.np);
    };
    for (int32_t u : h.list_up) {
        TreeUnit &x = t.unit[u];
        if (x.mode == kUnitPiece) x.solves_trunk = shared[trunk_of[h.cell_of[u]]];
        first(x);
    }
    for (int32_t u : h.list_down) {
        const TreeUnit &x = t.unit[u];
        if (x.mode != kUnitPiece) continue;
        const TreeUnit &y = t.unit[trunk_of[h.cell_of[u]]];
        last(x, y, down(x) + (x.solves_trunk ? alone(y) : 0));
    }
    for (int32_t u : h.list_top) {
        const TreeUnit &x = t.unit[u];
        if (shared[u]) {
            first(x);
            last(x, x, alone(x));
        } else {
            l.top.push_back(x);
            grow(l.lds_top, alone(x));
            grow(l.rows_a, (size_t)x.np);
        }
    }
    for (int32_t u : h.list_top_g) l.top_g.push_back(t.unit[u]);
    l.pos.resize(4 * h.pos_node.size());
    for (size_t p = 0; p < h.pos_node.size(); ++p) {
        l.pos[4 * p] = h.pos_node[p];
        l.pos[4 * p + 1] = h.pos_pnode[p];
        l.pos[4 * p + 2] = h.pos_src[p];
        l.pos[4 * p + 3] = h.pos_par[p] >= 0 ? -1 : -2;
    }
    for (int u = 0; u < U; ++u)
        for (int p = h.unit_pos[u]; p < h.unit_pos[u + 1]; ++p)
            if (const int src = h.pos_src[p]; src >= 0 && shared[u]) l.pos[4 * (size_t)src + 3] = p - h.unit_pos[u];
}

}  // namespace mech
