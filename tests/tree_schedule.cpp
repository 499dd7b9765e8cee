// tree_schedule.cpp -- replays the elimination schedule of the cable solve
// (mech_tree.h) on the CPU (tests/test_tree_schedule.py builds and runs it).
//
// Random trees, chains and stars with random conductances are cut at unit
// bounds from 1 node to larger than any cell.  Each unit is assembled, folded
// round by round and walked back as the kernels do it, once with a round's
// records in order and once in reverse order: a row that one record writes and
// another of the same round reads makes the two differ.  The solution must
// equal Hines elimination in long double.
//
// The coefficients below are positive with a dominant diagonal, so every
// elimination multiplies by factors below 1 and adds terms of one sign to the
// diagonal's excess; 1e-11 of the largest solution leaves four digits for the
// rounding of a few dozen rounds.  A wrong row or order moves it by O(1).
#include "mech_tree.h"

#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>

using namespace mech;

struct Rows { std::vector<double> S, T, U, N; };

// The tables as the device decodes them: four ints a record in a trunk whose
// rows are in global memory, else one packed word.
template <class T> static T at(const TreeTables &d, int u, int from, int q) {
    T x;
    const size_t o = (size_t)d.unit[u].block * 16 + from + sizeof(T) * q;
    memcpy(&x, &d.block.at(o), sizeof(T));
    (void)d.block.at(o + sizeof(T) - 1);
    return x;
}
struct Int4 { int32_t x, y, z, w; };
static FoldRec fold_at(const TreeTables &d, int u, int q, int &second) {
    second = -1;
    if (d.wide[u]) {
        const Int4 v = at<Int4>(d, u, d.unit[u].o_fold, q);
        return {v.x, v.y, v.z, v.w};
    }
    const uint64_t w = at<uint64_t>(d, u, d.unit[u].o_fold, q);
    auto row = [&](int shift) {
        const int x = (int)(w >> shift & 0xfff);
        return x == d.unit[u].np ? -1 : x;
    };
    second = row(36);
    const uint32_t m = (uint32_t)(w >> 48);
    return {row(0), row(12), row(24), m == kMoreNone ? -1 : (int32_t)m};
}
static ElimRec elim_at(const TreeTables &d, int u, int q) {
    if (d.wide[u]) {
        const Int4 v = at<Int4>(d, u, d.unit[u].o_elim, q);
        return {v.x, v.y, v.z};
    }
    const uint64_t w = at<uint64_t>(d, u, d.unit[u].o_elim, q);
    const int32_t i = (int32_t)(w & 0xfff), c = (int32_t)(w >> 24 & 0xfff);
    return {i, (int32_t)(w >> 12 & 0xfff), c == d.unit[u].np ? i : c};
}
static std::vector<int> list_at(const TreeTables &d, int u, int m) {
    std::vector<int> rows;
    for (bool last = m < 0; !last; ++m) {
        if (d.wide[u]) {
            const uint32_t x = at<uint32_t>(d, u, d.unit[u].o_more, m);
            rows.push_back((int)(x & ~kMoreLast));
            last = x & kMoreLast;
        } else {
            const uint16_t x = at<uint16_t>(d, u, d.unit[u].o_more, m);
            rows.push_back(x & 0xfff);
            last = x & 0x8000;
        }
    }
    return rows;
}
static std::vector<int> children_at(const TreeTables &d, int u, int i) {
    int c, m;
    if (d.wide[u]) {
        c = at<int32_t>(d, u, 0, 2 * i);
        m = at<int32_t>(d, u, 0, 2 * i + 1);
    } else {
        const uint32_t x = at<uint32_t>(d, u, 0, i);
        c = (x & 0xfff) == kNoRow ? -1 : (int)(x & 0xfff);
        m = x >> 12 == kChildNone ? -1 : (int)(x >> 12);
    }
    std::vector<int> rows = list_at(d, u, m);
    if (c >= 0) rows.insert(rows.begin(), c);
    return rows;
}

static void fold(Rows &r, const TreeTables &d, int u, int q) {
    int second;
    const FoldRec f = fold_at(d, u, q, second);
    auto up = [&](int i) {
        const double k = r.U[i] / r.S[i];
        r.S[f.t] -= r.U[i] * k;
        r.T[f.t] += k * r.T[i];
    };
    if (f.child >= 0) up(f.child);
    if (second >= 0) up(second);
    if (f.parent >= 0) {
        const double w = r.U[f.t], k = w / r.S[f.parent];
        r.S[f.t] -= w * k;
        r.T[f.t] += k * r.T[f.parent];
        r.N[f.parent] = w;
        r.U[f.t] = k * r.U[f.parent];
    }
    for (int i : list_at(d, u, f.more)) up(i);
}

int main() {
    std::mt19937_64 rng(20190506);
    std::uniform_real_distribution<double> uni(0.0, 1.0);
    int bad = 0, cases = 0;
    const int caps[] = {1, 2, 3, 7, 50, 257, 1024, 2594};
    for (int trial = 0; trial < 160; ++trial) {
        const int N = 1 + (int)(rng() % (trial < 80 ? 60 : 4000)), cap = caps[trial % 8];
        std::vector<int32_t> parent(N);
        for (int i = 0; i < N;) {
            int size = 1 + (int)(rng() % (trial % 3 == 0 ? 4000 : 100));
            if (i + size > N) size = N - i;
            parent[i] = -1;
            const int shape = (int)(rng() % 4);   // random tree, chain, star, short branches off a stem
            for (int j = 1; j < size; ++j)
                parent[i + j] = i + (shape == 0 ? (int)(rng() % j) : shape == 1 ? j - 1 : shape == 2 ? 0 : (j & 1 ? j - 1 : std::max(0, j - 2)));
            i += size;
        }
        std::vector<double> base(N), g(N), rhs(N);
        for (int i = 0; i < N; ++i) {
            base[i] = 0.01 + uni(rng);
            g[i] = parent[i] >= 0 ? 5.0 * uni(rng) : 0.0;
            rhs[i] = uni(rng) - 0.5;
        }
        // reference
        std::vector<long double> D(base.begin(), base.end()), R(rhs.begin(), rhs.end()), x(N);
        for (int i = 0; i < N; ++i)
            if (parent[i] >= 0) { D[i] += g[i]; D[parent[i]] += g[i]; }
        std::vector<long double> diag = D;
        for (int i = N - 1; i >= 0; --i)
            if (parent[i] >= 0) {
                D[parent[i]] -= (long double)g[i] * g[i] / D[i];
                R[parent[i]] += g[i] * R[i] / D[i];
            }
        long double big = 0;
        for (int i = 0; i < N; ++i) {
            x[i] = (R[i] + (parent[i] >= 0 ? g[i] * x[parent[i]] : 0)) / D[i];
            big = std::max(big, std::fabs(x[i]));
        }
        CableHost h;
        TreeSchedule s;
        if (!build_cable(N, parent.data(), cap, h, false).empty()) { ++bad; continue; }
        build_schedule(h, s);
        TreeTables d;
        tree_tables(h, s, d);
        const int U = (int)h.unit_mode.size(), P = (int)h.pos_node.size();
        std::vector<double> GT(P), GS(P), GX(P), got[2];
        for (int rev = 0; rev < 2; ++rev) {
            std::vector<double> sol(N, NAN);
            std::vector<Rows> rows(U);
            auto solve = [&](int u, bool up, bool down) {
                const int p0 = h.unit_pos[u], n = h.unit_pos[u + 1] - p0, nr = d.unit[u].nr;
                const TreeUnit &t = d.unit[u];
                Rows &r = rows[u];
                if (up) {
                    r.S.resize(n); r.T.resize(n); r.U.resize(n); r.N.assign(n, 0.0);
                    int listed = 0;
                    for (int i = 0; i < n; ++i) {
                        const int nd = h.pos_node[p0 + i], src = h.pos_src[p0 + i];
                        r.S[i] = src >= 0 ? GS[src] : (double)diag[nd];
                        r.T[i] = src >= 0 ? GT[src] : rhs[nd];
                        r.U[i] = g[nd];
                        for (int ch : children_at(d, u, i)) listed += h.pos_par[p0 + ch] == p0 + i;
                    }
                    int edges = 0;
                    for (int i = 0; i < n; ++i) edges += h.pos_par[p0 + i] >= 0;
                    if (listed != edges || at<int32_t>(d, u, t.o_re, nr) != edges || nr > kTreeRounds ||
                        (size_t)t.bytes > table_bound((size_t)n, d.wide[u]) || t.p0 != p0 || t.np != n ||
                        (!d.wide[u] && (size_t)t.bytes + 32 * ((size_t)n + 1) >
                                           (size_t)n * kCableLdsBytesPerNode + kCableLdsFixed)) ++bad;
                    for (int j = 0; j < nr; ++j) {
                        const int lo = at<int32_t>(d, u, t.o_rf, j), hi = at<int32_t>(d, u, t.o_rf, j + 1);
                        for (int q = lo; q < hi; ++q) fold(r, d, u, rev ? lo + hi - 1 - q : q);
                    }
                    for (int i = 0; i < n; ++i)
                        if (h.pos_par[p0 + i] < 0) { GS[p0 + i] = r.S[i]; GT[p0 + i] = r.T[i]; }
                }
                if (down) {
                    for (int i = 0; i < n; ++i) {
                        r.T[i] /= r.S[i]; r.U[i] /= r.S[i]; r.N[i] /= r.S[i];
                        if (h.unit_mode[u] == kUnitPiece && h.pos_par[p0 + i] < 0) r.T[i] = GX[p0 + i];
                    }
                    for (int j = nr - 1; j >= 0; --j) {
                        const int lo = at<int32_t>(d, u, t.o_re, j), hi = at<int32_t>(d, u, t.o_re, j + 1);
                        for (int q = lo; q < hi; ++q) {
                            const ElimRec e = elim_at(d, u, rev ? lo + hi - 1 - q : q);
                            r.T[e.i] += r.U[e.i] * r.T[e.p] + (e.c != e.i ? r.N[e.i] * r.T[e.c] : 0.0);
                        }
                    }
                    for (int i = 0; i < n; ++i) {
                        if (h.pos_src[p0 + i] >= 0) GX[h.pos_src[p0 + i]] = r.T[i];
                        else sol[h.pos_node[p0 + i]] = r.T[i];
                    }
                }
            };
            for (int u : h.list_up) solve(u, true, h.unit_mode[u] == kUnitFull);
            for (int u : h.list_top) solve(u, true, true);
            for (int u : h.list_top_g) solve(u, true, true);
            for (int u : h.list_down)
                if (h.unit_mode[u] == kUnitPiece) solve(u, false, true);
            got[rev] = sol;
        }
        long double err = 0;
        bool same = true;
        for (int i = 0; i < N; ++i) {
            const long double e = std::fabs(got[0][i] - x[i]);
            err = e <= err ? err : e;   // NaN counts
            same = same && got[0][i] == got[1][i];
        }
        for (int u = 0; u < U; ++u)   // rows of units in LDS fit 12 bits
            if (!d.wide[u] && h.unit_pos[u + 1] - h.unit_pos[u] > kCableLdsUnitMax) ++bad;
        if (!same || !(err <= 1e-11L * big)) {
            ++bad;
            std::printf("FAILED trial %d N %d cap %d: error %.3Lg of %.3Lg, orders %s\n", trial, N, cap, err, big,
                        same ? "agree" : "differ");
        }
        ++cases;
    }
    std::printf("%d cases, %d failed\n", cases, bad);
    return bad == 0 ? 0 : 1;
}
