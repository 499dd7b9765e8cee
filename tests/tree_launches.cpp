// tree_launches.cpp -- the launches of a cable solve on the CPU
// (tests/test_tree_launches.py builds and runs it).
//
// tests/tree_schedule.cpp replays the rounds of each unit by itself.  Here the
// launches run as they are planned (tree_launches): every workgroup has an LDS
// of the planned size and no more, finds its tables and rows in it where the
// kernels put them, and reads other units' rows only through the positions and
// the memory between the launches.  Trees whose trunks are solved by their
// pieces, in LDS in a launch of their own, and in global memory must all give
// the solution of Hines elimination in long double.
//
// The coefficients are positive with a dominant diagonal; 1e-11 of the largest
// solution leaves four digits for the rounding of a few dozen rounds, a wrong
// row or order moves it by O(1).
#define MECH_HD_INLINE static inline
#include "mech_math.h"
#include "mech_tree.h"

#include <cstdio>
#include <cstring>
#include <random>

using namespace mech;

struct Problem {
    int N;
    std::vector<int32_t> parent;
    std::vector<double> a, lk, g, v, rhs;   // area/100, 1e-3 cm/dt + d, conductance to the parent
};

// A workgroup's LDS, or global memory: rows of S, T, U, N and a unit's tables.
struct Rows {
    std::vector<char> &mem;
    size_t at;
    double &operator()(int i, int k) {
        const size_t o = at + 32 * (size_t)i + 8 * k;
        (void)mem.at(o + 7);
        return *reinterpret_cast<double *>(&mem.at(o));
    }
};
enum { kS, kT, kU, kN };
struct Tables {
    const std::vector<char> &mem;
    long at;   // of the block's first byte, copied or not
    const TreeUnit &u;
    template <class T> T get(long from, long q) const {
        T x;
        const size_t o = (size_t)(at + from + (long)sizeof(T) * q);
        (void)mem.at(o + sizeof(T) - 1);
        memcpy(&x, &mem.at(o), sizeof(T));
        return x;
    }
    std::vector<int> list(int m) const {
        std::vector<int> r;
        for (bool last = m < 0; !last; ++m) {
            if (u.wide) {
                const uint32_t x = get<uint32_t>(u.o_more, m);
                r.push_back((int)(x & ~kMoreLast));
                last = x & kMoreLast;
            } else {
                const uint16_t x = get<uint16_t>(u.o_more, m);
                r.push_back(x & 0xfff);
                last = x & 0x8000;
            }
        }
        return r;
    }
    std::vector<int> children(int i) const {
        const uint32_t x = u.wide ? 0 : get<uint32_t>(0, i);
        const int c = u.wide ? get<int32_t>(0, 2 * i) : (x & 0xfff) == kNoRow ? -1 : (int)(x & 0xfff);
        const int m = u.wide ? get<int32_t>(0, 2 * i + 1) : x >> 12 == kChildNone ? -1 : (int)(x >> 12);
        std::vector<int> r = list(m);
        if (c >= 0) r.insert(r.begin(), c);
        return r;
    }
    // a fold record: the row, its eliminated parent (or -1) and its eliminated children
    int fold(int q, int &parent, std::vector<int> &ch) const {
        int t, c, second = -1, m;
        if (u.wide) {
            t = get<int32_t>(u.o_fold, 4 * q);
            parent = get<int32_t>(u.o_fold, 4 * q + 1);
            c = get<int32_t>(u.o_fold, 4 * q + 2);
            m = get<int32_t>(u.o_fold, 4 * q + 3);
        } else {
            const uint64_t w = get<uint64_t>(u.o_fold, q);
            auto row = [&](int s) { return (int)(w >> s & 0xfff) == u.np ? -1 : (int)(w >> s & 0xfff); };
            t = row(0);
            parent = row(12);
            c = row(24);
            second = row(36);
            m = (uint32_t)(w >> 48) == kMoreNone ? -1 : (int)(w >> 48);
        }
        ch = list(m);
        if (second >= 0) ch.insert(ch.begin(), second);
        if (c >= 0) ch.insert(ch.begin(), c);
        return t;
    }
    void elim(int q, int &i, int &p, int &c) const {
        if (u.wide) {
            i = get<int32_t>(u.o_elim, 4 * q);
            p = get<int32_t>(u.o_elim, 4 * q + 1);
            c = get<int32_t>(u.o_elim, 4 * q + 2);
            if (c == i) c = -1;
        } else {
            const uint64_t w = get<uint64_t>(u.o_elim, q);
            i = (int)(w & 0xfff);
            p = (int)(w >> 12 & 0xfff);
            c = (int)(w >> 24 & 0xfff) == u.np ? -1 : (int)(w >> 24 & 0xfff);
        }
    }
};

struct Solver {
    const Problem &P;
    const TreeTables &t;
    const TreeLaunches &l;
    std::vector<char> G;
    std::vector<double> dv;

    int pos(const TreeUnit &u, int i, int k) const { return l.pos.at(4 * (size_t)(u.p0 + i) + k); }
    void assemble(const TreeUnit &u, Rows r, const Tables &tab, bool take) {
        Rows g{G, 0};
        for (int i = 0; i < u.np; ++i) {
            const int n = pos(u, i, 0), p = pos(u, i, 1), src = pos(u, i, 2);
            const double gu = P.g[n], f = gu * (P.v[p >= 0 ? p : n] - P.v[n]);
            r(i, kS) = take && src >= 0 ? g(src, kS) : fma(P.a[n], P.lk[n], gu);
            r(i, kT) = take && src >= 0 ? g(src, kT) : fma(P.a[n], P.rhs[n], f);
            r(i, kU) = gu;
            r(i, kN) = pos(u, i, 3) == -1 ? f : 0.0;
        }
        for (int i = 0; i < u.np; ++i)
            for (int c : tab.children(i)) {
                r(i, kS) += r(c, kU);
                r(i, kT) -= r(c, kN);
                r(c, kN) = 0.0;
            }
    }
    void up(const TreeUnit &u, Rows r, const Tables &tab) {
        std::vector<int> ch;
        for (int j = 0; j < u.nr; ++j)
            for (int q = tab.get<int32_t>(u.o_rf, j), e = tab.get<int32_t>(u.o_rf, j + 1); q < e; ++q) {
                int p;
                const int row = tab.fold(q, p, ch);
                auto pass = [&](int i, double w) {
                    const double f = w * rcp_d(r(i, kS));
                    r(row, kS) = fma(-w, f, r(row, kS));
                    r(row, kT) = fma(f, r(i, kT), r(row, kT));
                    return f;
                };
                for (int i : ch) pass(i, r(i, kU));
                if (p >= 0) {
                    const double w = r(row, kU), f = pass(p, w);
                    r(p, kN) = w;
                    r(row, kU) = f * r(p, kU);
                }
            }
    }
    static void quotient(Rows from, Rows to, int i) {
        const double s = from(i, kS), f = rcp_d(s);
        const double t = mech::fdiv(from(i, kT), s), x = from(i, kU) * f, n = from(i, kN) * f;
        to(i, kS) = s;
        to(i, kT) = t;
        to(i, kU) = x;
        to(i, kN) = n;
    }
    void down(const TreeUnit &u, Rows r, const Tables &tab) {
        for (int j = u.nr - 1; j >= 0; --j)
            for (int q = tab.get<int32_t>(u.o_re, j), e = tab.get<int32_t>(u.o_re, j + 1); q < e; ++q) {
                int i, p, c;
                tab.elim(q, i, p, c);
                r(i, kT) = fma(r(i, kN), c >= 0 ? r(c, kT) : 0.0, fma(r(i, kU), r(p, kT), r(i, kT)));
            }
    }
    void voltage(const TreeUnit &u, Rows r, bool hand) {
        for (int i = 0; i < u.np; ++i) {
            const int src = pos(u, i, 2);
            if (src >= 0) {
                if (hand) Rows{G, 0}(src, kT) = r(i, kT);
            } else {
                dv.at(pos(u, i, 0)) = r(i, kT);
            }
        }
    }
    const char *block(const TreeUnit &u) const { return &t.block.at(16 * (size_t)u.block); }
    void solve() {
        const size_t rows = l.pos.size() / 4;
        G.assign(32 * rows, (char)0xff);   // a NaN wherever nothing was handed over
        dv.assign(P.N, NAN);
        for (const TreeUnit &u : l.a) {
            std::vector<char> lds(l.lds_a);
            const size_t at = tree_row_bytes(u.np);
            const int up_bytes = tree_up_bytes(u.mode, u.bytes, u.o_re, u.o_fold);
            (void)lds.at(at + up_bytes - 1);
            memcpy(&lds.at(at), block(u), up_bytes);
            Rows r{lds, 0}, out{G, 32 * (size_t)u.p0};
            const Tables tab{lds, (long)at, u};
            assemble(u, r, tab, false);
            if (u.mode == kUnitTop) {
                for (int i = 0; i < u.np; ++i)
                    for (int k : {kS, kT}) out(i, k) = r(i, k);
                continue;
            }
            up(u, r, tab);
            for (int i = 0; i < u.np; ++i) {
                const double t0 = r(i, kT);
                quotient(r, u.mode == kUnitPiece ? out : r, i);
                if (u.mode == kUnitPiece && pos(u, i, 3) != -1) out(i, kT) = t0;
            }
            if (u.mode == kUnitPiece) continue;
            down(u, r, tab);
            voltage(u, r, false);
        }
        for (const auto *units : {&l.top, &l.top_g})
            for (const TreeUnit &u : *units) {
                std::vector<char> lds(units == &l.top ? l.lds_top : 0);
                const size_t at = tree_row_bytes(u.np);
                if (!u.wide) {
                    memcpy(&lds.at(at), block(u), u.bytes);
                    (void)lds.at(at + u.bytes - 1);
                }
                Rows r = u.wide ? Rows{G, 32 * (size_t)u.p0} : Rows{lds, 0};
                const Tables tab{u.wide ? t.block : lds, u.wide ? 16l * u.block : (long)at, u};
                assemble(u, r, tab, true);
                up(u, r, tab);
                for (int i = 0; i < u.np; ++i) quotient(r, r, i);
                down(u, r, tab);
                voltage(u, r, true);
            }
        for (size_t b = 0; b < l.b.size(); b += 2) {
            const TreeUnit &u = l.b[b], &trunk = l.b[b + 1];
            const bool piece = u.mode == kUnitPiece;
            std::vector<char> lds(l.lds_b);
            size_t at = 0;
            Rows x{lds, 0};
            long tab_at = 0;
            if (piece) {
                memcpy(&lds.at(0), &G.at(32 * (size_t)u.p0), 32 * (size_t)u.np);
                at = tree_row_bytes(u.np);
                const int from = u.o_re;
                memcpy(&lds.at(at), block(u) + from, u.bytes - from);
                tab_at = (long)at - from;
                at += u.bytes - from;
                (void)lds.at(at - 1);
            }
            if (!piece || u.solves_trunk) {
                Rows r{lds, at}, g{G, 0};
                const size_t ta = at + tree_row_bytes(trunk.np);
                memcpy(&lds.at(ta), block(trunk), trunk.bytes);
                (void)lds.at(ta + trunk.bytes - 1);
                const Tables tab{lds, (long)ta, trunk};
                for (int i = 0; i < trunk.np; ++i) {
                    const int src = pos(trunk, i, 2), from = src >= 0 ? src : trunk.p0 + i;
                    r(i, kS) = g(from, kS);
                    r(i, kT) = g(from, kT);
                    r(i, kU) = P.g[pos(trunk, i, 0)];
                    r(i, kN) = 0.0;
                }
                up(trunk, r, tab);
                for (int i = 0; i < trunk.np; ++i) quotient(r, r, i);
                down(trunk, r, tab);
                if (!piece) {
                    voltage(u, r, false);
                    continue;
                }
                for (int i = 0; i < u.np; ++i)
                    if (const int row = pos(u, i, 3); row >= 0) x(i, kT) = r(row, kT);
            }
            down(u, x, Tables{lds, tab_at, u});
            voltage(u, x, false);
        }
    }
};

int main() {
    std::mt19937_64 rng(20190507);
    std::uniform_real_distribution<double> uni(0.0, 1.0);
    int bad = 0, cases = 0, by_pieces = 0, alone = 0, wide = 0;
    const int caps[] = {1, 2, 3, 7, 50, 257, 1024, 2416};
    for (int trial = 0; trial < 288; ++trial) {
        const int cap = caps[trial % 8];
        Problem P;
        P.N = 1 + (int)(rng() % (trial < 96 ? 80 : 6000));
        P.parent.resize(P.N);
        for (int i = 0; i < P.N;) {
            const int size = std::min(P.N - i, 1 + (int)(rng() % (trial % 3 ? 6000 : 100))), shape = (int)(rng() % 6);
            const int stem = 1 + size / std::max(1, cap * 3 / 4);
            P.parent[i] = -1;
            for (int j = 1; j < size; ++j)   // random tree, chain, star, short branches off a stem, sections, a trunk of most of a unit
                P.parent[i + j] = i + (shape == 0 ? (int)(rng() % j) : shape == 1 ? j - 1 : shape == 2 ? 0 :
                                       shape == 3 ? (j & 1 ? j - 1 : std::max(0, j - 2)) :
                                       shape == 4 ? (rng() % 8 ? j - 1 : (int)(rng() % j)) : (j - 1) % stem ? j - 1 : 0);
            i += size;
        }
        for (auto *x : {&P.a, &P.lk, &P.g, &P.v, &P.rhs}) x->resize(P.N);
        for (int i = 0; i < P.N; ++i) {
            P.a[i] = 1.0 + uni(rng);
            P.lk[i] = 0.04 + 0.01 * uni(rng);
            P.g[i] = P.parent[i] >= 0 ? uni(rng) : 0.0;
            P.v[i] = -65.0 + uni(rng);
            P.rhs[i] = 0.1 * (uni(rng) - 0.5);
        }
        std::vector<long double> D(P.N), R(P.N), x(P.N);
        for (int i = 0; i < P.N; ++i) {
            D[i] += (long double)P.a[i] * P.lk[i];
            R[i] += (long double)P.a[i] * P.rhs[i];
            if (const int p = P.parent[i]; p >= 0) {
                const long double f = P.g[i] * ((long double)P.v[p] - P.v[i]);
                D[i] += P.g[i];
                D[p] += P.g[i];
                R[i] += f;
                R[p] -= f;
            }
        }
        for (int i = P.N - 1; i >= 0; --i)
            if (const int p = P.parent[i]; p >= 0) {
                D[p] -= P.g[i] * P.g[i] / D[i];
                R[p] += P.g[i] * R[i] / D[i];
            }
        long double big = 0, err = 0;
        for (int i = 0; i < P.N; ++i) {
            x[i] = (R[i] + (P.parent[i] >= 0 ? P.g[i] * x[P.parent[i]] : 0)) / D[i];
            big = std::max(big, std::fabs(x[i]));
        }
        CableHost h;
        TreeSchedule s;
        TreeTables t;
        TreeLaunches l;
        if (!build_cable(P.N, P.parent.data(), cap, h, false).empty()) { ++bad; continue; }
        build_schedule(h, s);
        tree_tables(h, s, t);
        // room beside the largest unit for a large trunk, a small one, or none
        size_t unit = 0;
        for (const TreeUnit &u : t.unit)
            if (!u.wide) unit = std::max(unit, (size_t)tree_row_bytes(u.np) + u.bytes);
        const size_t lds = unit + (size_t)(trial / 8 % 3) * unit / 2;
        tree_launches(h, t, lds, l);
        by_pieces += std::any_of(l.b.begin(), l.b.end(), [](const TreeUnit &u) { return u.solves_trunk; });
        alone += !l.top.empty();
        wide += !l.top_g.empty();
        Solver S{P, t, l, {}, {}};
        S.solve();
        for (int i = 0; i < P.N; ++i) {
            const long double e = std::fabs(S.dv[i] - x[i]);
            err = e <= err ? err : e;   // NaN counts
        }
        if (!(err <= 1e-11L * big) || l.lds_a > lds || l.lds_top > lds || l.lds_b > lds) {
            ++bad;
            std::printf("FAILED trial %d N %d: error %.3Lg of %.3Lg, LDS %zu %zu %zu of %zu\n", trial, P.N, err, big, l.lds_a,
                        l.lds_top, l.lds_b, lds);
        }
        ++cases;
    }
    if (by_pieces < 10 || alone < 10 || wide < 10) ++bad;
    std::printf("%d cases, %d with trunks solved by pieces, %d alone, %d in global memory, %d failed\n", cases, by_pieces, alone,
                wide, bad);
    return bad == 0 ? 0 : 1;
}
