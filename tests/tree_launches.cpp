// tree_launches.cpp -- the launches of a cable solve on the CPU
// (tests/test_tree_launches.py builds and runs it).
//
// tests/tree_schedule.cpp replays the rounds of each unit by itself.  Here the
// launches run as they are planned (tree_launches): every workgroup has an LDS
// of the planned size and no more, finds its tables and rows in it where the
// kernels put them, and reads other units' rows only through the positions and
// the memory between the launches.  Trees whose trunks are solved by their
// pieces, in LDS in a launch of their own, and in global memory must all give
// the solution of Hines elimination in long double, with a round's records in
// either order (a place that one record writes and another of its round reads
// makes the two differ).
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

// A workgroup's LDS, or global memory: rows of L, T, U, S and a unit's tables.
struct Rows {
    std::vector<char> &mem;
    size_t at;
    double &operator()(int i, int k) {
        const size_t o = at + 32 * (size_t)i + 8 * k;
        (void)mem.at(o + 7);
        return *reinterpret_cast<double *>(&mem.at(o));
    }
};
enum { kL, kT, kU, kS };
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
    // has the row a child left when it is eliminated?
    bool kid(int i) const { return get<uint32_t>(u.o_kid, i / 32) >> (i % 32) & 1; }
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
    bool reverse;
    std::vector<char> G;
    std::vector<double> dv, N;   // N: of a trunk in global memory

    int pos(const TreeUnit &u, int i, int k) const { return l.pos.at(4 * (size_t)(u.p0 + i) + k); }
    void assemble(const TreeUnit &u, Rows r, const Tables &tab, bool take) {
        Rows g{G, 0};
        std::vector<double> S(u.np), flow(u.np);
        if (u.wide) N.assign(u.np, 0.0);
        for (int i = 0; i < u.np; ++i) {
            const int n = pos(u, i, 0), p = pos(u, i, 1), src = pos(u, i, 2);
            flow[i] = P.g[n] * (P.v[p >= 0 ? p : n] - P.v[n]);
            r(i, kL) = take && src >= 0 ? g(src, kL) : P.a[n] * P.lk[n];
            r(i, kT) = take && src >= 0 ? g(src, kT) : fma(P.a[n], P.rhs[n], flow[i]);
            r(i, kU) = P.g[n];
        }
        for (int i = 0; i < u.np; ++i) {
            r(i, kS) = r(i, kL) + r(i, kU);
            for (int c : tab.children(i)) {
                r(i, kS) += r(c, kU);
                r(i, kT) -= flow[c];
            }
        }
    }
    // A round's records in order or, as threads may, in reverse; at most two for
    // each of the threads that a launch has.  N comes after the round in LDS, where
    // it takes the place of S.
    void up(const TreeUnit &u, Rows r, const Tables &tab, size_t rows) {
        std::vector<int> ch;
        std::vector<std::pair<int, double>> next;
        const int threads = (int)std::min<size_t>(1024, std::max<size_t>(64, (rows / 2 + 63) / 64 * 64));
        for (int j = 0; j < u.nr; ++j) {
            const int lo = tab.get<int32_t>(u.o_rf, j), hi = tab.get<int32_t>(u.o_rf, j + 1);
            if (!u.wide && (hi - lo > 2 * threads || u.np > 3 * threads)) r(0, kL) = NAN;
            for (int n = lo; n < hi; ++n) {
                int p;
                const int row = tab.fold(reverse ? lo + hi - 1 - n : n, p, ch);
                double L = r(row, kL), T = r(row, kT), S = r(row, kS), U = r(row, kU);
                auto pass = [&](int i, double w) {
                    const double f = w * rcp_d(r(i, kS));
                    S = fma(-w, f, S);
                    L = fma(f, r(i, kL), L);
                    T = fma(f, r(i, kT), T);
                    return f;
                };
                for (int i : ch) pass(i, r(i, kU));
                if (p >= 0) {
                    (u.wide ? N[p] : (next.push_back({p, 0.0}), next.back().second)) = U;
                    U = pass(p, U) * r(p, kU);
                }
                r(row, kL) = L;
                r(row, kT) = T;
                r(row, kU) = U;
                r(row, kS) = S;
            }
            for (auto &x : next) r(x.first, kS) = x.second;
            next.clear();
        }
    }
    void quotient(const TreeUnit &u, Rows from, Rows to, const Tables &tab, int i) {
        const double n = u.wide ? N[i] : tab.kid(i) ? from(i, kS) : 0.0;
        const double l = from(i, kL), s = l + (from(i, kU) + n), f = rcp_d(s);
        const double t = mech::fdiv(from(i, kT), s), x = from(i, kU) * f;
        to(i, kL) = l;
        to(i, kT) = t;
        to(i, kU) = x;
        to(i, kS) = n * f;
    }
    void down(const TreeUnit &u, Rows r, const Tables &tab) {
        for (int j = u.nr - 1; j >= 0; --j)
            for (int q = tab.get<int32_t>(u.o_re, j), e = tab.get<int32_t>(u.o_re, j + 1); q < e; ++q) {
                int i, p, c;
                tab.elim(q, i, p, c);
                r(i, kT) = fma(r(i, kS), c >= 0 ? r(c, kT) : 0.0, fma(r(i, kU), r(p, kT), r(i, kT)));
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
            const int up_bytes = tree_up_bytes(u.mode, u.bytes, u.o_re, u.o_kid);
            (void)lds.at(at + up_bytes - 1);
            memcpy(&lds.at(at), block(u), up_bytes);
            Rows r{lds, 0}, out{G, 32 * (size_t)u.p0};
            const Tables tab{lds, (long)at, u};
            assemble(u, r, tab, false);
            if (u.mode == kUnitTop) {
                for (int i = 0; i < u.np; ++i)
                    for (int k : {kL, kT, kU, kS}) out(i, k) = r(i, k);
                continue;
            }
            up(u, r, tab, l.rows_a);
            for (int i = 0; i < u.np; ++i) {
                const double t0 = r(i, kT);
                quotient(u, r, u.mode == kUnitPiece ? out : r, tab, i);
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
                up(u, r, tab, l.rows_a);
                for (int i = 0; i < u.np; ++i) quotient(u, r, r, tab, i);
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
                    const int src = pos(trunk, i, 2), own = trunk.p0 + i, from = src >= 0 ? src : own;
                    r(i, kL) = g(from, kL);
                    r(i, kT) = g(from, kT);
                    r(i, kU) = g(own, kU);
                    r(i, kS) = src >= 0 ? g(src, kL) + g(own, kU) : g(own, kS);
                }
                up(trunk, r, tab, l.rows_b);
                for (int i = 0; i < trunk.np; ++i) quotient(trunk, r, r, tab, i);
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

static std::vector<long double> reference(const Problem &P) {
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
    for (int i = 0; i < P.N; ++i) x[i] = (R[i] + (P.parent[i] >= 0 ? P.g[i] * x[P.parent[i]] : 0)) / D[i];
    return x;
}

// Hines elimination, leaves to root and back, in double: a row's own terms first,
// a child's coupling with what it folds.
static std::vector<double> hines(const Problem &P) {
    std::vector<double> D(P.N), R(P.N), x(P.N);
    for (int i = 0; i < P.N; ++i) {
        const int p = P.parent[i];
        const double k = P.g[i] / P.a[i];
        D[i] = P.lk[i] + k;
        R[i] = fma(k, p >= 0 ? P.v[p] - P.v[i] : 0.0, P.rhs[i]);
    }
    for (int i = P.N - 1; i >= 0; --i)
        if (const int p = P.parent[i]; p >= 0) {
            const double k = P.g[i] / P.a[p], f = k / D[i];
            D[p] += fma(-f, P.g[i] / P.a[i], k);
            R[p] += fma(f, R[i], -(k * (P.v[p] - P.v[i])));
        }
    for (int i = 0; i < P.N; ++i) x[i] = fma(P.g[i] / P.a[i], P.parent[i] >= 0 ? x[P.parent[i]] : 0.0, R[i]) / D[i];
    return x;
}

// The rounding of dv is no larger than Hines elimination's: rms over branched
// cells of 1000 compartments at one voltage with random currents, at the axial
// conductances of micrometre-thick dendrites and at ten times those.
static int rounding() {
    std::mt19937_64 rng(20190508);
    std::uniform_real_distribution<double> uni(0.0, 1.0);
    int bad = 0;
    for (double scale : {1.0, 10.0})
        for (int cap : {256, 1024}) {
            Problem P;
            P.N = 40000;
            for (int first = 0; first < P.N; first += 1000)
                for (int j = 0, left = 0; j < 1000; ++j) {
                    const int at = left > 0 ? j - 1 : (int)(rng() % std::max(1, j));
                    left = left > 0 ? left - 1 : (int)(rng() % 14);
                    const double diam = 0.5 + 2.5 * uni(rng), len = 10.0 + 20.0 * uni(rng);
                    P.parent.push_back(j ? first + at : -1);
                    P.a.push_back(0.0314159265 * diam * len);
                    P.g.push_back(j ? scale * 0.785398163 * diam * diam / len : 0.0);
                    P.lk.push_back(0.0415 + 1e-3 * uni(rng));
                    P.v.push_back(-65.0);
                    P.rhs.push_back(0.02 * (uni(rng) - 0.5));
                }
            CableHost h;
            TreeSchedule s;
            TreeTables t;
            TreeLaunches l;
            if (!build_cable(P.N, P.parent.data(), cap, h, false).empty()) return 1;
            build_schedule(h, s);
            tree_tables(h, s, t);
            tree_launches(h, t, 150000, l);
            Solver S{P, t, l, false, {}, {}, {}};
            S.solve();
            const std::vector<long double> x = reference(P);
            const std::vector<double> y = hines(P);
            long double e = 0, f = 0;
            for (int i = 0; i < P.N; ++i) {
                e += (S.dv[i] - x[i]) * (S.dv[i] - x[i]);
                f += (y[i] - x[i]) * (y[i] - x[i]);
            }
            const double ratio = (double)std::sqrt(e / f);
            if (!(ratio <= 1.0)) ++bad;
            std::printf("rounding, conductances x%g, units of %d: %.2f of Hines elimination's\n", scale, cap, ratio);
        }
    return bad;
}

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
        const std::vector<long double> x = reference(P);
        long double big = 0, err = 0;
        for (long double y : x) big = std::max(big, std::fabs(y));
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
        Solver S{P, t, l, false, {}, {}, {}}, V{P, t, l, true, {}, {}, {}};
        S.solve();
        V.solve();
        for (int i = 0; i < P.N; ++i) {
            const long double e = std::fabs(S.dv[i] - x[i]);
            err = e <= err ? err : e;   // NaN counts
        }
        if (!(err <= 1e-11L * big) || S.dv != V.dv || l.lds_a > lds || l.lds_top > lds || l.lds_b > lds) {
            ++bad;
            std::printf("FAILED trial %d N %d: error %.3Lg of %.3Lg, LDS %zu %zu %zu of %zu\n", trial, P.N, err, big, l.lds_a,
                        l.lds_top, l.lds_b, lds);
        }
        ++cases;
    }
    if (by_pieces < 10 || alone < 10 || wide < 10) ++bad;
    bad += rounding();
    std::printf("%d cases, %d with trunks solved by pieces, %d alone, %d in global memory, %d failed\n", cases, by_pieces, alone,
                wide, bad);
    return bad == 0 ? 0 : 1;
}
