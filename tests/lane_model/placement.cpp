// Replays, on the CPU, where a wavefront of the kernel with a search in every
// lane puts its frames: 64 searches of one instance, each with its own part of
// cap entries, and one worst-case area behind them that a single search at a
// time may continue into.  The rule that sends a child there is the library's
// (lane_enters_area, mcs_layout.h); the arbitration is the kernel's.  Fails
// if two searches are in the area together, or if an entry past a part's end
// is written by a search that did not enter the area.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "mcs_layout.h"

typedef unsigned __int128 W;
static int popc(W x) {
    return __builtin_popcountll((uint64_t)x) + __builtin_popcountll((uint64_t)(x >> 64));
}
static int ctz(W x) {
    return (uint64_t)x ? __builtin_ctzll((uint64_t)x) : 64 + __builtin_ctzll((uint64_t)(x >> 64));
}

struct Cls {
    W L, R;
};
struct Frame {
    std::vector<Cls> c;
    int base = 0, d = 0, v = 0, sel = 0, bound = 0;
    bool fresh = true, unm = false;
    W rest = 0;
};
struct Pair {
    int n, bound = 0;
    std::vector<W> g, h;
    std::vector<Cls> root;
};

static std::vector<W> graph(std::mt19937_64 &rng, int n, double p, int labels, std::vector<int> &lab) {
    std::vector<W> a(n, 0), b(n, 0);
    for (int i = 0; i < n; i++)
        for (int j = i + 1; j < n; j++)
            if ((double)(rng() >> 11) * 0x1.0p-53 < p) {
                a[i] |= (W)1 << j;
                a[j] |= (W)1 << i;
            }
    std::vector<int> ord(n), at(n), l(n);
    for (int i = 0; i < n; i++)
        ord[i] = i;
    std::stable_sort(ord.begin(), ord.end(), [&](int x, int y) { return popc(a[x]) > popc(a[y]); });
    for (int i = 0; i < n; i++)
        at[ord[i]] = i;
    lab.resize(n);
    for (int i = 0; i < n; i++) {
        lab[i] = (int)(rng() % (uint64_t)labels);
        for (W x = a[ord[i]]; x; x &= x - 1)
            b[i] |= (W)1 << at[ctz(x)];
    }
    return b;
}

static Pair make(std::mt19937_64 &rng, int n, double p, double share) {
    Pair q;
    q.n = n;
    const int labels = std::max(1, (int)std::ceil(share * n));
    std::vector<int> lg, lh;
    q.g = graph(rng, n, p, labels, lg);
    q.h = graph(rng, n, p, labels, lh);
    for (int l = 0; l < labels; l++) {
        Cls c{0, 0};
        for (int i = 0; i < n; i++) {
            c.L |= (W)(lg[i] == l) << i;
            c.R |= (W)(lh[i] == l) << i;
        }
        if (c.L && c.R) {
            q.root.push_back(c);
            q.bound += std::min(popc(c.L), popc(c.R));
        }
    }
    return q;
}

struct Wave {
    const Pair &q;
    const int he, cap;
    std::vector<Frame> st[64];
    int inc = 0;
    long long nodes = 0, at_cap = 0, entered = 0, waited = 0;
    bool bad = false;

    Wave(const Pair &p, int word, int c) : q(p), he(mcs::lane_hdr_entries(word)), cap(c) {
        Frame f;
        f.c = q.root;
        f.bound = q.bound;
        st[0].push_back(f);
    }
    static bool open(const Frame &f) { return f.rest || f.unm || f.fresh; }
    bool in_area(int l) const { return !st[l].empty() && st[l].back().base >= cap; }

    // Brings the top frame to a partner to evaluate; false: the lane is idle.
    bool ready(int l) {
        auto &s = st[l];
        while (!s.empty()) {
            Frame &f = s.back();
            if (f.bound <= inc) {
                s.pop_back();
            } else if (f.fresh) {
                if (f.c.empty()) {
                    s.pop_back();
                    continue;
                }
                int key = 1 << 30;
                for (size_t k = 0; k < f.c.size(); k++) {
                    const int x = (std::max(popc(f.c[k].L), popc(f.c[k].R)) << 8) | ctz(f.c[k].L);
                    if (x < key)
                        key = x, f.sel = (int)k;
                }
                f.v = key & 255;
                f.rest = f.c[f.sel].R;
                f.fresh = false;
                f.unm = true;
            } else if (f.rest) {
                return true;
            } else if (f.unm) {
                nodes++;
                f.unm = false;
                Cls &c = f.c[f.sel];
                f.bound -= popc(c.L) <= popc(c.R);
                c.L &= ~((W)1 << f.v);
                if (!c.L)
                    f.c.erase(f.c.begin() + f.sel);
                f.fresh = true;
            } else {
                s.pop_back();
            }
        }
        return false;
    }
    void step() {
        struct Child {
            bool found = false;
            int w = 0;
            Frame f;
        } ch[64];
        for (int l = 0; l < 64; l++) {
            if (!ready(l))
                continue;
            Frame &f = st[l].back();
            const int w = ctz(f.rest);
            f.rest &= f.rest - 1;
            nodes++;
            Frame x;
            x.d = f.d + 1;
            x.bound = x.d;
            for (const Cls &c : f.c) {
                const W cl = c.L & ~((W)1 << f.v), cr = c.R & ~((W)1 << w);
                for (int e = 0; e < 2; e++) {
                    const Cls p{e ? cl & q.g[f.v] : cl & ~q.g[f.v], e ? cr & q.h[w] : cr & ~q.h[w]};
                    if (p.L && p.R) {
                        x.c.push_back(p);
                        x.bound += std::min(popc(p.L), popc(p.R));
                    }
                }
            }
            if (x.bound > inc) {
                ch[l].found = true;
                ch[l].w = w;
                ch[l].f = x;
            }
        }
        int owner = -1, first = -1;
        for (int l = 0; l < 64; l++) {
            if (in_area(l))
                owner = l;
            if (!ch[l].found)
                continue;
            const Frame &f = st[l].back();
            const int nb = f.base + he + (int)f.c.size(), need = he + ch[l].f.bound - f.d - 1;
            if (first < 0 && mcs::lane_enters_area(f.base, nb, need, cap))
                first = l;
        }
        for (int l = 0; l < 64; l++) {
            if (!ch[l].found)
                continue;
            Frame &f = st[l].back();
            int nb = f.base + he + (int)f.c.size();
            const int need = he + ch[l].f.bound - f.d - 1;
            if (f.base < cap && nb == cap)
                at_cap++;
            if (mcs::lane_enters_area(f.base, nb, need, cap)) {
                if (owner >= 0 || l != first) {
                    f.rest |= (W)1 << ch[l].w;
                    nodes--;
                    waited++;
                    continue;
                }
                entered++;
                nb = cap;
            } else if (f.base < cap && nb + he + (int)ch[l].f.c.size() > cap) {
                bad = true;  // written past the lane's own part
            }
            inc = std::max(inc, ch[l].f.d);
            if (ch[l].f.c.empty())
                continue;
            ch[l].f.base = nb;
            st[l].push_back(ch[l].f);
        }
        int in = 0;
        for (int l = 0; l < 64; l++)
            in += in_area(l);
        bad = bad || in > 1;
        // idle lanes take the lowest open frames below the others' tops
        for (int t = 0, v = 0; t < 64 && v < 64; t++) {
            if (!st[t].empty())
                continue;
            for (; v < 64 && st[t].empty(); v++)
                for (size_t k = 0; k + 1 < st[v].size(); k++) {
                    Frame &f = st[v][k];
                    if (!open(f) || f.bound <= inc)
                        continue;
                    Frame x = f;
                    x.base = 0;
                    f.rest = 0;
                    f.unm = f.fresh = false;
                    st[t].push_back(x);
                    break;
                }
        }
    }
    bool busy() const {
        return std::any_of(st, st + 64, [](const std::vector<Frame> &s) { return !s.empty(); });
    }
};

// args: bits, n, p, labels per vertex, pairs, node limit per pair, cap
int main(int argc, char **argv) {
    if (argc != 8)
        return 2;
    const int bits = atoi(argv[1]), n = atoi(argv[2]), pairs = atoi(argv[5]), cap = atoi(argv[7]);
    const double p = atof(argv[3]), share = atof(argv[4]);
    std::mt19937_64 rng(7);
    long long at_cap = 0, entered = 0, waited = 0;
    int bad = 0;
    for (int i = 0; i < pairs; i++) {
        const Pair q = make(rng, n, p, share);
        Wave w(q, bits / 8, cap);
        while (w.busy() && w.nodes < atoll(argv[6]))
            w.step();
        at_cap += w.at_cap;
        entered += w.entered;
        waited += w.waited;
        bad += w.bad;
    }
    std::printf("at_cap %lld entered %lld waited %lld bad %d\n", at_cap, entered, waited, bad);
    return 0;
}
