// The transitions of mcs_team.h on the CPU, in every order in which some of a
// workgroup's wavefronts stop with work left and others run dry.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <thread>
#include <vector>

#include "mcs_team.h"

struct Ops {
    template <typename T>
    static T add(T *p, T x) {
        return __atomic_fetch_add(p, x, __ATOMIC_RELAXED);
    }
    template <typename T>
    static T swap(T *p, T x) {
        return __atomic_exchange_n(p, x, __ATOMIC_RELAXED);
    }
};

// Four wavefronts that say at once, again and again, whether there is work:
// the changes they hand in sum to what was said last.
static int idle_counts() {
    int bad = 0;
    for (int round = 0; round < 20; round++) {
        mcs::Team T;
        std::memset(&T, 0, sizeof T);
        long long count = 0;
        std::vector<std::thread> ws;
        for (unsigned w = 0; w < 4; w++)
            ws.emplace_back([&, w] {
                unsigned x = 12345u + w;
                for (int i = 0; i < 100000; i++) {
                    x = x * 1664525u + 1013904223u;
                    Ops::add(&count, (long long)mcs::team_idle<Ops>(T, x >> 31));
                }
            });
        for (std::thread &t : ws)
            t.join();
        bad += count != (long long)T.idle;
    }
    return bad;
}

int main() {
    int orders = 0, bad = 0;
    for (int stops = 0; stops < 16; stops++) {  // which of four wavefronts stop
        std::vector<int> ord = {0, 1, 2, 3};
        do {
            mcs::Team T;
            std::memset(&T, 0, sizeof T);
            const int unit = 5;
            T.ref[unit] = 1 + 4;
            T.left = 4;
            unsigned long long in = 0, sum = 0;
            bool ended = false;
            for (int w : ord) {
                const unsigned long long mine = 100ull << (8 * w);
                sum += mine;
                if ((stops >> w) & 1) {
                    mcs::team_stop<Ops>(T, unit, mine);
                } else {
                    unsigned long long total = 0;
                    if (mcs::team_leave<Ops>(T, unit, mine, &total)) {
                        ended = true;
                        in += total;
                    }
                }
                if (Ops::add(&T.left, ~0u) == 1u)
                    for (int u = 0; u < 16; u++)
                        in += mcs::team_rest<Ops>(T, u);
            }
            orders++;
            bad += in != sum || ended != (stops == 0);
        } while (std::next_permutation(ord.begin(), ord.end()));
    }
    const int miscounted = idle_counts();
    std::printf("orders %d bad %d idle %d\n", orders, bad, miscounted);
    bad += miscounted;
    return bad != 0;
}
