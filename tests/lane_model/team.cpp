// The transitions of mcs_team.h on the CPU, in every order in which some of a
// workgroup's wavefronts stop with work left and others run dry.
#include <algorithm>
#include <cstdio>
#include <cstring>
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
    std::printf("orders %d bad %d\n", orders, bad);
    return bad != 0;
}
