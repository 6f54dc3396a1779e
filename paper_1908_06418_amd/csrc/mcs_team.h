// What the wavefronts of a workgroup of the lane kernel share in LDS, and the
// transitions on it that several of them may make at once.  Ops: relaxed
// atomics, the kernel's on LDS at workgroup scope.
#pragma once

#include "mcs_layout.h"

namespace mcs {

constexpr int kTeamStats = 10;
struct Team {
    unsigned hungry;      // bit w: wavefront w waits for a frame
    unsigned done;        // the search is over
    unsigned looked;      // ticks of the last look at the rings (low word)
    unsigned idle;        // 1: the workgroup is counted as idle
    unsigned full[16];    // 1: a frame for wavefront w is in its stack, its
    unsigned long long box[16][6];  //    header here (x, y; unit; partners)
    // work units: one instance each, on one or more of the wavefronts
    unsigned ref[16];     // 0: free; 1 + the wavefronts on it
    int inst[16];
    int inc[16];          // the incumbent as last seen or raised
    unsigned seen[16];    // ticks of the last look at it
    unsigned long long nodes[16];  // counted by wavefronts that have left
    unsigned left;        // wavefronts that have not ended
    int max_stack;
    unsigned long long st[kTeamStats];  // the wavefronts' statistics
};
static_assert(sizeof(Team) <= kLaneTeamBytes, "the host leaves room for it in LDS");

// A wavefront without work leaves the unit, with `mine` nodes counted on it.
// True for the last one: it hands in *total and frees the unit.
template <class Ops>
[[gnu::always_inline]] constexpr bool team_leave(Team &T, int unit, unsigned long long mine, unsigned long long *total) {
    Ops::add(&T.nodes[unit], mine);
    if (Ops::add(&T.ref[unit], ~0u) != 2u)
        return false;
    *total = Ops::swap(&T.nodes[unit], 0ull);
    return true;
}
// A wavefront stops with work left.  It stays counted in the unit, so that
// nobody ends it.
template <class Ops>
[[gnu::always_inline]] constexpr void team_stop(Team &T, int unit, unsigned long long mine) {
    Ops::add(&T.nodes[unit], mine);
}
// The workgroup's last wavefront, once all others have ended: the nodes of a
// unit that nobody has handed in (wavefronts that left it after one stopped
// there are not its last).
template <class Ops>
[[gnu::always_inline]] constexpr unsigned long long team_rest(Team &T, int unit) {
    return Ops::swap(&T.nodes[unit], 0ull);
}
// Whether the workgroup is without work, said by any of its wavefronts: what to
// add to its XCD's count.
template <class Ops>
[[gnu::always_inline]] constexpr int team_idle(Team &T, unsigned idle) {
    return (int)idle - (int)Ops::swap(&T.idle, idle);
}

}  // namespace mcs
