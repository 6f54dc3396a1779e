// McSplit search with one depth-first search per lane (gfx950).
//
// A wavefront runs 64 searches, one per lane; all 64 advance in lock step
// through the phases of one step (below).  Everything a search keeps -- the
// frame's depth, selected class, v, partners left, bound -- is an ordinary
// vector register, and the classes of its top frame are walked one after
// another by a loop whose trip count is the largest class count of the
// wavefront.  Against one search per 8-lane segment (mcs_seg.hip) the
// per-search bookkeeping, which was most of that kernel's instructions, is
// shared by 64 searches instead of 8, and the Eq. 1 sum needs no reduction:
// it is the loop's own running sum.
//
// What a search node costs here, per class of the frame: two ANDs, four
// population counts, two subtractions, two minima and an add (undirected
// rows of 32 bits; twice the ANDs and counts at 64).  v and w need not be
// struck from the classes for the bound: neither is its own neighbour, so
// both are counted in the part without the edge, on either side once, which
// makes that part's minimum one too large: bound = d + sum instead of
// d + 1 + sum.
//
// Bound: VALU issue, on batches that fill the chip.  The 4,096 pairs of 10 to
// 35 vertices take 7 to 10 VALU instructions a node (28 with segments) and fill
// 85 to 92% of the issue slots, 95% of the lanes holding a search; 43% of the
// lane slots do work, since a loop over classes runs for the wavefront's
// longest frame.  60 pairs of 30 vertices: 425 ms with segments, 86 here; 256
// of 10 to 33: 636 and 166.  What is left of a small search is a chain of steps of
// about 1 us: one pair of 16 vertices takes 3.6 ms with segments, 0.5 here.
//
// All lanes of a wavefront work on one instance, so its incumbent is a
// scalar and its adjacency rows (up to 64 vertices) are in LDS once.
//
// Memory of a search: a stack of entries of one class each; a frame is a
// header (lane_hdr_entries) and its classes.  The stack's upper end is in LDS,
// a ring of rc entries per lane (entry e in slot e mod rc): a frame is
// created, split for its partners and returned to there, and an entry is
// written to HBM only when a deeper one needs its slot.  Most of a search's
// steps stay near the leaves, within the two to four frames that the ring
// holds.  In HBM a lane's part has room for cap entries; the wavefront has
// one more area for the worst case, m(m+1)/2 classes and m + 1 headers, which
// one lane at a time may continue into when its own part is full (the others
// wait with the child that did not fit, or go on with other work).
//
// One step, for the lanes that need each phase:
//   pop       -- the top frame has nothing left: return to the parent;
//   unmatched -- its partners are done: bound the "v unmatched" child;
//   fetch     -- a frame returned to that has left the ring comes back;
//   select    -- a new frame (or one that has just lost v) chooses its class
//                and v;
//   evaluate  -- the next two partners w: split and bound;
//   descend   -- the surviving child's non-empty parts become the top frame.
//
// Work sharing, on three levels.  Idle lanes take whole frames from busy
// lanes of their wavefront, all of them at once (steal()): the lowest open
// frame of the lanes where it is shallowest, or (undirected rows of up to 64
// bits) of those whose top frame has the highest bound.  A wavefront with
// no work raises its bit in the workgroup's LDS; a busy one that sees it
// writes a frame straight into the idle one's stack (feed()).  Between
// workgroups frames travel as records through the per-XCD rings of
// mcs_layout.h; only one idle wavefront of a workgroup looks there at a time.
// Each costs one L2-wide release and one acquire, so that the other two levels
// carry most of the frames.  A work unit, for the termination counts, is one instance on one
// wavefront, however many of its lanes work on it.
#include "mcs_device.h"
#include "mcs_policy.h"
#include "mcs_team.h"

namespace mcs {

namespace {

// Rounds of pop and unmatched per step: half of the unmatched children are
// pruned and their lanes pop on (two rounds: the same time within 2%, four
// too).
constexpr int kPops = 3;
// Class reads in flight per lane (narrow rows; 2 with wide ones).
constexpr int kReads = 4;
// Idle lanes look for frames in their wavefront once there are so many, or
// after so many steps (8 to 28 lanes: within 3%).
constexpr int kIdleLanes = 12, kStealSteps = 8;
// Frames may lie so much deeper than the shallowest open one to be taken, or
// their lanes' bounds so much below the highest (steal()): with 0 too few
// lanes are served (six pairs of 30 vertices one by one 53 ms); 2 to 5 take the
// same time within 5%.
constexpr int kStealSpan = 9, kStealBounds = 5;
// A wavefront feeds waiting siblings once every kFeedSteps while it is rich
// (so many lanes busy), and now and then anyway.  Feeding at every step cuts
// the work into units of a few nodes: twice the time on small searches.
constexpr int kFeedSteps = 4, kFeedRich = 48, kFeedAnyway = 64;
// A waiting wavefront whose siblings can feed it looks at the rings so much
// less often.
constexpr unsigned kFedGap = 16;

// With a node limit or a dead-end forecast a wavefront hands its nodes in after
// so many (fewer for small ones: held_back()), or so many steps.  Handed in at
// every check, every four steps, a
// limit that is never met cost 60 pairs of 30 vertices 98 ms instead of 82 and a
// forecast 166; so they take 83 and 85.
constexpr int kFlushNodes = 1000;
constexpr unsigned kFlushSteps = 128;

// Flags of a search's top frame.
constexpr int kUnm = 1;        // the "v unmatched" child is still to do
constexpr int kLe = 2;         // |L_sel| <= |R_sel|: that child's bound is one lower
constexpr int kOne = 4;        // |L_sel| == 1: its class empties with v
constexpr int kSel = 8;        // class and v are to be chosen
constexpr int kPatch = 16;     // (with kSel) v is to be taken out of the selected class first
constexpr int kRow = 32;       // v's G rows are to be loaded
constexpr int kBig = 8;        // (saved headers) the child frame starts the worst-case area
constexpr int kPolV = 64;      // the policy has yet to choose v,
constexpr int kPolW = 128;     // to put the partners in order
constexpr int kSaved = kUnm | kLe | kOne;

constexpr unsigned kErrMapping = 2;  // codes of DevGlobals::error
constexpr unsigned kErrStack = 3;
constexpr unsigned kErrRecord = 1;

typedef unsigned long long u64w;
typedef u64w v2u64 __attribute__((ext_vector_type(2)));
typedef v2u64 v2u64_a8 __attribute__((aligned(8)));
template <typename T>
using lds_ptr = __attribute__((address_space(3))) T *;
// An HBM access whose base is wave-uniform and whose offset is 32-bit.
template <typename T>
using glb_ptr = __attribute__((address_space(1))) T *;

// The launch parameters where the kernel got them: scalar loads, so that a
// field that is needed now and then takes no register in between.
using KernArgs = __attribute__((address_space(4))) SearchParams;

// Lane `from`'s x (every lane of the wavefront active).
DEV int shfl_any(int x, int from) { return __builtin_amdgcn_ds_bpermute(from << 2, x); }

template <typename T>
DEV T ld_wg(T *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
template <typename T>
DEV void st_wg(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
struct WgOps {
    template <typename T>
    DEV T add(T *p, T x) {
        return __hip_atomic_fetch_add(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    template <typename T>
    DEV T swap(T *p, T x) {
        return __hip_atomic_exchange(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
};

}  // namespace

template <typename W, bool DIR, bool POL>
struct LaneSearch {
    static constexpr int NB = bits_of<W>();
    static constexpr int NR = DIR ? 4 : 2;                  // row sets, and parts of a class
    static constexpr int EB = 2 * (int)sizeof(W);           // bytes of a stack entry: one class
    static constexpr int EW = EB / 8;                       // its 64-bit words
    static constexpr int HE = lane_hdr_entries((int)sizeof(W));  // entries of a frame header
    static constexpr int NP = EB >= 16 ? EB / 16 : 1;       // 16-byte pieces of an entry
    static constexpr bool LROWS = sizeof(W) <= 8;           // rows in LDS

    static_assert(!(POL && sizeof(W) > 8), "the policy takes rows of at most 64 bits");

    struct Ent {
        u64w w[EW];
    };
    // A frame header: two 32-bit words and the partners left.
    //   x: base of the frame below (16 bits) | K << 16 | d << 24
    //   y: v | sel << 8 | bound << 16 | flags << 24
    struct Hdr {
        uint32_t x, y;
        W r;
    };

    const KernArgs &P;
    Team &T;
    int cap, rc, reprune, arows;
    float rinv;          // 1 / rc
    int lane, wv;
    uint32_t stride, map_bytes, big_off, big_cap;
    glb_ptr<char> wst;   // the wavefront's stacks in HBM
    lds_ptr<char> lbuf;  // the wavefront's rings: [rc][64 lanes], NP planes
    lds_ptr<W> lrow;     // (up to 64 vertices) the instance's rows: [NR][arows]
    const W *grow;       // the instance's rows in HBM: [NR][NB]

    // ---- per-lane state ----
    int t, base, pbase, bslot, K, d, v, sel, bound, flags;
    int lo_t, lo_base;   // the lowest frame that may still have work
    int wlo, wslot;      // the ring's lowest entry, and its slot
    W rrem, go, gi;
    uint32_t c_child, c_unm, c_ncls, c_pushed;  // since the last flush
    int max_used;

    // ---- wave-level ----
    int inst, rows_inst, inc, target, inc_slot, twin, dead_on;
    int unit;            // the unit the wavefront works on, or -1
    bool stop, roots_left;
    int my_ring, steal_from, other, since_check;
    unsigned flushed;    // the step of the last flush
    int flush_at;        // nodes that make the next one
    u64w t_start, n_steps, n_lanes, n_don, n_pops, n_busy, n_sleep, n_big;
    u64w n_child, n_ncls, n_pushed;

    __device__ __forceinline__ LaneSearch(const KernArgs &p, Team &tm, lds_ptr<char> lds, int wave_in_block,
                          long long wave)
        : P(p), T(tm) {
        lane = lane_id();
        wv = wave_in_block;
        cap = sc(p.cap_classes);
        rc = sc(p.lane_rc);
        rinv = 1.0f / (float)rc;
        reprune = sc(p.reprune);
        arows = sc(p.arows);
        stride = (uint32_t)sc(p.lane_stride);
        map_bytes = (uint32_t)sc(p.lane_map_bytes);
        big_off = 64u * stride;
        big_cap = (uint32_t)sc(p.lane_big);
        wst = (glb_ptr<char>)(p.hstack + (size_t)wave * (size_t)p.hstack_stride);
        lbuf = lds;
        lrow = (lds_ptr<W>)(lds + rc * 64 * EB);
        grow = (const W *)p.adj;
        inst = rows_inst = -1;
        inc = target = inc_slot = dead_on = 0;
        twin = -1;
        unit = -1;
        t = -1;
        base = pbase = bslot = K = d = v = sel = bound = flags = 0;
        lo_t = lo_base = wlo = wslot = 0;
        rrem = go = gi = (W)0;
        c_child = c_unm = c_ncls = c_pushed = 0;
        max_used = 0;
        stop = false;
        roots_left = true;
        my_ring = (int)(blockIdx.x & (kRings - 1));
        steal_from = other = my_ring;
        since_check = 0;
        flushed = 0;
        flush_at = held_back();
        t_start = n_steps = n_lanes = n_don = n_pops = n_busy = n_sleep = n_big = 0;
        n_child = n_ncls = n_pushed = 0;
    }

    // ---- stack entries ----

    // Byte offset of entry e of lane l's stack in HBM: its own part below
    // cap, the wavefront's worst-case area from cap on.
    __device__ __forceinline__ uint32_t at(int l, int e) const {
        return e < cap ? (uint32_t)l * stride + map_bytes + (uint32_t)e * EB
                       : big_off + (uint32_t)(e - cap) * EB;
    }
    // Slot of entry e (e < 2^16 and rc < 2^8: the rounded quotient is exact).
    __device__ __forceinline__ int slot_of(int e) const {
        return e - rc * (int)(((float)e + 0.5f) * rinv);
    }
    __device__ __forceinline__ int wrap(int s) const {  // s < 2 rc
        return (int)umin((uint32_t)s, (uint32_t)(s - rc));
    }
    __device__ __forceinline__ Ent hget(uint32_t off) const {
        Ent x;
        if constexpr (EW == 1) {
            x.w[0] = *(glb_ptr<u64w>)(wst + off);
        } else {
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const v2u64 q = *(glb_ptr<v2u64_a8>)(wst + off + 16 * i);
                x.w[2 * i] = q[0];
                x.w[2 * i + 1] = q[1];
            }
        }
        return x;
    }
    __device__ __forceinline__ void hput(uint32_t off, const Ent &x) const {
        if constexpr (EW == 1) {
            *(glb_ptr<u64w>)(wst + off) = x.w[0];
        } else {
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                v2u64 q = {x.w[2 * i], x.w[2 * i + 1]};
                *(glb_ptr<v2u64_a8>)(wst + off + 16 * i) = q;
            }
        }
    }
    __device__ __forceinline__ Ent lget(int l, int slot) const {
        const int i = slot * 64 + l;
        Ent x;
        if constexpr (EW == 1) {
            x.w[0] = ((lds_ptr<u64w>)lbuf)[i];
        } else {
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const v2u64 q = ((lds_ptr<v2u64>)lbuf)[i + j * 64 * rc];
                x.w[2 * j] = q[0];
                x.w[2 * j + 1] = q[1];
            }
        }
        return x;
    }
    __device__ __forceinline__ void lput(int l, int slot, const Ent &x) const {
        const int i = slot * 64 + l;
        if constexpr (EW == 1) {
            ((lds_ptr<u64w>)lbuf)[i] = x.w[0];
        } else {
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                v2u64 q = {x.w[2 * j], x.w[2 * j + 1]};
                ((lds_ptr<v2u64>)lbuf)[i + j * 64 * rc] = q;
            }
        }
    }
    // Entry e of lane l's stack, whose ring starts at wl.
    __device__ __forceinline__ Ent eget(int l, int e, int wl) const {
        return e >= wl ? lget(l, slot_of(e)) : hget(at(l, e));
    }
    __device__ __forceinline__ void eput(int l, int e, int wl, const Ent &x) const {
        if (e >= wl)
            lput(l, slot_of(e), x);
        else
            hput(at(l, e), x);
    }
    DEV Ent pack(const Cls<W> &c) {
        Ent x;
        if constexpr (EW == 1) {
            x.w[0] = (u64w)(uint32_t)c.L | ((u64w)(uint32_t)c.R << 32);
        } else {
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                x.w[i] = word64(c.L, i);
                x.w[NP + i] = word64(c.R, i);
            }
        }
        return x;
    }
    DEV Cls<W> unpack(const Ent &x) {
        Cls<W> c;
        if constexpr (EW == 1) {
            c.L = (W)(uint32_t)x.w[0];
            c.R = (W)(uint32_t)(x.w[0] >> 32);
        } else {
            uint64_t w[2 * NP];
#pragma unroll
            for (int i = 0; i < 2 * NP; ++i)
                w[i] = x.w[i];
            c.L = from_words<W>(w);
            c.R = from_words<W>(w + NP);
        }
        return c;
    }
    __device__ __forceinline__ Hdr get_hdr(int l, int e, int wl) const {
        Hdr h;
        const Ent a = eget(l, e, wl);
        h.x = (uint32_t)a.w[0];
        h.y = (uint32_t)(a.w[0] >> 32);
        if constexpr (EW == 1) {
            h.r = (W)(uint32_t)eget(l, e + 1, wl).w[0];
        } else {
            uint64_t w[NP];
#pragma unroll
            for (int i = 0; i < NP; ++i)
                w[i] = a.w[1 + i];
            h.r = from_words<W>(w);
        }
        return h;
    }
    __device__ __forceinline__ void put_hdr(int l, int e, int wl, const Hdr &h) const {
        Ent a = {};
        a.w[0] = (u64w)h.x | ((u64w)h.y << 32);
        if constexpr (EW == 1) {
            eput(l, e, wl, a);
            Ent b;
            b.w[0] = (u64w)(uint32_t)h.r;
            eput(l, e + 1, wl, b);
        } else {
#pragma unroll
            for (int i = 0; i < NP; ++i)
                a.w[1 + i] = word64(h.r, i);
            eput(l, e, wl, a);
        }
    }
    __device__ __forceinline__ glb_ptr<uint16_t> map_at(int l) const {
        return (glb_ptr<uint16_t>)(wst + (uint32_t)l * stride);
    }
    // Class k of the lane's top frame.
    __device__ __forceinline__ Cls<W> cget(int k) const { return unpack(eget(lane, base + HE + k, wlo)); }
    __device__ __forceinline__ void cput(int k, const Cls<W> &c) const { eput(lane, base + HE + k, wlo, pack(c)); }

    // f(class k) for each class of the top frames of the lanes that call
    // this, in step.  far: some lane's frame is not all in its ring, or may
    // lose entries to the calls.
    template <typename F>
    __device__ __forceinline__ void each_class(bool far, F f) const {
        if (!far) {
            // (U reads in flight at a time)
            constexpr int U = EW <= 2 ? kReads : 2;
            int s = wrap(bslot + HE);
            for (int k = 0; ballot(k < K) != 0; k += U) {
                Ent x[U];
#pragma unroll
                for (int i = 0; i < U; ++i) {
                    x[i] = lget(lane, s);
                    s = wrap(s + 1);
                }
#pragma unroll
                for (int i = 0; i < U; ++i)
                    if (k + i < K)
                        f(k + i, unpack(x[i]));
            }
        } else {
            for (int k = 0; ballot(k < K) != 0; ++k)
                if (k < K)
                    f(k, cget(k));
        }
    }

    // The ring's lowest entry goes to HBM.
    __device__ __forceinline__ void evict() {
        hput(at(lane, wlo), lget(lane, wslot));
        wlo += 1;
        wslot = wrap(wslot + 1);
    }

    __device__ __forceinline__ W row(int set, int i) const {
        if constexpr (LROWS)
            return lrow[set * arows + i];
        else
            return ld_w(grow + set * NB + i);
    }

    // ---- incumbent ----

    __device__ __forceinline__ int cap_inc(int x) const { return (target > 0 && x >= target) ? 255 : x; }
    __device__ __forceinline__ void set_inc(int x) {
        x = cap_inc(x);
        inc = x > inc ? x : inc;
    }
    // The incumbent, or 255 where the instance needs no more search.
    __device__ __forceinline__ int read_inc() const {
        int g = 0;
        if (lane == 0) {
            g = ld_rlx(&P.inc[inc_slot]);
            if (twin >= 0 && ld_rlx(&P.open[twin]) == 0 && !ld_rlx(&P.dead[twin]))
                g = 255;  // the twin's search already finished
            if (dead_on && ld_rlx(&P.dead[inst]))
                g = 255;  // given up as a dead end
        }
        return rl(g, 0);
    }

    // Lane l's map (size vertex pairs) is a common induced subgraph: raise
    // the instance's incumbent; the wavefront that raised it to `size` writes
    // that size's mapping slot.
    __device__ __forceinline__ void improve(int l, int size) {
        const DevInst di = P.inst[inst];
        if (size > sc(di.nG < di.nH ? (int)di.nG : (int)di.nH)) {
            fail(kErrMapping);  // only from a broken class partition
            return;
        }
        int old = 0;
        if (lane == 0)
            old = a_max(&P.inc[inc_slot], size);
        old = rl(old, 0);
        if (old < size) {
            wave_sync();
            uint16_t *dst = P.maps + di.map_off + size * (size - 1) / 2;
            const glb_ptr<uint16_t> m = map_at(l);
            for (int j = lane; j < size; j += 64)
                dst[j] = m[j];
            const u64w pend = lanes_total(c_child) + lanes_total(c_unm);
            if (lane == 0) {
                a_max64(&P.t_best[inst], ((u64w)size << 48) | (now_ticks() & 0xFFFFFFFFFFFFull));
                a_max64(&P.best_nodes[inst], ld_rlx(&P.nodes[inst]) + pend);
            }
        }
        set_inc(old > size ? old : size);
        if (lane == 0)
            __hip_atomic_fetch_max(&T.inc[unit], inc, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
    }

    // ---- the phases of a step ----

    __device__ __forceinline__ void pop() {
        rrem = (W)0;
        flags = 0;
        t -= 1;
        if (t < 0)
            return;
        base = pbase;
        bslot = slot_of(base);
        const Hdr h = get_hdr(lane, base, wlo);
        pbase = (int)(h.x & 0xFFFFu);
        K = (int)((h.x >> 16) & 0xFFu);
        d = (int)(h.x >> 24);
        v = (int)(h.y & 0xFFu);
        sel = (int)((h.y >> 8) & 0xFFu);
        bound = (int)((h.y >> 16) & 0xFFu);
        if (t < lo_t) {
            lo_t = t;
            lo_base = base;
        }
        if (reprune && bound <= inc)
            return;  // nothing here can beat the incumbent: pop again
        flags = (int)(h.y >> 24) & kSaved;
        rrem = h.r;
        if (rrem != (W)0)
            flags |= kRow;
    }

    // The "v unmatched" child takes its parent's place: only the selected
    // class loses v.
    __device__ __forceinline__ void unmatched() {
        const int ub = bound - ((flags & kLe) ? 1 : 0);
        c_unm += 1;
        if (ub <= inc || ((flags & kOne) && K == 1)) {
            flags = 0;  // pruned, or no class is left
            return;
        }
        bound = ub;
        flags = (flags & kOne) | kSel | kPatch;
    }

    // The top frame (its upper rc entries) back into the ring.
    __device__ __forceinline__ void fetch() {
        const int end = base + HE + K;
        const int lo = end - rc > base ? end - rc : base;
        const int hi = wlo < end ? wlo : end;
        int s = slot_of(lo);
        wlo = lo;
        wslot = s;
        for (int e = lo; ballot(e < hi) != 0; e += 4) {
            // (four loads in flight; past hi the last entry again)
            Ent x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                x[i] = hget(at(lane, e + i < hi ? e + i : hi - 1));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (e + i < hi)
                    lput(lane, s, x[i]);
                s = wrap(s + 1);
            }
        }
    }

    __device__ __forceinline__ void select() {
        if (flags & kPatch) {
            if (flags & kOne) {
                // the class empties on the G side: the last one takes its place
                K -= 1;
                if (sel != K)
                    cput(sel, cget(K));
            } else {
                Cls<W> c = cget(sel);
                c.L = c.L & ~bit_at<W>(v);
                cput(sel, c);
            }
        }
        // the class of smallest max(|L|, |R|), ties to the smallest G vertex
        uint32_t key = 0xFFFFFFFFu;
        each_class(ballot(base < wlo) != 0, [&](int k, const Cls<W> &c) {
            const int nl = popc(c.L), nr = popc(c.R);
            key = umin(key, ((uint32_t)(nl > nr ? nl : nr) << 16) | ((uint32_t)ctz(c.L) << 8) |
                                (uint32_t)k);
        });
        v = (int)((key >> 8) & 0xFFu);
        sel = (int)(key & 0xFFu);
        const Cls<W> c = cget(sel);
        const int nl = popc(c.L), nr = popc(c.R);
        rrem = c.R;
        flags = kUnm | kRow | (nl <= nr ? kLe : 0) | (nl == 1 ? kOne : 0);
        if (POL && d <= P.policy_depth)
            flags |= ((P.policy_mode & 1) ? kPolV : 0) | ((P.policy_mode & 2) ? kPolW : 0);
    }

    // ---- learned branching policy ----

    // A lane's partner orders, 64 bytes for each |M| up to the policy's depth,
    // lie between its mapping and its stack.
    __device__ __forceinline__ uint32_t order_at(int l, int fd) const {
        return (uint32_t)l * stride + map_bytes - 64u * (uint32_t)(P.policy_levels - fd);
    }

    // The policy's choices for the top frame of lane l, made by the whole
    // wavefront: v of the selected class, and the order of its partners.
    // (The network is evaluated for one vertex at a time, a hidden unit per
    // lane: some 10,000 instructions a frame, but only the shallow ones come
    // here, and all of their subtrees' frames take the lanes' own path: 24
    // pairs of 28 vertices take 32 ms, and 147 with a search per wavefront.
    // Deeper orders go to that kernel, by the plan's rule.)
    __device__ __forceinline__ void consult(int l) {
        wave_sync();  // (entries and orders written by other lanes)
        const int fK = rl(K, l), fd = rl(d, l), fsel = rl(sel, l), fb = rl(base, l);
        const int fl = rl(flags, l), fw = rl(wlo, l);
        Cls<W> c;
        c.L = c.R = (W)0;
        if (lane < fK)
            c = unpack(eget(l, fb + HE + lane, fw));
        const W sl = rl(c.L, fsel), sr = rl(c.R, fsel);
        const DevInst di = P.inst[inst];
        const int nl = popc(sl), nr = popc(sr);
#pragma unroll 1
        for (int side = 0; side < 2; ++side) {  // (one copy of the scorer)
            if (!(fl & (side ? kPolW : kPolV)))
                continue;
            const W cand = side ? sr : sl;
            const uint32_t key = score_key(
                policy_score(side, cand, c, fK, fd, nl, nr, sc((int)(side ? di.nH : di.nG))), cand);
            if (side == 0) {
                const uint32_t best = ~wave_min(~key);
                const int x = ctz((uint64_t)ballot(key == best));
                if (lane == l)
                    v = x;
            } else {
                int rank = 0;
                for (W rest = cand; rest; rest &= rest - 1) {
                    const int u = ctz(rest);
                    const uint32_t ku = rl(key, u);
                    rank += ku > key || (ku == key && u < lane) ? 1 : 0;
                }
                if (key != 0)
                    *(glb_ptr<uint8_t>)(wst + order_at(l, fd) + (uint32_t)rank) = (uint8_t)lane;
            }
        }
        if (lane == l)
            flags &= ~(kPolV | kPolW);
        wave_sync();
    }
    // (lane u) vertex u's score as an ordered integer, 0 if it is no candidate
    __device__ __forceinline__ uint32_t score_key(float score, const W &cand) const {
        const uint32_t b = __float_as_uint(score);
        const bool is_cand = lane < NB && ((cand >> (lane & (NB - 1))) & 1);
        return is_cand ? ((b & 0x80000000u) ? ~b : (b | 0x80000000u)) : 0u;
    }
    // Lane u returns the score of vertex u of cand, a class side of a frame
    // with fK classes (lane k holds class k) and fd matches: the features
    // of oracle/policy.py, the network in single precision from the
    // half-precision parameters.
    __device__ __forceinline__ float policy_score(int side, const W &cand, const Cls<W> &c, int fK, int fd, int nl,
                                  int nr, int n) {
        const float inv = 1.f / (float)(n > 0 ? n : 1);
        // this lane's class: its set on this side, and its size bucket
        W mine = (W)0;
        int bsh = 0;
        if (lane < fK) {
            const int x = popc(c.L), y = popc(c.R), m = x < y ? x : y;
            const int bq = m <= 1 ? 0 : m == 2 ? 1 : m <= 4 ? 2 : m <= 8 ? 3 : m <= 16 ? 4 : 5;
            mine = side ? c.R : c.L;
            bsh = 8 * bq;
        }
        const int ul = lane & (NB - 1);
        const bool is_cand = lane < NB && ((cand >> ul) & 1);
        int mydeg = 0;
        if (is_cand)
            mydeg = popc(both_rows(side, ul));
        const int dmax = (int)~wave_min(~(uint32_t)mydeg);
        const uint16_t *w = P.policy;
        float w1[kPolicyF];
#pragma unroll
        for (int f = 0; f < kPolicyF; ++f)
            w1[f] = hf(w[kOffW1 + lane * kPolicyF + f]);
        const float b1 = hf(w[kOffB1 + lane]), b2 = hf(w[kOffB2 + lane]);
        const float w3 = hf(w[kOffW3 + lane]), b3 = hf(w[kOffB3]);
        const uint4 *w2 = (const uint4 *)(w + kOffW2 + lane * kPolicyH);  // 16-byte aligned
        float out = 0.f;
        for (W rest = cand; rest; rest &= rest - 1) {
            const int u = sc((int)ctz(rest));
            const W row = sc(both_rows(side, u));
            const int deg = popc(row);
            // neighbours of u per class, summed per size bucket (each sum is
            // at most deg < 64, so 8-bit fields cannot carry)
            const u64w packed = (u64w)popc(row & mine) << bsh;
            const int lo = wave_sum((int)(uint32_t)packed);
            const int hi = wave_sum((int)(uint32_t)(packed >> 32));
            float x[kPolicyF];
            x[0] = deg * inv;
            x[1] = nl * inv;
            x[2] = nr * inv;
            x[3] = fd * inv;
            x[4] = fK * inv;
            int tot = 0;
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                const int cq = q < 4 ? (lo >> (8 * q)) & 0xFF : (hi >> (8 * (q - 4))) & 0xFF;
                x[6 + q] = cq * inv;
                tot += cq;
            }
            x[5] = tot * inv;
            x[12] = (float)side;
            x[13] = deg == dmax ? 1.f : 0.f;
            x[14] = 0.f;
            x[15] = 1.f;
            float h1 = b1;
#pragma unroll
            for (int f = 0; f < kPolicyF; ++f)
                h1 += w1[f] * x[f];
            h1 = h1 > 0.f ? h1 : 0.f;
            float a2 = b2;
#pragma unroll 1
            for (int i = 0; i < kPolicyH / 8; ++i) {
                const uint4 q = w2[i];
                const uint32_t pk[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    a2 += hf((uint16_t)(pk[e] & 0xFFFFu)) * rlf(h1, 8 * i + 2 * e);
                    a2 += hf((uint16_t)(pk[e] >> 16)) * rlf(h1, 8 * i + 2 * e + 1);
                }
            }
            const float z = b3 + fwave_sum(w3 * (a2 > 0.f ? a2 : 0.f));
            out = lane == u ? z : out;
        }
        return out;
    }
    __device__ __forceinline__ W both_rows(int side, int u) const {
        W r = row(side, u);
        if constexpr (DIR)
            r = r | row(2 + side, u);
        return r;
    }
    // Whether the lane's top frame has its partners in the policy's order.
    __device__ __forceinline__ bool ordered() const {
        return POL && d <= P.policy_depth && (P.policy_mode & 2);
    }
    // The first two partners left in that order (w1 = w0 if there is one).
    __device__ __forceinline__ void next_ordered(int &w0, int &w1) const {
        const int want = popc(rrem) > 1 ? 2 : 1;
        const uint32_t o = order_at(lane, d);
        int found = 0;
        for (int q = 0; q < 8 && ballot(found < want) != 0; ++q) {
            const u64w x = *(glb_ptr<u64w>)(wst + o + 8u * (uint32_t)q);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int u = (int)(x >> (8 * j)) & 0xFF;
                if (found < want && u < NB && ((rrem >> (u & (NB - 1))) & 1)) {
                    w0 = found == 0 ? u : w0;
                    w1 = u;
                    found += 1;
                }
            }
        }
    }

    // Parts of class c for the child (v, w) by adjacency letter; v and w are
    // still in the part without edges.
    __device__ __forceinline__ void split(const Cls<W> &c, const W &ho, const W &hi, W *pl, W *pr) const {
        if constexpr (!DIR) {
            pl[1] = c.L & go;
            pr[1] = c.R & ho;
            pl[0] = c.L ^ pl[1];
            pr[0] = c.R ^ pr[1];
        } else {
            const W lo1 = c.L & go, ro1 = c.R & ho;
            const W lo0 = c.L ^ lo1, ro0 = c.R ^ ro1;
            pl[3] = lo1 & gi;
            pr[3] = ro1 & hi;
            pl[1] = lo1 ^ pl[3];
            pr[1] = ro1 ^ pr[3];
            pl[2] = lo0 & gi;
            pr[2] = ro0 & hi;
            pl[0] = lo0 ^ pl[2];
            pr[0] = ro0 ^ pr[2];
        }
    }

    // The next two partners of v (or the one that is left): their children's
    // Eq. 1 bounds, from one pass over the classes and one count of v's side.
    // The first that survives is (w, b); a second one that is pruned is done
    // too, one that would survive waits until the search is back.
    __device__ __forceinline__ bool evaluate(int &w, int &b) {
        int w0 = ctz(rrem);
        W r1 = rrem & (rrem - (W)1);
        const bool two = r1 != (W)0;
        int w1 = two ? ctz(r1) : w0;
        if constexpr (POL) {
            if (ordered()) {
                next_ordered(w0, w1);
                r1 = rrem & ~bit_at<W>(w0);
            }
        }
        const W ho0 = row(1, w0), ho1 = row(1, w1);
        W hi0 = (W)0, hi1 = (W)0;
        if constexpr (DIR) {
            hi0 = row(3, w0);
            hi1 = row(3, w1);
        }
        int s0 = d, s1 = d;  // (v and w each count once in the selected class: d + 1 - 1)
        each_class(ballot(base < wlo) != 0, [&](int, const Cls<W> &c) {
            if constexpr (!DIR) {
                const int l1 = popc(c.L & go), l0 = popc(c.L) - l1, rt = popc(c.R);
                const int x = popc(c.R & ho0), y = popc(c.R & ho1);
                s0 += (l1 < x ? l1 : x) + (l0 < rt - x ? l0 : rt - x);
                s1 += (l1 < y ? l1 : y) + (l0 < rt - y ? l0 : rt - y);
            } else {
                const W lo1 = c.L & go;
                const int l3 = popc(lo1 & gi), l1 = popc(lo1) - l3, l2 = popc(c.L & gi) - l3;
                const int l0 = popc(c.L) - l1 - l2 - l3, rt = popc(c.R);
                const auto add = [&](const W &ho, const W &hi, int &s) {
                    const W ro1 = c.R & ho;
                    const int r3 = popc(ro1 & hi), q1 = popc(ro1) - r3, q2 = popc(c.R & hi) - r3;
                    const int q0 = rt - q1 - q2 - r3;
                    s += (l0 < q0 ? l0 : q0) + (l1 < q1 ? l1 : q1) + (l2 < q2 ? l2 : q2) +
                         (l3 < r3 ? l3 : r3);
                };
                add(ho0, hi0, s0);
                add(ho1, hi1, s1);
            }
        });
        const bool f0 = s0 > inc, f1 = two && s1 > inc;
        const bool second = two && !(f0 && f1);  // it is done as well
        rrem = !second ? r1 : POL ? r1 & ~bit_at<W>(w1) : r1 & (r1 - (W)1);
        c_child += second ? 2u : 1u;
        c_ncls += (uint32_t)(second ? 2 * K : K);
        w = f0 ? w0 : w1;
        b = f0 ? s0 : s1;
        return f0 || f1;
    }

    // The child (v, w) of bound b becomes the top frame: its classes with
    // both sides non-empty.  Each of them adds at least one to b, so there
    // are at most b - d - 1.  nb: where its frame starts.
    __device__ __forceinline__ void descend(int w, int b, int nb) {
        const W ho = row(1, w);
        W hi = (W)0;
        if constexpr (DIR)
            hi = row(3, w);
        const W vb = bit_at<W>(v), wb = bit_at<W>(w);
        if (ballot(nb >= cap && base < cap) != 0) {
            // entries jump to the worst-case area: the ring starts anew there
            if (nb >= cap && base < cap) {
                for (int n = base + HE + K - wlo; n > 0; --n)
                    evict();
                wlo = nb;
                wslot = slot_of(nb);
            }
        }
        // Class k is still in the ring when its turn comes: the k classes
        // before it left at most NR k parts, which pushed out at most
        // (K + 2 HE + NR k) - rc entries of this frame, at most HE + k.
        const bool far = ballot(base < wlo || K + HE + (NR - 1) * (K - 1) > rc) != 0;
        // the child's header, written when the search leaves it for a child
        for (int i = 0; i < HE; ++i)
            if (nb + i - wlo >= rc)
                evict();
        const int cslot = slot_of(nb);
        int s = wrap(cslot + HE), K2 = 0;
        int room = rc - (nb + HE - wlo);  // parts that fit before entries must go
        each_class(far, [&](int, const Cls<W> &c) {
            W pl[NR], pr[NR];
            split(c, ho, hi, pl, pr);
            pl[0] = pl[0] & ~vb;
            pr[0] = pr[0] & ~wb;
#pragma unroll
            for (int a = 0; a < NR; ++a) {
                if (pl[a] != (W)0 && pr[a] != (W)0) {
                    if (K2 >= room) {
                        evict();
                        room += 1;
                    }
                    Cls<W> x;
                    x.L = pl[a];
                    x.R = pr[a];
                    lput(lane, s, pack(x));
                    s = wrap(s + 1);
                    K2 += 1;
                }
            }
        });
        map_at(lane)[d] = (uint16_t)(v | (w << 8));
        if (K2 == 0)
            return;  // nothing left to split: the parent goes on
        Hdr h;
        h.x = (uint32_t)pbase | ((uint32_t)K << 16) | ((uint32_t)d << 24);
        h.y = (uint32_t)v | ((uint32_t)sel << 8) | ((uint32_t)bound << 16) |
              ((uint32_t)(flags & kSaved) << 24) |
              ((base < cap && nb >= cap) ? (uint32_t)kBig << 24 : 0u);
        h.r = rrem;
        put_hdr(lane, base, wlo, h);
        c_pushed += (uint32_t)K2;
        pbase = base;
        base = nb;
        bslot = cslot;
        t += 1;
        K = K2;
        d += 1;
        bound = b;
        rrem = (W)0;
        flags = kSel;
        const int used = nb + HE + K2;
        max_used = used > max_used ? used : max_used;
    }

    __device__ __forceinline__ void step() {
        // pop and unmatched, in turns while lanes need them: half of the
        // unmatched children are pruned, and their lanes pop on
        for (int i = 0; i < kPops; ++i) {
            const bool need_pop = t >= 0 && rrem == (W)0 && !(flags & (kUnm | kSel));
            if (ballot(need_pop)) {
                if (need_pop)
                    pop();
            } else if (i > 0) {
                break;
            }
            const bool need_unm = rrem == (W)0 && (flags & kUnm);
            if (ballot(need_unm))
                if (need_unm)
                    unmatched();
        }
        const bool need_ld = (rrem != (W)0 || (flags & kSel)) && base < wlo &&
                             (wlo > base + HE + K - rc);
        if (ballot(need_ld))
            if (need_ld)
                fetch();
        const bool need_sel = (flags & kSel) != 0;
        if (ballot(need_sel))
            if (need_sel)
                select();
        if constexpr (POL)
            for (uint64_t pm = ballot(t >= 0 && (flags & (kPolV | kPolW))); pm != 0; pm &= pm - 1)
                consult(ctz(pm));
        if (flags & kRow) {
            go = row(0, v);
            if constexpr (DIR)
                gi = row(2, v);
            flags &= ~kRow;
        }
        bool found = false;
        int w = 0, b = 0;
        if (ballot(rrem != (W)0))
            if (rrem != (W)0)
                found = evaluate(w, b);
        if (ballot(found)) {
            // where the child's frame starts: above this one, or, where it
            // might not fit, in the wavefront's worst-case area, if no other
            // lane is in it (a lane that has to wait takes its child back)
            int nb = base + HE + K;
            const bool big = found && lane_enters_area(base, nb, HE + (b - d - 1), cap);
            const uint64_t wants = ballot(big);
            if (wants) {
                const uint64_t owner = ballot(t >= 0 && base >= cap);
                if (big) {
                    if (owner != 0 || lane != ctz(wants)) {
                        found = false;
                        rrem = rrem | bit_at<W>(w);
                        c_child -= 1;
                        c_ncls -= (uint32_t)K;
                    } else {
                        nb = cap;
                    }
                }
            }
            const uint64_t in_big = ballot(found && nb >= cap);
            if (in_big) {
                n_big += (unsigned)__builtin_popcountll(in_big);
                const bool over = found && nb >= cap &&
                                  (uint32_t)(nb - cap + HE + (b - d - 1)) > big_cap;
                if (ballot(over)) {
                    fail(kErrStack);  // a broken invariant: past the worst case
                    found = found && !over;
                }
            }
            const int size = d + 1;
            uint64_t up = ballot(found && size > inc);
            if (found)
                descend(w, b, nb);
            while (up) {
                const int l = ctz(up);
                up &= up - 1;
                const int sz = rl(size, l);
                if (sz > inc)
                    improve(l, sz);
            }
        }
        n_steps += 1;
    }

    // ---- work sharing inside the wavefront ----

    // Idle lanes take the lowest open frame of busy lanes, one each, from
    // the lanes whose lowest open frame is (nearly) the shallowest: a frame
    // near the leaves is gone in a few steps.  Undirected rows of up to 64
    // bits: from the lanes whose top frame has (nearly) the highest bound,
    // which finds large mappings sooner (six pairs of 30 vertices one by one 45
    // ms by depth and 38 by bound, 4,096 of 10 to 22 34 and 25; the 4,096 of 10
    // to 35, where a few very sparse pairs decide, show little beyond their
    // spread: 11.2 to 19.8 s by depth, mean 14.8 of 28 launches, 8.9 to 21.9 by
    // bound, mean 14.0 of 42; the other kinds of pairs were slower that way: 60 directed labelled
    // pairs 4.0 and 4.5 ms, 254 vertices 55 and 67).
    __device__ __forceinline__ void steal() {
        const bool is_i = t < 0;
        bool is_v = t >= 0 && lo_t < t;
        constexpr bool BY_BOUND = LROWS && !DIR;
        const uint32_t depth = !is_v      ? 0xFFFFu
                               : BY_BOUND ? (uint32_t)(255 - bound)
                                          : (uint32_t)(d - t + lo_t);
        const uint64_t im = ballot(is_i);
        const int ni = __builtin_popcountll(im);
        uint32_t most = wave_min(depth);
        uint64_t vm = ballot(is_v && depth <= most);
        for (int i = 0; i < (BY_BOUND ? kStealBounds : kStealSpan) && __builtin_popcountll(vm) < ni; ++i)
            vm = ballot(is_v && depth <= ++most);
        is_v = is_v && depth <= most;
        const int nv = __builtin_popcountll(vm);
        const int n = ni < nv ? ni : nv;
        if (n == 0)
            return;
        // the j-th victim and the j-th idle lane, in lane j
        const int ri = mbcnt(im), rv = mbcnt(vm);
        const int vj = __builtin_amdgcn_ds_permute((is_v ? rv : nv + mbcnt(~vm)) << 2, lane);
        const int ij = __builtin_amdgcn_ds_permute((is_i ? ri : ni + mbcnt(~im)) << 2, lane);
        const int vl = shfl_any(vj, ri), tl = shfl_any(ij, rv);
        const bool thief = is_i && ri < n, robbed = is_v && rv < n;
        int fb = shfl_any(lo_base, vl), ft = shfl_any(lo_t, vl);
        const int vt = shfl_any(t, vl), vw = shfl_any(wlo, vl);
        wave_sync();  // (entries written by other lanes)
        bool got = false;
        Hdr h;
        h.x = h.y = 0;
        h.r = (W)0;
        for (;;) {
            const bool look = thief && !got && ft < vt;
            if (ballot(look) == 0)
                break;
            if (look) {
                h = get_hdr(vl, fb, vw);
                got = open_frame(h);
                if (!got) {
                    fb = next_frame(fb, h);
                    ft += 1;
                }
            }
        }
        // the victim's lowest open frame is above the one taken
        const int rb = shfl_any(got ? next_frame(fb, h) : fb, tl);
        const int rt = shfl_any(got ? ft + 1 : ft, tl);
        if (robbed) {
            lo_base = rb;
            lo_t = rt;
        }
        if (got) {
            Hdr e = h;
            e.r = (W)0;
            e.y &= ~((uint32_t)kUnm << 24);
            put_hdr(vl, fb, vw, e);  // nothing is left of it there
            K = (int)((h.x >> 16) & 0xFFu);
            start_frame((int)(h.x >> 24), h.y, h.r);
            wlo = HE + K > rc ? HE + K - rc : 0;
            wslot = slot_of(wlo);
            for (int k = 0; ballot(k < K) != 0; k += 4) {
                Ent x[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    x[i] = eget(vl, fb + HE + (k + i < K ? k + i : K - 1), vw);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (k + i < K)
                        eput(lane, HE + k + i, wlo, x[i]);
            }
            if (POL && ordered()) {
                v2u64 x[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    x[i] = *(glb_ptr<v2u64>)(wst + order_at(vl, d) + 16u * i);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    *(glb_ptr<v2u64>)(wst + order_at(lane, d) + 16u * i) = x[i];
            }
            for (int j = 0; ballot(j < d) != 0; j += 32) {
                // (up to 32 pairs in flight; past d, within the map, anything)
                v2u64 x[4];
                const uint32_t top = map_bytes - 16u;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    x[i] = *(glb_ptr<v2u64>)(wst + (uint32_t)vl * stride +
                                             umin(2u * (uint32_t)j + 16u * i, top));
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (j + 8 * i < d)
                        *(glb_ptr<v2u64>)(wst + (uint32_t)lane * stride + 2u * j + 16u * i) = x[i];
            }
        }
        n_don += (unsigned)__builtin_popcountll(ballot(got));
        wave_sync();
    }

    // Whether a frame below a top still has work, and where the one above it
    // starts.
    __device__ __forceinline__ bool open_frame(const Hdr &h) const {
        return (h.r != (W)0 || ((h.y >> 24) & kUnm)) &&
               !(reprune && (int)((h.y >> 16) & 0xFFu) <= inc);
    }
    __device__ __forceinline__ int next_frame(int fb, const Hdr &h) const {
        return ((h.y >> 24) & kBig) ? cap : fb + HE + (int)((h.x >> 16) & 0xFFu);
    }

    // The lane's only frame, from a header's fields (K and the ring are set
    // by the caller).
    __device__ __forceinline__ void start_frame(int fd, uint32_t y, const W &r) {
        t = 0;
        base = pbase = bslot = 0;
        lo_t = lo_base = 0;
        d = fd;
        v = (int)(y & 0xFFu);
        sel = (int)((y >> 8) & 0xFFu);
        bound = (int)((y >> 16) & 0xFFu);
        rrem = r;
        flags = ((int)(y >> 24) & kSaved) | (r != (W)0 ? kRow : 0);
    }

    // ---- work sharing between wavefronts ----

    __device__ __forceinline__ void raise_flag(unsigned bits) {
        if (lane == 0) {
            if (bits & kFlagStop)
                __hip_atomic_store(&P.g->stop, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            for (int k = 0; k < kRings; ++k)
                __hip_atomic_fetch_or(&P.g->xcd[k].flag, bits, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __device__ __forceinline__ void fail(unsigned code) {
        if (lane == 0)
            __hip_atomic_store(&P.g->error, code, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        raise_flag(kFlagStop);
        stop = true;  // (this wavefront leaves at the end of the step)
    }

    // The lane with the shallowest open frame below its top, of |M| at most
    // deepest, gives it away: the lane (-1: none), the frame and its header, as
    // scalars.  The frame is not marked yet.
    __device__ __forceinline__ int pick_frame(int deepest, int &fb, Hdr &h) {
        for (int tries = 0; tries < 4; ++tries) {
            const bool c = t >= 0 && lo_t < t;
            const uint32_t key = wave_min(c ? ((uint32_t)(d - t + lo_t) << 8) | (uint32_t)lane
                                            : ~0u);
            if (key == ~0u || (int)(key >> 8) > deepest)
                return -1;
            const int l = (int)(key & 63u);
            int ft = rl(lo_t, l);
            const int lt = rl(t, l), lw = rl(wlo, l);
            fb = rl(lo_base, l);
            while (ft < lt) {
                h = get_hdr(l, fb, lw);
                h.x = sc(h.x);
                h.y = sc(h.y);
                h.r = sc(h.r);
                if (open_frame(h))
                    break;
                fb = next_frame(fb, h);
                ft += 1;
            }
            if (lane == l) {
                lo_base = fb;
                lo_t = ft;
            }
            if (ft < lt && (int)(h.x >> 24) <= deepest)
                return l;
        }
        return -1;
    }
    // Nothing is left of lane l's frame fb.
    __device__ __forceinline__ void gave(int l, int fb, Hdr h) {
        h.r = (W)0;
        h.y &= ~((uint32_t)kUnm << 24);
        const int lw = rl(wlo, l);
        if (lane == l) {
            lo_base = next_frame(fb, h);
            lo_t += 1;
        }
        if (lane == 0)
            put_hdr(l, fb, lw, h);
        n_don += 1;
    }

    // A free slot in ring `from`, else in the next rings.
    __device__ __forceinline__ bool reserve(int from, int &ring, u64w &ticket) {
        const u64w mask = (u64w)P.ring_slots - 1;
        int ok = 0, rr = 0;
        u64w tk = 0;
        if (lane == 0) {
            for (int k = 0; k < kRings && !ok; ++k) {
                const int r = (from + k) & (kRings - 1);
                u64w *sq = P.seq + (size_t)r * P.ring_slots;
                for (int tries = 0; tries < 4; ++tries) {
                    const u64w tl = ld_rlx(&P.g->ring[r].tail);
                    const u64w s = ld_rlx(&sq[tl & mask]);
                    if (s == tl) {
                        if (cas64(&P.g->ring[r].tail, tl, tl + 1)) {
                            ok = 1;
                            rr = r;
                            tk = tl;
                            break;
                        }
                    } else if (s < tl) {
                        break;  // this ring is full
                    }
                }
            }
        }
        ok = rl(ok, 0);
        ring = rl(rr, 0);
        ticket = rl_ull(tk, 0);
        return ok != 0;
    }

    // A frame to the queue; false if there is none, or no slot is free.
    __device__ __forceinline__ bool donate(int to) {
        int fb = 0;
        Hdr h;
        const int l = pick_frame(P.donate_depth, fb, h);
        if (l < 0)
            return false;
        u64w ticket;
        int ring;
        if (!reserve(to, ring, ticket))
            return false;
        const u64w mask = (u64w)P.ring_slots - 1;
        const size_t idx = (size_t)ring * P.ring_slots + (size_t)(ticket & mask);
        uint8_t *slot = P.slots + idx * (size_t)P.slot_bytes;
        const int fK = (int)((h.x >> 16) & 0xFFu), fd = (int)(h.x >> 24), lw = rl(wlo, l);
        RecHdr<W> rh;
        rh.inst = (uint32_t)inst;
        rh.K = (uint8_t)fK;
        rh.d = (uint8_t)fd;
        rh.v = (uint8_t)(h.y & 0xFFu);
        rh.sel = (uint8_t)((h.y >> 8) & 0xFFu);
        rh.bound = (uint8_t)((h.y >> 16) & 0xFFu);
        rh.flags = (uint8_t)((h.y >> 24) & kSaved);
        rh.lsel = rh.rsel = 0;
        rh.pad[0] = rh.pad[1] = rh.pad[2] = rh.pad[3] = 0;
        rh.rrem = h.r;
        if (lane == 0)
            *(RecHdr<W> *)slot = rh;
        // mapping (four pairs a word) and classes
        u64w *rmap = (u64w *)(slot + rec_map_off<W>());
        for (int i = lane; 4 * i < fd; i += 64)
            rmap[i] = *(glb_ptr<u64w>)(wst + (uint32_t)l * stride + 8u * i);
        u64w *rcls = (u64w *)(slot + rec_cls_off<W>());
        for (int i = lane; i < fK; i += 64) {
            const Ent x = eget(l, fb + HE + i, lw);
#pragma unroll
            for (int q = 0; q < EW; ++q)
                rcls[(size_t)i * EW + q] = x.w[q];
        }
        gave(l, fb, h);
        if (lane == 0) {  // the record is a unit of its own
            a_add_rlx(&P.open[inst], 1);
            a_add_rlx(&P.g->open_total, 1);
        }
        // every word of the record has been written, and its unit counted,
        // before its sequence number says so (at agent scope: its reader may
        // sit behind another L2)
        if (lane == 0)
            st_rel(&P.seq[idx], ticket + 1);
        wave_sync();
        return true;
    }

    // A frame to the waiting wavefront w of the workgroup: its classes and
    // mapping into lane 0 of that wavefront's stacks, its header into the
    // box.
    __device__ __forceinline__ void feed(unsigned hungry) {
        wave_sync();
        int fb = 0;
        Hdr h;
        const int l = pick_frame(255, fb, h);
        if (l < 0)
            return;
        const int w = (int)ctz(hungry);
        unsigned old = 0;
        if (lane == 0)
            old = __hip_atomic_fetch_and(&T.hungry, ~(1u << w), __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_WORKGROUP);
        if (!((unsigned)rl((int)old, 0) & (1u << w)))
            return;  // another wavefront serves it, or it found work
        const int fK = (int)((h.x >> 16) & 0xFFu), fd = (int)(h.x >> 24), lw = rl(wlo, l);
        const glb_ptr<char> ws = wst + (long long)(w - wv) * P.hstack_stride;
        for (int i = lane; 4 * i < fd; i += 64)
            *(glb_ptr<u64w>)(ws + 8u * i) = *(glb_ptr<u64w>)(wst + (uint32_t)l * stride + 8u * i);
        if (POL && fd <= P.policy_depth && lane < 8)
            *(glb_ptr<u64w>)(ws + order_at(0, fd) + 8u * (uint32_t)lane) =
                *(glb_ptr<u64w>)(wst + order_at(l, fd) + 8u * (uint32_t)lane);
        const uint32_t dst = at(0, HE);
        for (int i = lane; i < fK; i += 64) {
            const Ent x = eget(l, fb + HE + i, lw);
#pragma unroll
            for (int q = 0; q < EW; ++q)
                *(glb_ptr<u64w>)(ws + dst + (uint32_t)i * EB + 8u * q) = x.w[q];
        }
        if (lane == 0) {
            T.box[w][0] = (u64w)h.x | ((u64w)h.y << 32);
            T.box[w][1] = (u64w)(uint32_t)unit;
            __hip_atomic_fetch_add(&T.ref[unit], 1u, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
            for (int q = 0; q < (NB + 63) / 64; ++q)
                T.box[w][2 + q] = word64(h.r, q);
        }
        gave(l, fb, h);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        if (lane == 0)
            st_wg(&T.full[w], 1u);
    }
    // The frame that a sibling has put into this wavefront's stack.
    __device__ __forceinline__ void accept() {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        const u64w a = rl_ull(T.box[wv][0], 0);
        const int u = (int)rl_ull(T.box[wv][1], 0);
        uint64_t rw[4];
#pragma unroll
        for (int q = 0; q < (NB + 63) / 64; ++q)
            rw[q] = rl_ull(T.box[wv][2 + q], 0);
        if (lane == 0)
            st_wg(&T.full[wv], 0u);
        unit = u;
        enter(rl(ld_wg(&T.inst[u]), 0));
        set_inc(rl(ld_wg(&T.inc[u]), 0));
        begin(0, (uint32_t)a, (uint32_t)(a >> 32), from_words<W>(rw));
        n_pops += 1;
    }
    // Lane l starts on a frame of the instance whose classes and mapping are
    // in its part in HBM.
    __device__ __forceinline__ void begin(int l, uint32_t x, uint32_t y, const W &r) {
        if (lane == l) {
            K = (int)((x >> 16) & 0xFFu);
            start_frame((int)(x >> 24), y, r);
            wlo = HE + K;
            wslot = slot_of(wlo);
            if (bound <= inc) {
                rrem = (W)0;
                flags = 0;
            }
        }
    }

    // A unit of instance i came from outside the workgroup.
    __device__ __forceinline__ void new_unit(int i) {
        int u = 0;
        if (lane == 0) {
            // (one of 16 is free: each taken one has a wavefront on it)
            for (u = wv;; u = (u + 1) & 15) {
                unsigned want = 0;
                if (__hip_atomic_compare_exchange_strong(&T.ref[u], &want, 2u, __ATOMIC_RELAXED,
                                                         __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_WORKGROUP))
                    break;
            }
        }
        unit = rl(u, 0);
        enter(i);
        set_inc(read_inc());
        if (lane == 0) {
            st_wg(&T.inst[unit], i);
            st_wg(&T.inc[unit], inc);
            st_wg(&T.seen[unit], (unsigned)now_ticks());
        }
    }
    // The wavefront works on instance i from now on.
    __device__ __forceinline__ void enter(int i) {
        const DevInst di = P.inst[i];
        inst = i;
        target = sc((int)di.target);
        inc_slot = sc((int)di.inc_slot);
        twin = sc((int)di.twin);
        dead_on = sc((int)di.dead_on);
        grow = (const W *)P.adj + (size_t)i * (NR * NB);
        if constexpr (LROWS) {
            if (rows_inst != i) {
                for (int q = lane; q < NR * arows; q += 64)
                    lrow[q] = grow[(q / arows) * NB + q % arows];
                rows_inst = i;
                wave_sync();
            }
        }
        inc = 0;
    }

    // Take a queued node into lane 0: from this XCD's ring, else from one
    // other ring, a different one on each call.
    __device__ __forceinline__ bool take_record() {
        const int l = 0;
        const u64w mask = (u64w)P.ring_slots - 1;
        int ok = 0, rr = 0;
        u64w hd = 0;
        if (lane == 0) {
            steal_from = (steal_from + 1) & (kRings - 1);
            if (steal_from == my_ring)
                steal_from = (steal_from + 1) & (kRings - 1);
            for (int k = 0; k < 2 && !ok; ++k) {
                const int r = k == 0 ? my_ring : steal_from;
                u64w *sq = P.seq + (size_t)r * P.ring_slots;
                for (int tries = 0; tries < 4; ++tries) {
                    const u64w h = ld_rlx(&P.g->ring[r].head);
                    const u64w s = ld_rlx(&sq[h & mask]);
                    if (s == h + 1) {
                        if (cas64(&P.g->ring[r].head, h, h + 1)) {
                            ok = 1;
                            rr = r;
                            hd = h;
                            break;
                        }
                    } else if (s < h + 1) {
                        break;  // empty, or its producer is still writing
                    }
                }
            }
        }
        steal_from = rl(steal_from, 0);
        ok = rl(ok, 0);
        if (!ok)
            return false;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        hd = rl_ull(hd, 0);
        const int ring = rl(rr, 0);
        const size_t idx = (size_t)ring * P.ring_slots + (size_t)(hd & mask);
        uint8_t *slot = P.slots + idx * (size_t)P.slot_bytes;
        const RecHdr<W> rh = *(const RecHdr<W> *)slot;
        const int ri = sc((int)rh.inst);
        const int rK = sc((int)rh.K), rd = sc((int)rh.d);
        const uint32_t y = sc((uint32_t)rh.v | ((uint32_t)rh.sel << 8) |
                              ((uint32_t)rh.bound << 16) | ((uint32_t)rh.flags << 24));
        const W rr_ = sc((W)rh.rrem);
        if (!record_fits(ri, rK, rd, P.count, P.frames)) {
            fail(kErrRecord);  // (a broken invariant: no such frame)
            return false;
        }
        // the record's words go straight to lane l's stack
        u64w *rmap = (u64w *)(slot + rec_map_off<W>());
        for (int i = lane; 4 * i < rd; i += 64)
            *(glb_ptr<u64w>)(wst + (uint32_t)l * stride + 8u * i) = rmap[i];
        u64w *rcls = (u64w *)(slot + rec_cls_off<W>());
        const uint32_t dst = at(l, HE);
        for (int i = lane; i < rK * EW; i += 64)
            *(glb_ptr<u64w>)(wst + dst + 8u * i) = rcls[i];
        // every lane's loads of the slot have returned before it is handed back
        __builtin_amdgcn_s_waitcnt(0);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        if (lane == 0)
            st_rlx(&P.seq[idx], hd + (u64w)P.ring_slots);
        wave_sync();
        new_unit(ri);
        begin(l, ((uint32_t)rK << 16) | ((uint32_t)rd << 24), y, rr_);
        // (a record holds no order: the scores are those it was made from)
        if (POL && lane == l && rrem != (W)0 && ordered())
            flags |= kPolW;
        n_pops += 1;
        return true;
    }

    // The next unstarted instance (its work unit was counted by the reset).
    __device__ __forceinline__ bool claim_instance() {
        if (!roots_left)
            return false;
        int i = -1;
        if (lane == 0) {
            const unsigned nx = ld_rlx(&P.g->next_inst);
            if (nx < (unsigned)P.count) {
                const unsigned x = a_addu(&P.g->next_inst, 1u);
                if (x < (unsigned)P.count)
                    i = (int)x;
            }
        }
        i = rl(i, 0);
        if (i < 0) {
            roots_left = false;
            return false;
        }
        const DevInst di = P.inst[i];
        const Cls<W> *rcl = (const Cls<W> *)P.rootcls + sc((int)di.cls_off);
        const int k0 = sc((int)di.K0);
        int sum = 0;
        for (int k = lane; k < k0; k += 64) {
            const Cls<W> c = ld_cls(rcl + k);
            hput(at(0, HE + k), pack(c));
            const int nl = popc(c.L), nr = popc(c.R);
            sum += nl < nr ? nl : nr;
        }
        const int b = wave_sum(sum);
        wave_sync();
        new_unit(i);
        begin(0, (uint32_t)k0 << 16, (uint32_t)b << 16, (W)0);
        if (lane == 0) {
            c_unm += 1;  // the root
            flags = (k0 == 0 || b <= inc) ? 0 : kSel;
        }
        return true;
    }

    // No lane has work left.  The last wavefront to leave a unit ends it.
    __device__ __forceinline__ void finish_unit() {
        const u64w mine = count_nodes();
        if (lane == 0) {
            u64w total = 0;
            if (team_leave<WgOps>(T, unit, mine, &total)) {
                add_nodes(total);
                if (!stop) {
                    if (a_add_rlx(&P.open[inst], -1) == 1)
                        __hip_atomic_store(&P.t_proof[inst], now_ticks(), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                    if (a_add_rlx(&P.g->open_total, -1) == 1)
                        raise_flag(kFlagDone);
                }
                st_wg(&T.ref[unit], 0u);
            }
        }
        unit = -1;
    }

    // ---- counts ----

    // The nodes counted since the last call.
    __device__ __forceinline__ u64w count_nodes() {
        const u64w child = lanes_total(c_child), sum = child + lanes_total(c_unm);
        n_child += child;
        n_ncls += lanes_total(c_ncls);
        n_pushed += lanes_total(c_pushed);
        c_child = c_unm = c_ncls = c_pushed = 0;
        return sum;
    }
    // (lane 0) Nodes to the instance's count; true: the limit has been passed
    // (whoever passes it tells the others).
    __device__ __forceinline__ bool add_nodes(u64w n) {
        if (n == 0)
            return false;
        a_add64(&P.nodes[inst], n);
        if (P.node_limit <= 0)
            return false;
        const u64w before = a_add64(&P.g->node_total, n), limit = (u64w)P.node_limit;
        if (before <= limit && before + n > limit)
            raise_flag(kFlagStop);
        return before + n > limit;
    }
    __device__ __forceinline__ void flush_nodes() {
        const u64w n = count_nodes();
        int over = 0;
        if (lane == 0)
            over = add_nodes(n) ? 1 : 0;
        if (rl(over, 0))
            stop = true;
    }
    __device__ __forceinline__ long long launched() const {
        return (long long)gridDim.x * (blockDim.x >> 6);
    }
    // Nodes that a wavefront may hold back: over all wavefronts a sixteenth of
    // the limit, a quarter of what a forecast waits for.
    __device__ __forceinline__ int held_back() const {
        const long long all = launched();
        int x = kFlushNodes;
        while (x > 1 && ((P.node_limit > 0 && 16 * all * x > P.node_limit) ||
                         (P.dead_abs > 0 && 4 * all * x > P.dead_abs)))
            x >>= 1;
        return x;
    }
    // Steps between checks.  Up to 128 children are evaluated in one: a limit of
    // no more than a few of them per wavefront is looked at after each.
    __device__ __forceinline__ int check_every() const {
        const bool near = P.node_limit > 0 && P.node_limit < 2048 * launched();
        return near ? 1 : sc(P.check_interval);
    }
    DEV u64w lanes_total(uint32_t x) {
        // (16-bit pieces: 64 of them sum below 2^31)
        return (u64w)(unsigned)wave_sum((int)(x & 0xFFFFu)) +
               ((u64w)(unsigned)wave_sum((int)(x >> 16)) << 16);
    }

    // Dead-end forecast (paper Sec. IV.A), as in the other kernels.
    __device__ __forceinline__ void forecast_dead_ends() {
        if (!dead_on)
            return;
        int give_up = 0;
        if (lane == 0) {
            const u64w n = ld_rlx(&P.nodes[inst]);
            const u64w b = ld_rlx(&P.best_nodes[inst]);
            const u64w since = n > b ? n - b : 0ull;
            u64w thr = (u64w)P.dead_abs;
            if (P.dead_rel > 0 && (u64w)P.dead_rel * b > thr)
                thr = (u64w)P.dead_rel * b;
            if (since > thr) {
                st_rlx(&P.dead[inst], 1);
                give_up = 1;
            }
        }
        if (rl(give_up, 0))
            inc = 255;
    }

    // True once every P.check_ticks for one of the workgroup's wavefronts.
    __device__ __forceinline__ bool my_turn(unsigned *last) {
        int mine = 0;
        if (lane == 0) {
            unsigned old = ld_wg(last);
            const unsigned now = (unsigned)now_ticks();
            mine = now - old >= (unsigned)P.check_ticks &&
                   __hip_atomic_compare_exchange_strong(last, &old, now, __ATOMIC_RELAXED,
                                                        __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        return rl(mine, 0) != 0;
    }

    // Periodic.  What all XCDs share is looked at by one wavefront of the
    // workgroup at a time: lines that thousands of wavefronts read and raise
    // cost tens of microseconds each.
    __device__ __forceinline__ void check() {
        since_check = 0;
        if (rl((int)ld_wg(&T.done), 0)) {
            stop = true;
            return;
        }
        set_inc(rl(ld_wg(&T.inc[unit]), 0));
        if (my_turn(&T.seen[unit])) {
            set_inc(read_inc());
            if (lane == 0)
                __hip_atomic_fetch_max(&T.inc[unit], inc, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        if (P.node_limit > 0 || P.dead_abs > 0) {
            if ((unsigned)n_steps - flushed >= kFlushSteps ||
                wave_sum((int)(c_child + c_unm)) >= flush_at) {
                flushed = (unsigned)n_steps;
                flush_nodes();
                if (P.dead_abs > 0)
                    forecast_dead_ends();
            }
        } else if (ballot((c_child | c_unm | c_ncls | c_pushed) > (1u << 30))) {
            flush_nodes();
        }
        if (my_turn(&T.looked))
            look_out();
    }

    // Limits, and frames for the rings: while workgroups of this XCD, or of
    // another one (a different one each time), are idle and their ring holds
    // fewer.
    __device__ __forceinline__ void look_out() {
        other = (other + 1) & (kRings - 1);
        if (other == my_ring)
            other = (other + 1) & (kRings - 1);
        u64w x = 0;
        {
            // six lines in one round trip
            const int q = lane < 3 ? my_ring : other, f = lane < 3 ? lane : lane - 3;
            u64w *at = f == 0   ? (u64w *)&P.g->xcd[q]
                       : f == 1 ? (u64w *)&P.g->ring[q].tail
                                : (u64w *)&P.g->ring[q].head;
            if (lane < 6)
                x = ld_rlx(at);
        }
        const u64w ctl = rl_ull(x, 0);
        if ((unsigned)ctl) {
            stop = true;
            return;
        }
        if (now_ticks() - t_start > P.limit_ticks) {
            raise_flag(kFlagStop);
            stop = true;
            return;
        }
        const long long waiting = (long long)(rl_ull(x, 1) - rl_ull(x, 2));
        const long long waiting_o = (long long)(rl_ull(x, 4) - rl_ull(x, 5));
        const int idle = (int)(ctl >> 32), idle_o = (int)(rl_ull(x, 3) >> 32);
        int want = idle > waiting ? (int)(idle - waiting) : 0;
        if (waiting < P.donate_low && want < 1)
            want = 1;
        const bool want_o = idle_o > waiting_o;
        if (want == 0 && !want_o)
            return;
        wave_sync();
        bool more = true;
        // (one each: four or sixteen at a time were no faster, the L2-wide
        // releases cost more than the earlier start gains)
        for (int i = 0; i < 2 && more; ++i)
            if (i == 0 ? want > 0 : want_o)
                more = donate(i == 0 ? my_ring : other);
    }

    // An idle wavefront takes the next instance, or waits for a sibling's
    // frame.  The first of the idle siblings looks at the rings meanwhile,
    // seldom while others of the workgroup are busy (they will feed it).
    // False: the search is over.
    __device__ __forceinline__ void count_idle(unsigned idle) {
        // (two of them may look at the rings, and take work, at the same time)
        if (lane == 0) {
            const int change = team_idle<WgOps>(T, idle);
            if (change != 0)
                a_add_rlx(&P.g->xcd[my_ring].idle, change);
        }
    }
    __device__ __forceinline__ bool wait_work(bool claim) {
        // (a sibling may write this wavefront's stack from here on: its own
        // stores there have completed)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);
        const u64w t_sleep = now_ticks();
        const unsigned bit = 1u << wv, all = (2u << ((blockDim.x >> 6) - 1u)) - 1u;
        unsigned gap = 1, left = 1;
        bool listed = false, fed = false, first = true;
        for (;;) {
            if (first && !claim) {
                first = false;
                continue;
            }
            if (!first) {
                if (!listed) {
                    if (lane == 0)
                        __hip_atomic_fetch_or(&T.hungry, bit, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_WORKGROUP);
                    listed = true;
                }
                __builtin_amdgcn_s_sleep(8);
                if (rl((int)ld_wg(&T.full[wv]), 0)) {
                    fed = true;
                    break;
                }
                const bool over = rl((int)ld_wg(&T.done), 0) != 0;
                const unsigned hungry = (unsigned)rl((int)ld_wg(&T.hungry), 0);
                if (left != 0)
                    left -= 1;
                if (hungry == all && left > gap)
                    left = gap;
                if (!over && (left != 0 || (hungry & (bit - 1u)) != 0))
                    continue;
                const bool alone = hungry == all;  // nobody here can feed it
                unsigned old = 0;
                if (lane == 0)
                    old = __hip_atomic_fetch_and(&T.hungry, ~bit, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP);
                listed = false;
                if (!((unsigned)rl((int)old, 0) & bit)) {
                    // a sibling has taken the bit off: its frame is on its way
                    while (!rl((int)ld_wg(&T.full[wv]), 0))
                        __builtin_amdgcn_s_sleep(2);
                    fed = true;
                    break;
                }
                if (over)
                    break;
                count_idle(alone ? 1 : 0);
                unsigned fl = 0;
                if (lane == 0)
                    fl = ld_rlx(&P.g->xcd[my_ring].flag);
                if (rl((int)fl, 0))
                    break;  // stopped, or no work is left anywhere
                if (now_ticks() - t_start > P.limit_ticks) {
                    raise_flag(kFlagStop);
                    break;
                }
                if (take_record())
                    break;
                gap = gap < (unsigned)P.backoff_max ? 2 * gap : gap;
                left = alone ? gap : kFedGap * gap;
            }
            first = false;
            if (claim_instance())
                break;
        }
        if (fed)
            accept();
        if (unit >= 0)
            count_idle(0);
        n_sleep += now_ticks() - t_sleep;
        return unit >= 0;
    }

    __device__ __forceinline__ void main_loop() {
        t_start = now_ticks();
        const int check_interval = check_every();
        int since_steal = 0, since_feed = 0;
        u64w t_busy0 = t_start;
        // the first instances go to the first wavefronts of all workgroups
        bool claim = (unsigned)wv * gridDim.x < (unsigned)P.count;
        for (;;) {
            const uint64_t am = ballot(t >= 0);
            if (am == 0) {
                if (unit >= 0) {
                    finish_unit();
                    n_busy += now_ticks() - t_busy0;
                }
                if (!wait_work(claim))
                    break;
                claim = true;
                t_busy0 = now_ticks();
            } else if (am != ~0ull) {
                const int idle = 64 - __builtin_popcountll(am);
                if (idle >= kIdleLanes || ++since_steal >= kStealSteps) {
                    since_steal = 0;
                    steal();
                }
            }
            n_lanes += (unsigned)__builtin_popcountll(ballot(t >= 0));
            step();
            if (stop)
                break;
            if (++since_feed >= kFeedSteps &&
                (__builtin_popcountll(ballot(t >= 0)) >= kFeedRich || since_feed >= kFeedAnyway)) {
                const unsigned hungry = (unsigned)rl((int)ld_wg(&T.hungry), 0);
                if (hungry) {
                    feed(hungry);
                    since_feed = 0;
                }
            }
            if (++since_check >= check_interval) {
                check();
                if (stop)
                    break;
            }
        }
        if (lane == 0)
            st_wg(&T.done, 1u);
        if (unit >= 0) {
            n_busy += now_ticks() - t_busy0;
            const u64w n = count_nodes();
            if (lane == 0)
                team_stop<WgOps>(T, unit, n);
        }
        const int mu = (int)~wave_min(~(uint32_t)max_used);
        int last = 0;
        if (lane == 0) {
            const u64w x[kTeamStats] = {n_steps, n_child, n_lanes, n_don, n_pops,
                                        n_busy, n_big, n_pushed, n_sleep, n_ncls};
            for (int i = 0; i < kTeamStats; ++i)
                __hip_atomic_fetch_add(&T.st[i], x[i], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            __hip_atomic_fetch_max(&T.max_stack, mu, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
            last = (int)__hip_atomic_fetch_add(&T.left, ~0u, __ATOMIC_ACQ_REL,
                                               __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        if (rl(last, 0) == 1) {
            // the workgroup's last wavefront hands in its sums
            static_assert(offsetof(SearchStats, node_classes) == 8 * kTeamStats, "in this order");
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            if (lane < 16) {
                const u64w n = team_rest<WgOps>(T, lane);
                if (n != 0)
                    a_add64(&P.nodes[T.inst[lane]], n);
            }
            SearchStats *g = &P.g->st[my_ring];
            if (lane < kTeamStats)
                a_add64(&g->batches + lane, T.st[lane]);
            else if (lane == kTeamStats)
                __hip_atomic_fetch_max(&g->max_stack, T.max_stack, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
        }
    }
};

// Up to 64 vertices a workgroup may hold a CU's 16 wavefronts (128 VGPRs);
// wider rows take more registers, and workgroups of at most 8.
template <typename W, bool DIR, bool POL>
__global__ void __launch_bounds__(sizeof(W) <= 8 ? 1024 : 512) mcs_lane_kernel(SearchParams Pk) {
    extern __shared__ __align__(16) char smem[];
    __shared__ Team T;
    const KernArgs &P = *(const KernArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    if (threadIdx.x == 0) {
        // (before the barrier: no wavefront of the workgroup starts earlier)
        a_min64(&P.g->st[blockIdx.x & (kRings - 1)].t0, now_ticks());
        T.hungry = 0;
        T.done = 0;
        T.looked = 0;
        T.idle = 0;
        T.left = blockDim.x >> 6;
        T.max_stack = 0;
    }
    if (threadIdx.x < kTeamStats)
        T.st[threadIdx.x] = 0;
    if (threadIdx.x < 16) {
        T.full[threadIdx.x] = 0;
        T.ref[threadIdx.x] = 0;
        T.nodes[threadIdx.x] = 0;
    }
    __syncthreads();
    const int wv = sc((int)threadIdx.x >> 6);
    LaneSearch<W, DIR, POL> s(P, T, (lds_ptr<char>)smem + (size_t)wv * (size_t)Pk.lds_per_wave, wv,
                         sc((int)(blockIdx.x * (blockDim.x >> 6)) + wv));
    s.main_loop();
}

}  // namespace mcs

// The kernel for rows of word_bytes (4, 8, 16 or 32; with the learned policy
// at most 8), directed or not.
template <typename W>
static void *lane_kernel(int directed, int policy) {
    using namespace mcs;
    if constexpr (sizeof(W) <= 8)
        if (policy)
            return directed ? (void *)mcs_lane_kernel<W, true, true>
                            : (void *)mcs_lane_kernel<W, false, true>;
    return policy     ? nullptr
           : directed ? (void *)mcs_lane_kernel<W, true, false>
                      : (void *)mcs_lane_kernel<W, false, false>;
}
extern "C" void *mcs_internal_lane_kernel(int word_bytes, int directed, int policy) {
    using namespace mcs;
    switch (word_bytes) {
    case 4: return lane_kernel<uint32_t>(directed, policy);
    case 8: return lane_kernel<uint64_t>(directed, policy);
    case 16: return lane_kernel<u128>(directed, policy);
    case 32: return lane_kernel<u256>(directed, policy);
    }
    return nullptr;
}
