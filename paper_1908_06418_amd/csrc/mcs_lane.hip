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
// Memory of a search:
//   * its class stack, in HBM (mostly served by L2): frames one after
//     another, each a header and its classes.  The stack of one lane holds
//     cap entries; the wavefront has one more area with room for the worst
//     case, m(m+1)/2 classes and m + 1 headers, which one lane at a time may
//     continue into when its own part is full (the others wait with the
//     child that did not fit, or go on with other work);
//   * in LDS, the first kc classes of its top frame and of that frame's
//     parent (two buffers, by the parity of the frame's index), so that a
//     frame is split for all its partners, and a parent is returned to from
//     a child without children, without touching the HBM copy.  Registers
//     keep the parent's header for the same case.  A frame is written to the
//     HBM stack when the search first descends from it.
//
// One step, for the lanes that need each phase:
//   pop       -- the top frame has nothing left: return to the parent;
//   unmatched -- its partners are done: bound the "v unmatched" child;
//   load      -- a frame returned to without its LDS copy is fetched;
//   select    -- a new frame (or one that has just lost v) chooses its class
//                and v;
//   evaluate  -- up to kEvals partners w: split and bound, until one
//                survives;
//   descend   -- the surviving child's non-empty parts become the top frame.
//
// Work sharing: idle lanes take whole frames from busy lanes of the same
// wavefront, all of them at once (steal()): the shallowest open frame below
// the victim's top, with its remaining partners and its "v unmatched" child.
// Between wavefronts frames travel as records through the per-XCD rings of
// mcs_layout.h, one per check.  A record's words are written and read with
// agent-scope (write-through) accesses, so handing one over needs no
// write-back or invalidation of an XCD's L2.  A work unit, for the
// termination counts, is one instance on one wavefront, however many of its
// lanes work on it.
#include "mcs_device.h"

namespace mcs {

namespace {

constexpr int kEvals = 2;      // partners evaluated per step at most
constexpr int kPops = 2;       // pop/unmatched rounds per step at most

// Flags of a search's top frame.
constexpr int kUnm = 1;        // the "v unmatched" child is still to do
constexpr int kLe = 2;         // |L_sel| <= |R_sel|: that child's bound is one lower
constexpr int kOne = 4;        // |L_sel| == 1: its class empties with v
constexpr int kSel = 8;        // class and v are to be chosen
constexpr int kPatch = 16;     // (with kSel) v is to be taken out of the selected class first
constexpr int kDirty = 32;     // the HBM copy is missing or old
constexpr int kInLds = 64;     // the LDS buffer holds the frame's first kc classes
constexpr int kRow = 128;      // v's G rows are to be loaded
constexpr int kBig = 8;        // (saved headers) the child frame starts the worst-case area
constexpr int kSaved = kUnm | kLe | kOne;

constexpr unsigned kErrMapping = 2;  // codes of DevGlobals::error
constexpr unsigned kErrStack = 3;

typedef unsigned long long v2u64 __attribute__((ext_vector_type(2)));
typedef v2u64 v2u64_a8 __attribute__((aligned(8)));
template <typename T>
using lds_ptr = __attribute__((address_space(3))) T *;
// An HBM access whose base is wave-uniform and whose offset is 32-bit.
template <typename T>
using glb_ptr = __attribute__((address_space(1))) T *;

// Lane `from`'s x (every lane of the wavefront active).
DEV int shfl_any(int x, int from) { return __builtin_amdgcn_ds_bpermute(from << 2, x); }

// 64-bit words of a queued record, written and read past the L2s' private
// lines (agent scope), so that no fence has to write back or invalidate one.
DEV void st_agent(unsigned long long *p, unsigned long long v) { st_rlx(p, v); }
DEV unsigned long long ld_agent(const unsigned long long *p) {
    return ld_rlx((unsigned long long *)p);
}

}  // namespace

template <typename W, bool DIR>
struct LaneSearch {
    static constexpr int NB = bits_of<W>();
    static constexpr int NR = DIR ? 4 : 2;                  // row sets, and parts of a class
    static constexpr int EB = 2 * (int)sizeof(W);           // bytes of a stack entry: one class
    static constexpr int HE = lane_hdr_entries((int)sizeof(W));  // entries of a frame header
    static constexpr int NP = EB >= 16 ? EB / 16 : 1;       // 16-byte pieces of a class

    // A frame header: two 32-bit words and the partners left.
    //   x: base of the frame below (16 bits) | K << 16 | d << 24
    //   y: v | sel << 8 | bound << 16 | flags << 24
    struct Hdr {
        uint32_t x, y;
        W r;
    };

    const SearchParams &P;
    int cap, kc, reprune;
    int lane;
    uint32_t stride, map_bytes, big_off, big_cap;
    glb_ptr<char> wst;   // the wavefront's stacks in HBM
    lds_ptr<char> lbuf;  // the wavefront's class buffers: [2][kc][64 lanes], NP planes
    const W *gadj;

    // ---- per-lane state ----
    int inst, inc, target;
    int t, base, pbase, K, d, v, sel, bound, flags;
    int lo_t, lo_base;   // the lowest frame that may still have work
    W rrem, go, gi;
    const W *rows;       // the instance's adjacency rows: [NR][NB]
    bool pv;             // c_*: the parent's header; its LDS buffer is intact
    uint32_t c_x, c_y;
    W c_r;
    bool fin;
    uint32_t c_child, c_unm, c_ncls, c_pushed;  // since the last flush
    int max_used;

    // ---- wave-level ----
    bool stop, roots_left;
    int my_ring, steal_from, since_check;
    unsigned long long t_start, n_steps, n_don, n_pops, n_busy, n_sleep, n_big;
    unsigned long long n_child, n_ncls, n_pushed;  // (per lane)

    __device__ LaneSearch(const SearchParams &p, lds_ptr<char> lds, long long wave) : P(p) {
        lane = lane_id();
        cap = sc(p.cap_classes);
        kc = sc(p.lane_kc);
        reprune = sc(p.reprune);
        stride = (uint32_t)sc(p.lane_stride);
        map_bytes = (uint32_t)sc(p.lane_map_bytes);
        big_off = 64u * stride;
        big_cap = (uint32_t)sc(p.lane_big);
        wst = (glb_ptr<char>)(p.hstack + (size_t)wave * (size_t)p.hstack_stride);
        lbuf = lds;
        gadj = (const W *)p.adj;
        inst = -1;
        inc = target = 0;
        t = -1;
        base = pbase = K = d = v = sel = bound = flags = 0;
        lo_t = lo_base = 0;
        rrem = go = gi = (W)0;
        rows = gadj;
        pv = false;
        c_x = c_y = 0;
        c_r = (W)0;
        fin = false;
        c_child = c_unm = c_ncls = c_pushed = 0;
        max_used = 0;
        stop = false;
        roots_left = true;
        my_ring = (int)(blockIdx.x & (kRings - 1));
        steal_from = my_ring;
        since_check = 0;
        t_start = n_steps = n_don = n_pops = n_busy = n_sleep = n_big = 0;
        n_child = n_ncls = n_pushed = 0;
    }

    // ---- the stack in HBM ----

    // Byte offset of entry i of lane l's stack: its own part below cap, the
    // wavefront's worst-case area from cap on.
    __device__ uint32_t at(int l, int i) const {
        return i < cap ? (uint32_t)l * stride + map_bytes + (uint32_t)i * EB
                       : big_off + (uint32_t)(i - cap) * EB;
    }
    // (entries of 32-bit rows are 8 bytes: no more alignment than that)
    __device__ v2u64 ld16(uint32_t off) const { return *(glb_ptr<v2u64_a8>)(wst + off); }
    __device__ void st16(uint32_t off, unsigned long long a, unsigned long long b) const {
        v2u64 x = {a, b};
        *(glb_ptr<v2u64_a8>)(wst + off) = x;
    }
    __device__ Cls<W> gget(uint32_t off) const {
        Cls<W> c;
        if constexpr (sizeof(W) == 4) {
            const unsigned long long x = *(glb_ptr<unsigned long long>)(wst + off);
            c.L = (uint32_t)x;
            c.R = (uint32_t)(x >> 32);
        } else {
            uint64_t w[2 * NP];
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const v2u64 x = ld16(off + 16 * i);
                w[2 * i] = x[0];
                w[2 * i + 1] = x[1];
            }
            c.L = from_words<W>(w);
            c.R = from_words<W>(w + NP);
        }
        return c;
    }
    __device__ void gput(uint32_t off, const Cls<W> &c) const {
        if constexpr (sizeof(W) == 4) {
            *(glb_ptr<unsigned long long>)(wst + off) =
                (unsigned long long)(uint32_t)c.L | ((unsigned long long)(uint32_t)c.R << 32);
        } else {
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int j = 2 * i;
                st16(off + 16 * i, j < NP ? word64(c.L, j) : word64(c.R, j - NP),
                     j + 1 < NP ? word64(c.L, j + 1) : word64(c.R, j + 1 - NP));
            }
        }
    }
    __device__ Hdr ld_hdr(uint32_t off) const {
        Hdr h;
        const v2u64 a = ld16(off);
        h.x = (uint32_t)a[0];
        h.y = (uint32_t)(a[0] >> 32);
        if constexpr (sizeof(W) <= 8) {
            h.r = (W)a[1];
        } else {
            uint64_t w[NP];
#pragma unroll
            for (int i = 0; i < NP / 2; ++i) {
                const v2u64 x = ld16(off + 16 + 16 * i);
                w[2 * i] = x[0];
                w[2 * i + 1] = x[1];
            }
            h.r = from_words<W>(w);
        }
        return h;
    }
    __device__ void st_hdr(uint32_t off, const Hdr &h) const {
        const unsigned long long a = (unsigned long long)h.x | ((unsigned long long)h.y << 32);
        if constexpr (sizeof(W) <= 8) {
            st16(off, a, (unsigned long long)h.r);
        } else {
            st16(off, a, 0);
#pragma unroll
            for (int i = 0; i < NP / 2; ++i)
                st16(off + 16 + 16 * i, word64(h.r, 2 * i), word64(h.r, 2 * i + 1));
        }
    }
    __device__ glb_ptr<uint16_t> map_at(int l) const {
        return (glb_ptr<uint16_t>)(wst + (uint32_t)l * stride);
    }

    // ---- the top frame's classes ----

    // Class k (< kc) of lane l's LDS buffer `par`.
    __device__ Cls<W> lget(int l, int par, int k) const {
        const int i = (par * kc + k) * 64 + l;
        Cls<W> c;
        if constexpr (sizeof(W) == 4) {
            const unsigned long long x = ((lds_ptr<unsigned long long>)lbuf)[i];
            c.L = (uint32_t)x;
            c.R = (uint32_t)(x >> 32);
        } else {
            uint64_t w[2 * NP];
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const v2u64 x = ((lds_ptr<v2u64>)lbuf)[i + j * 128 * kc];
                w[2 * j] = x[0];
                w[2 * j + 1] = x[1];
            }
            c.L = from_words<W>(w);
            c.R = from_words<W>(w + NP);
        }
        return c;
    }
    __device__ void lput(int l, int par, int k, const Cls<W> &c) const {
        const int i = (par * kc + k) * 64 + l;
        if constexpr (sizeof(W) == 4) {
            ((lds_ptr<unsigned long long>)lbuf)[i] =
                (unsigned long long)(uint32_t)c.L | ((unsigned long long)(uint32_t)c.R << 32);
        } else {
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const int q = 2 * j;
                v2u64 x = {q < NP ? word64(c.L, q) : word64(c.R, q - NP),
                           q + 1 < NP ? word64(c.L, q + 1) : word64(c.R, q + 1 - NP)};
                ((lds_ptr<v2u64>)lbuf)[i + j * 128 * kc] = x;
            }
        }
    }
    // Class k of the lane's own top frame (in its LDS buffer, or past it).
    __device__ Cls<W> cget(int k) const {
        return k < kc ? lget(lane, t & 1, k) : gget(at(lane, base + HE + k));
    }
    __device__ void cput(int k, const Cls<W> &c) const {
        if (k < kc)
            lput(lane, t & 1, k, c);
        else
            gput(at(lane, base + HE + k), c);
    }
    // f(k, class k, k < kc) for each class of the top frames of the lanes
    // that call this, in step.
    template <typename F>
    __device__ void each_class(F f) const {
        const int par = t & 1;
        int k = 0;
        for (; k < kc && ballot(k < K) != 0; ++k)
            if (k < K)
                f(k, lget(lane, par, k), true);
        if (ballot(k < K) != 0) {
            const uint32_t off = at(lane, base + HE);
            for (; ballot(k < K) != 0; ++k)
                if (k < K)
                    f(k, gget(off + (uint32_t)k * EB), false);
        }
    }

    // ---- incumbent ----

    __device__ int cap_inc(int x) const { return (target > 0 && x >= target) ? 255 : x; }
    __device__ void set_inc(int x) {
        x = cap_inc(x);
        inc = x > inc ? x : inc;
    }

    // The path of this lane's map (size vertex pairs) is a common induced
    // subgraph: raise the instance's incumbent; the search that raised it to
    // `size` writes that size's mapping slot.
    __device__ void improve(int size) {
        const DevInst di = P.inst[inst];
        if (size > (di.nG < di.nH ? (int)di.nG : (int)di.nH)) {
            fail_lane(kErrMapping);  // only from a broken class partition
            return;
        }
        const int old = a_max(&P.inc[di.inc_slot], size);
        if (old < size) {
            uint16_t *dst = P.maps + di.map_off + size * (size - 1) / 2;
            const glb_ptr<uint16_t> m = map_at(lane);
            for (int j = 0; j < size; ++j)
                dst[j] = m[j];
            a_max64(&P.t_best[inst], ((unsigned long long)size << 48) |
                                         (now_ticks() & 0xFFFFFFFFFFFFull));
            a_max64(&P.best_nodes[inst], ld_rlx(&P.nodes[inst]) + c_child + c_unm);
        }
        set_inc(old > size ? old : size);
    }

    // ---- the phases of a step ----

    __device__ void pop() {
        rrem = (W)0;
        flags = 0;
        if (t == 0) {
            t = -1;
            fin = true;
            return;
        }
        t -= 1;
        Hdr h;
        if (pv) {
            h.x = c_x;
            h.y = c_y;
            h.r = c_r;
            flags = kInLds;
        } else {
            h = ld_hdr(at(lane, pbase));
        }
        pv = false;
        base = pbase;
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
        if (reprune && bound <= inc) {
            flags = 0;  // nothing here can beat the incumbent: pop again
            return;
        }
        flags |= (int)(h.y >> 24) & kSaved;
        rrem = h.r;
        if (rrem != (W)0)
            flags |= kRow;
    }

    // The "v unmatched" child takes its parent's place: only the selected
    // class loses v.
    __device__ void unmatched() {
        const int ub = bound - ((flags & kLe) ? 1 : 0);
        c_unm += 1;
        if (ub <= inc || ((flags & kOne) && K == 1)) {
            flags = 0;  // pruned, or no class is left
            return;
        }
        bound = ub;
        flags = (flags & (kOne | kInLds | kDirty)) | kSel | kPatch;
    }

    // The first kc classes of a frame returned to, back into its buffer.
    __device__ void fetch() {
        const uint32_t off = at(lane, base + HE);
        const int n = K < kc ? K : kc;
        for (int k = 0; ballot(k < n) != 0; ++k)
            if (k < n)
                lput(lane, t & 1, k, gget(off + (uint32_t)k * EB));
        flags |= kInLds;
    }

    __device__ void select() {
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
            flags |= kDirty;
        }
        // the class of smallest max(|L|, |R|), ties to the smallest G vertex
        uint32_t key = 0xFFFFFFFFu;
        each_class([&](int k, const Cls<W> &c, bool) {
            const int nl = popc(c.L), nr = popc(c.R);
            key = umin(key, ((uint32_t)(nl > nr ? nl : nr) << 16) | ((uint32_t)ctz(c.L) << 8) |
                                (uint32_t)k);
        });
        v = (int)((key >> 8) & 0xFFu);
        sel = (int)(key & 0xFFu);
        const Cls<W> c = cget(sel);
        const int nl = popc(c.L), nr = popc(c.R);
        rrem = c.R;
        flags = (flags & (kDirty | kInLds)) | kUnm | kRow | (nl <= nr ? kLe : 0) |
                (nl == 1 ? kOne : 0);
    }

    // Parts of class c for the child (v, w) by adjacency letter; v and w are
    // still in the part without edges.
    __device__ void split(const Cls<W> &c, const W &ho, const W &hi, W *pl, W *pr) const {
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

    // The next partner w of v: the child's Eq. 1 bound.
    __device__ bool evaluate(int &w, int &b) {
        w = ctz(rrem);
        rrem = rrem & (rrem - (W)1);
        const W ho = ld_w(rows + NB + w);
        W hi = (W)0;
        if constexpr (DIR)
            hi = ld_w(rows + 3 * NB + w);
        int sum = d;  // (v and w each count once in the selected class: d + 1 - 1)
        each_class([&](int, const Cls<W> &c, bool) {
            if constexpr (!DIR) {
                const int l1 = popc(c.L & go), r1 = popc(c.R & ho);
                const int l0 = popc(c.L) - l1, r0 = popc(c.R) - r1;
                sum += (l1 < r1 ? l1 : r1) + (l0 < r0 ? l0 : r0);
            } else {
                W pl[4], pr[4];
                split(c, ho, hi, pl, pr);
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const int nl = popc(pl[a]), nr = popc(pr[a]);
                    sum += nl < nr ? nl : nr;
                }
            }
        });
        b = sum;
        c_child += 1;
        c_ncls += (uint32_t)K;
        return sum > inc;
    }

    // The child (v, w) of bound b becomes the top frame: its non-empty
    // classes, each side non-empty.  Each of them adds at least one to b, so
    // there are at most b - d - 1.  nb: where its frame starts.
    __device__ void descend(int w, int b, int nb) {
        const W ho = ld_w(rows + NB + w);
        W hi = (W)0;
        if constexpr (DIR)
            hi = ld_w(rows + 3 * NB + w);
        const uint32_t own = at(lane, base + HE);
        const uint32_t sub = at(lane, nb + HE);
        const int npar = (t + 1) & 1;
        const bool save = (flags & kDirty) != 0;
        const W vb = bit_at<W>(v), wb = bit_at<W>(w);
        int K2 = 0;
        each_class([&](int k, const Cls<W> &c, bool lds) {
            if (lds && save)
                gput(own + (uint32_t)k * EB, c);
            W pl[NR], pr[NR];
            split(c, ho, hi, pl, pr);
            pl[0] = pl[0] & ~vb;
            pr[0] = pr[0] & ~wb;
#pragma unroll
            for (int a = 0; a < NR; ++a) {
                if (pl[a] != (W)0 && pr[a] != (W)0) {
                    Cls<W> x;
                    x.L = pl[a];
                    x.R = pr[a];
                    if (K2 < kc)
                        lput(lane, npar, K2, x);
                    else
                        gput(sub + (uint32_t)K2 * EB, x);
                    K2 += 1;
                }
            }
        });
        flags &= ~kDirty;
        Hdr h;
        h.x = (uint32_t)pbase | ((uint32_t)K << 16) | ((uint32_t)d << 24);
        h.y = (uint32_t)v | ((uint32_t)sel << 8) | ((uint32_t)bound << 16) |
              ((uint32_t)(flags & kSaved) << 24) |
              ((base < cap && nb >= cap) ? (uint32_t)kBig << 24 : 0u);
        h.r = rrem;
        map_at(lane)[d] = (uint16_t)(v | (w << 8));
        if (d + 1 > inc)
            improve(d + 1);
        if (K2 == 0)
            return;  // nothing left to split: the parent goes on
        st_hdr(at(lane, base), h);
        c_x = h.x;
        c_y = h.y;
        c_r = h.r;
        pv = true;
        c_pushed += (uint32_t)K2;
        pbase = base;
        base = nb;
        t += 1;
        K = K2;
        d += 1;
        bound = b;
        rrem = (W)0;
        flags = kSel | kDirty | kInLds;
        const int used = nb + HE + K2;
        max_used = used > max_used ? used : max_used;
    }

    __device__ void step() {
        // pop and unmatched, twice if lanes need it: half of the unmatched
        // children are pruned, and their lanes pop on
        for (int i = 0; i < kPops; ++i) {
            const bool need_pop =
                t >= 0 && rrem == (W)0 && !(flags & (kUnm | kSel));
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
        const bool need_ld = (rrem != (W)0 || (flags & kSel)) && !(flags & kInLds);
        if (ballot(need_ld))
            if (need_ld)
                fetch();
        const bool need_sel = (flags & kSel) != 0;
        if (ballot(need_sel))
            if (need_sel)
                select();
        if (flags & kRow) {
            go = ld_w(rows + v);
            if constexpr (DIR)
                gi = ld_w(rows + 2 * NB + v);
            flags &= ~kRow;
        }
        bool found = false;
        int w = 0, b = 0;
        for (int i = 0; i < kEvals; ++i) {
            const bool ev = rrem != (W)0 && !found;
            if (ballot(ev) == 0)
                break;
            if (ev)
                found = evaluate(w, b);
        }
        if (ballot(found)) {
            // where the child's frame starts: above this one, or, where it
            // might not fit, in the wavefront's worst-case area, if no other
            // lane is in it (a lane that has to wait takes its child back)
            int nb = base + HE + K;
            const bool big = found && nb < cap && nb + HE + (b - d - 1) > cap;
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
            if (ballot(found && nb >= cap)) {
                n_big += (unsigned)__builtin_popcountll(ballot(found && nb >= cap));
                if (found && nb >= cap &&
                    (uint32_t)(nb - cap + HE + (b - d - 1)) > big_cap) {
                    fail_lane(kErrStack);  // a broken invariant: past the worst case
                    found = false;
                }
            }
            const int inc0 = inc;
            if (found)
                descend(w, b, nb);
            uint64_t up = ballot(inc > inc0);
            while (up) {  // (rare) tell the wavefront's other searches
                const int l = ctz(up);
                up &= up - 1;
                const int li = rl(inst, l), lv = rl(inc, l);
                if (inst == li && lv > inc)
                    inc = lv;
            }
        }
        n_steps += 1;
        if (ballot(fin))
            finish_units();
    }

    // ---- work sharing inside the wavefront ----

    // Idle lanes take the lowest open frame of busy lanes, one each: lane
    // j-th idle from the j-th lane with a frame below its top.
    __device__ void steal() {
        const bool is_i = t < 0, is_v = t >= 0 && lo_t < t;
        const uint64_t im = ballot(is_i), vm = ballot(is_v);
        const int ni = __builtin_popcountll(im), nv = __builtin_popcountll(vm);
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
        const int vt = shfl_any(t, vl);
        const int vinst = shfl_any(inst, vl), vinc = shfl_any(inc, vl);
        const int vtarget = shfl_any(target, vl);
        wave_sync_global();  // frames written by other lanes
        bool got = false;
        Hdr h;
        h.x = h.y = 0;
        h.r = (W)0;
        for (;;) {
            const bool look = thief && !got && ft < vt;
            if (ballot(look) == 0)
                break;
            if (look) {
                h = ld_hdr(at(vl, fb));
                const int hb = (int)((h.y >> 16) & 0xFFu), hf = (int)(h.y >> 24);
                if ((h.r != (W)0 || (hf & kUnm)) && !(reprune && hb <= vinc)) {
                    got = true;
                } else {
                    fb = (hf & kBig) ? cap : fb + HE + (int)((h.x >> 16) & 0xFFu);
                    ft += 1;
                }
            }
        }
        // the victim's side: its lowest open frame is at or above the one taken
        const int rb = shfl_any(fb, tl), rt = shfl_any(ft, tl), rg = shfl_any(got ? 1 : 0, tl);
        if (robbed) {
            lo_base = rb;
            lo_t = rt;
            if (rg && pv && pbase == rb) {
                c_r = (W)0;
                c_y &= ~((uint32_t)kUnm << 24);
            }
        }
        if (got) {
            Hdr e = h;
            e.r = (W)0;
            e.y &= ~((uint32_t)kUnm << 24);
            st_hdr(at(vl, fb), e);  // nothing is left of it there
            if (inst != vinst)
                flush_lane();
            inst = vinst;
            inc = vinc;
            target = vtarget;
            rows = gadj + (size_t)inst * (NR * NB);
            K = (int)((h.x >> 16) & 0xFFu);
            start_frame((int)(h.x >> 24), h.y, h.r);
            flags |= kDirty;
            const uint32_t src = at(vl, fb + HE);
            const uint32_t dst = at(lane, HE);
            for (int k = 0; ballot(k < K) != 0; ++k) {
                if (k < K) {
                    const Cls<W> c = gget(src + (uint32_t)k * EB);
                    if (k < kc)
                        lput(lane, 0, k, c);
                    else
                        gput(dst + (uint32_t)k * EB, c);
                }
            }
            for (int j = 0; ballot(j < d) != 0; j += 8)
                if (j < d) {
                    const v2u64 x = ld16((uint32_t)vl * stride + 2u * j);
                    st16((uint32_t)lane * stride + 2u * j, x[0], x[1]);
                }
        }
        n_don += (unsigned)__builtin_popcountll(ballot(got));
        wave_sync_global();
    }

    // The lane's only frame, from a header's fields (K is set).
    __device__ void start_frame(int fd, uint32_t y, const W &r) {
        t = 0;
        base = pbase = 0;
        lo_t = lo_base = 0;
        pv = false;
        d = fd;
        v = (int)(y & 0xFFu);
        sel = (int)((y >> 8) & 0xFFu);
        bound = (int)((y >> 16) & 0xFFu);
        rrem = r;
        flags = ((int)(y >> 24) & kSaved) | kInLds | (r != (W)0 ? kRow : 0);
    }

    // ---- work sharing between wavefronts ----

    __device__ void raise_flag(unsigned bits) {
        if (lane == 0)
            raise_any(bits);
    }
    __device__ void raise_any(unsigned bits) {
        if (bits & kFlagStop)
            __hip_atomic_store(&P.g->stop, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int k = 0; k < kRings; ++k)
            __hip_atomic_fetch_or(&P.g->xcd[k].flag, bits, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
    }
    // A check failed in the lanes that call this (possibly few of them).
    __device__ void fail_lane(unsigned code) {
        __hip_atomic_store(&P.g->error, code, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        raise_any(kFlagStop);
    }

    // A free slot in this XCD's ring, else in the next rings.
    __device__ bool reserve(int &ring, unsigned long long &ticket) {
        const unsigned long long mask = (unsigned long long)P.ring_slots - 1;
        int ok = 0, rr = 0;
        unsigned long long tk = 0;
        if (lane == 0) {
            for (int k = 0; k < kRings && !ok; ++k) {
                const int r = (my_ring + k) & (kRings - 1);
                unsigned long long *sq = P.seq + (size_t)r * P.ring_slots;
                for (int tries = 0; tries < 4; ++tries) {
                    const unsigned long long tl = ld_rlx(&P.g->ring[r].tail);
                    const unsigned long long s = ld_rlx(&sq[tl & mask]);
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

    // Lane l's lowest open frame below its top goes to the queue; false if
    // it has none, or no slot is free.
    __device__ bool donate(int l) {
        int fb = rl(lo_base, l), ft = rl(lo_t, l);
        const int lt = rl(t, l), linc = rl(inc, l);
        Hdr h;
        bool got = false;
        while (ft < lt) {
            h = ld_hdr(at(l, fb));
            h.x = sc(h.x);
            h.y = sc(h.y);
            h.r = sc(h.r);
            const int hb = (int)((h.y >> 16) & 0xFFu), hf = (int)(h.y >> 24);
            if ((h.r != (W)0 || (hf & kUnm)) && !(reprune && hb <= linc)) {
                got = true;
                break;
            }
            fb = (hf & kBig) ? cap : fb + HE + (int)((h.x >> 16) & 0xFFu);
            ft += 1;
        }
        if (lane == l) {
            lo_base = fb;
            lo_t = ft;
        }
        if (!got || (int)(h.x >> 24) > P.donate_depth)
            return false;
        unsigned long long ticket;
        int ring;
        if (!reserve(ring, ticket))
            return false;
        const unsigned long long mask = (unsigned long long)P.ring_slots - 1;
        const size_t idx = (size_t)ring * P.ring_slots + (size_t)(ticket & mask);
        uint8_t *slot = P.slots + idx * (size_t)P.slot_bytes;
        const int fK = (int)((h.x >> 16) & 0xFFu), fd = (int)(h.x >> 24);
        const int ji = rl(inst, l);
        RecHdr<W> rh;
        rh.inst = (uint32_t)ji;
        rh.K = (uint8_t)fK;
        rh.d = (uint8_t)fd;
        rh.v = (uint8_t)(h.y & 0xFFu);
        rh.sel = (uint8_t)((h.y >> 8) & 0xFFu);
        rh.bound = (uint8_t)((h.y >> 16) & 0xFFu);
        rh.flags = (uint8_t)((h.y >> 24) & kSaved);
        rh.lsel = rh.rsel = 0;
        rh.pad[0] = rh.pad[1] = rh.pad[2] = rh.pad[3] = 0;
        rh.rrem = h.r;
        constexpr int HW = (int)(sizeof(RecHdr<W>) + 7) / 8;
        if (lane == 0) {
            unsigned long long ws[HW] = {};
            __builtin_memcpy(ws, &rh, sizeof(rh));
            for (int i = 0; i < HW; ++i)
                st_agent((unsigned long long *)slot + i, ws[i]);
        }
        // mapping (four pairs a word) and classes
        unsigned long long *rmap = (unsigned long long *)(slot + rec_map_off<W>());
        for (int i = lane; 4 * i < fd; i += 64)
            st_agent(rmap + i, *(glb_ptr<unsigned long long>)(wst + (uint32_t)l * stride + 8u * i));
        unsigned long long *rcls = (unsigned long long *)(slot + rec_cls_off<W>());
        const uint32_t src = at(l, fb + HE);
        for (int i = lane; i < fK * (EB / 8); i += 64)
            st_agent(rcls + i, *(glb_ptr<unsigned long long>)(wst + src + 8u * i));
        if (lane == 0) {
            h.r = (W)0;
            h.y &= ~((uint32_t)kUnm << 24);
            st_hdr(at(l, fb), h);  // nothing is left of it here
            a_add_rlx(&P.open[ji], 1);
            a_add_rlx(&P.g->open_total, 1);
        }
        if (lane == l && pv && pbase == fb) {
            c_r = (W)0;
            c_y &= ~((uint32_t)kUnm << 24);
        }
        // every word of the record has been written before its sequence
        // number says so
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);
        if (lane == 0)
            st_rlx(&P.seq[idx], ticket + 1);
        wave_sync_global();
        n_don += 1;
        return true;
    }

    // Lane l works on instance i from now on (per-lane values; uniform i).
    __device__ void enter(int i) {
        if (inst != i)
            flush_lane();
        const DevInst di = P.inst[i];
        inst = i;
        target = (int)di.target;
        rows = gadj + (size_t)i * (NR * NB);
        inc = 0;
        set_inc(read_inc(di, i));
    }
    // The incumbent, or 255 where the instance needs no more search.
    __device__ int read_inc(const DevInst &di, int i) const {
        int g = ld_rlx(&P.inc[di.inc_slot]);
        if (di.twin >= 0 && ld_rlx(&P.open[di.twin]) == 0 && !ld_rlx(&P.dead[di.twin]))
            g = 255;  // the twin's search already finished
        if (di.dead_on && ld_rlx(&P.dead[i]))
            g = 255;  // given up as a dead end
        return g;
    }
    // One more unit of instance i arrived: if the wavefront already works on
    // it, the two are one from now on.
    __device__ void merge_unit(int i) {
        if (ballot(t >= 0 && inst == i) != 0 && lane == 0) {
            a_add_rlx(&P.open[i], -1);
            a_add_rlx(&P.g->open_total, -1);
        }
    }

    // Take a queued node into lane l: from this XCD's ring, else from one
    // other ring, a different one on each call.
    __device__ bool take_record(int l) {
        const unsigned long long mask = (unsigned long long)P.ring_slots - 1;
        int ok = 0, rr = 0;
        unsigned long long hd = 0;
        if (lane == 0) {
            steal_from = (steal_from + 1) & (kRings - 1);
            if (steal_from == my_ring)
                steal_from = (steal_from + 1) & (kRings - 1);
            for (int k = 0; k < 2 && !ok; ++k) {
                const int r = k == 0 ? my_ring : steal_from;
                unsigned long long *sq = P.seq + (size_t)r * P.ring_slots;
                for (int tries = 0; tries < 4; ++tries) {
                    const unsigned long long h = ld_rlx(&P.g->ring[r].head);
                    const unsigned long long s = ld_rlx(&sq[h & mask]);
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
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        hd = rl_ull(hd, 0);
        const int ring = rl(rr, 0);
        const size_t idx = (size_t)ring * P.ring_slots + (size_t)(hd & mask);
        const uint8_t *slot = P.slots + idx * (size_t)P.slot_bytes;
        constexpr int HW = (int)(sizeof(RecHdr<W>) + 7) / 8;
        unsigned long long ws[HW];
        for (int i = 0; i < HW; ++i)
            ws[i] = ld_agent((const unsigned long long *)slot + i);
        RecHdr<W> rh;
        __builtin_memcpy(&rh, ws, sizeof(rh));
        const int ri = sc((int)rh.inst);
        const int rK = sc((int)rh.K), rd = sc((int)rh.d);
        const uint32_t y = sc((uint32_t)rh.v | ((uint32_t)rh.sel << 8) |
                              ((uint32_t)rh.bound << 16) | ((uint32_t)rh.flags << 24));
        const W rr_ = sc((W)rh.rrem);
        // the record's words go straight to lane l's stack
        const unsigned long long *rmap = (const unsigned long long *)(slot + rec_map_off<W>());
        for (int i = lane; 4 * i < rd; i += 64)
            *(glb_ptr<unsigned long long>)(wst + (uint32_t)l * stride + 8u * i) =
                ld_agent(rmap + i);
        const unsigned long long *rcls = (const unsigned long long *)(slot + rec_cls_off<W>());
        const uint32_t dst = at(l, HE);
        for (int i = lane; i < rK * (EB / 8); i += 64)
            *(glb_ptr<unsigned long long>)(wst + dst + 8u * i) = ld_agent(rcls + i);
        // every lane's loads of the slot have returned before it is handed back
        __builtin_amdgcn_s_waitcnt(0);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        if (lane == 0)
            st_rlx(&P.seq[idx], hd + (unsigned long long)P.ring_slots);
        wave_sync_global();
        merge_unit(ri);
        if (lane == l) {
            enter(ri);
            K = rK;
            start_frame(rd, y, rr_);
            flags &= ~kInLds;  // (all of it is in HBM)
            if (bound <= inc) {
                rrem = (W)0;
                flags = 0;
            }
        }
        n_pops += 1;
        return true;
    }

    // The next unstarted instances, one per idle lane (their work units were
    // counted by the reset): several at a time while there are many more
    // than wavefronts.
    __device__ bool claim_instances() {
        if (!roots_left)
            return false;
        const uint64_t im = ballot(t < 0);
        int first = 0, n = 0;
        if (lane == 0) {
            const unsigned nx = ld_rlx(&P.g->next_inst);
            if (nx < (unsigned)P.count) {
                const unsigned left = (unsigned)P.count - nx;
                unsigned want = left / (2u * gridDim.x * (blockDim.x >> 6));
                const unsigned room = (unsigned)__builtin_popcountll(im);
                want = want < 1u ? 1u : want > room ? room : want;
                if (P.single_wave)
                    want = 1;
                const unsigned x = a_addu(&P.g->next_inst, want);
                if (x < (unsigned)P.count) {
                    first = (int)x;
                    n = (int)((unsigned)P.count - x < want ? (unsigned)P.count - x : want);
                }
            }
        }
        first = rl(first, 0);
        n = rl(n, 0);
        if (n == 0) {
            roots_left = false;
            return false;
        }
        const int r = mbcnt(im);
        if (t < 0 && r < n) {
            const int i = first + r;
            enter(i);
            const DevInst di = P.inst[i];
            const Cls<W> *rc = (const Cls<W> *)P.rootcls + di.cls_off;
            const uint32_t dst = at(lane, HE);
            K = (int)di.K0;
            int sum = 0;
            for (int k = 0; ballot(k < K) != 0; ++k) {
                if (k < K) {
                    const Cls<W> c = ld_cls(rc + k);
                    if (k < kc)
                        lput(lane, 0, k, c);
                    else
                        gput(dst + (uint32_t)k * EB, c);
                    const int nl = popc(c.L), nr = popc(c.R);
                    sum += nl < nr ? nl : nr;
                }
            }
            c_unm += 1;  // the root
            start_frame(0, (uint32_t)sum << 16, (W)0);
            flags = (K == 0 || sum <= inc) ? 0 : kSel | kDirty | kInLds;
        }
        return true;
    }

    // Lanes whose last frame ended: a unit of the wavefront ends with the
    // last lane on its instance.
    __device__ void finish_units() {
        uint64_t fm = ballot(fin);
        while (fm) {
            const int ji = rl(inst, ctz(fm));
            fm &= ~ballot(inst == ji);
            if (ballot(t >= 0 && inst == ji) == 0) {
                if (P.node_limit > 0)
                    flush_nodes();
                if (lane == 0 && !stop) {
                    const int r = a_add_rlx(&P.open[ji], -1);
                    if (r == 1)
                        __hip_atomic_store(&P.t_proof[ji], now_ticks(), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                    if (a_add_rlx(&P.g->open_total, -1) == 1)
                        raise_any(kFlagDone);
                }
            }
        }
        fin = false;
    }

    // ---- counts ----

    // The lane's nodes since its last flush, to its instance's count.
    __device__ void flush_lane() {
        if (c_child + c_unm != 0)
            a_add64(&P.nodes[inst], (unsigned long long)c_child + c_unm);
        n_child += c_child;
        n_ncls += c_ncls;
        n_pushed += c_pushed;
        c_child = c_unm = c_ncls = c_pushed = 0;
    }
    __device__ void flush_nodes() {
        const unsigned long long np = (unsigned long long)c_child + c_unm;
        const unsigned long long sum = lanes_total(np);
        flush_lane();
        if (lane == 0 && sum && P.node_limit > 0) {
            const unsigned long long tot = a_add64(&P.g->node_total, sum) + sum;
            if ((long long)tot > P.node_limit)
                raise_any(kFlagStop);
        }
    }
    DEV unsigned long long lanes_total(unsigned long long x) {
        // (24-bit pieces: 64 of them sum below 2^31)
        return (unsigned long long)(unsigned)wave_sum((int)(x & 0xFFFFFFu)) +
               ((unsigned long long)(unsigned)wave_sum((int)((x >> 24) & 0xFFFFFFu)) << 24) +
               ((unsigned long long)(unsigned)wave_sum((int)((x >> 48) & 0xFFFFu)) << 48);
    }

    // Dead-end forecast (paper Sec. IV.A), as in the other kernels.
    __device__ void forecast_dead_ends() {
        if (t >= 0 && P.inst[inst].dead_on) {
            const unsigned long long n = ld_rlx(&P.nodes[inst]);
            const unsigned long long b = ld_rlx(&P.best_nodes[inst]);
            const unsigned long long since = n > b ? n - b : 0ull;
            unsigned long long thr = (unsigned long long)P.dead_abs;
            if (P.dead_rel > 0 && (unsigned long long)P.dead_rel * b > thr)
                thr = (unsigned long long)P.dead_rel * b;
            if (since > thr) {
                st_rlx(&P.dead[inst], 1);
                inc = 255;
            }
        }
    }

    // Periodic: refresh incumbents, honour limits, keep the queue stocked.
    __device__ void check() {
        since_check = 0;
        unsigned fl = 0;
        unsigned long long hd = 0, tl = 0;
        const bool may_donate = !P.single_wave && P.donate_low >= 0;
        if (lane == 0) {
            fl = ld_rlx(&P.g->xcd[my_ring].flag);
            if (may_donate) {
                tl = ld_rlx(&P.g->ring[my_ring].tail);
                hd = ld_rlx(&P.g->ring[my_ring].head);
            }
        }
        if (t >= 0) {
            const DevInst di = P.inst[inst];
            set_inc(read_inc(di, inst));
        }
        if (rl(fl, 0)) {
            stop = true;
            return;
        }
        if (now_ticks() - t_start > P.limit_ticks) {
            raise_flag(kFlagStop);
            stop = true;
            return;
        }
        if (P.node_limit > 0 || P.dead_abs > 0 ||
            ballot((c_child | c_unm | c_ncls | c_pushed) > (1u << 30)))
            flush_nodes();
        if (P.dead_abs > 0)
            forecast_dead_ends();
        if (may_donate) {
            long long waiting = (long long)(rl_ull(tl, 0) - rl_ull(hd, 0));
            if (waiting < P.donate_low) {
                wave_sync_global();
                // the shallowest frames first
                for (int tries = 0; tries < 4 && waiting < P.donate_low; ++tries) {
                    const bool c = t >= 0 && lo_t < t;
                    const uint32_t key =
                        wave_min(c ? ((uint32_t)(d - t + lo_t) << 8) | (uint32_t)lane : ~0u);
                    if (key == ~0u)
                        break;
                    if (donate((int)(key & 63u)))
                        waiting += 1;
                }
            }
        }
    }

    // Work for a wavefront with idle lanes; false if none was found.
    __device__ bool refill() {
        if (!P.single_wave) {
            const uint64_t im = ballot(t < 0);
            if (take_record(ctz(im)))
                return true;
        } else if (ballot(t >= 0) != 0) {
            return false;  // one search only: the sequential order
        }
        return claim_instances();
    }

    __device__ void main_loop() {
        t_start = now_ticks();
        if (lane == 0)
            a_min64(&P.g->t0, t_start);
        const int check_interval = sc(P.check_interval);
        const bool share = !P.single_wave && P.donate_low >= 0;
        int backoff = 0, look = 0, look_gap = 8, since_steal = 0;
        unsigned long long t_busy0 = 0;
        bool busy = false;
        for (;;) {
            uint64_t am = ballot(t >= 0);
            if (am != ~0ull) {
                const int idle = 64 - __builtin_popcountll(am);
                if (share && am != 0 && (idle >= 8 || ++since_steal >= 4)) {
                    since_steal = 0;
                    steal();
                    am = ballot(t >= 0);
                }
                // a wavefront with no work at all, or (now and then: a failed
                // look costs a queue round trip) with few lanes busy, looks
                // outside
                if (am == 0 || (__builtin_popcountll(am) <= 32 && ++look >= look_gap)) {
                    look = 0;
                    if (refill())
                        look_gap = 8;
                    else if (am != 0)
                        look_gap = look_gap < 512 ? 2 * look_gap : 512;
                }
            }
            if (ballot(t >= 0) == 0) {
                if (busy) {
                    n_busy += now_ticks() - t_busy0;
                    busy = false;
                }
                unsigned fl = 0;
                if (lane == 0)
                    fl = ld_rlx(&P.g->xcd[my_ring].flag);
                if (rl(fl, 0))
                    break;  // stopped, or no work is left anywhere
                if (now_ticks() - t_start > P.limit_ticks) {
                    raise_flag(kFlagStop);
                    break;
                }
                const int bmax = P.backoff_max;
                backoff = backoff ? (2 * backoff < bmax ? 2 * backoff : bmax) : 1;
                const unsigned long long t_sleep = now_ticks();
                for (int i = 0; i < backoff; ++i)
                    __builtin_amdgcn_s_sleep(127);
                n_sleep += now_ticks() - t_sleep;
                continue;
            }
            backoff = 0;
            if (!busy) {
                t_busy0 = now_ticks();
                busy = true;
            }
            step();
            if (stop)
                break;
            if (++since_check >= check_interval) {
                check();
                if (stop)
                    break;
            }
        }
        if (busy)
            n_busy += now_ticks() - t_busy0;
        flush_lane();
        const unsigned long long child = lanes_total(n_child), ncls = lanes_total(n_ncls),
                                 pushed = lanes_total(n_pushed);
        const int mu = (int)~wave_min(~(uint32_t)max_used);
        if (lane == 0) {
            a_add64(&P.g->batches, n_steps);
            a_add64(&P.g->children, child);
            a_add64(&P.g->lane_slots, child);
            a_add64(&P.g->donations, n_don);
            a_add64(&P.g->pops, n_pops);
            a_add64(&P.g->busy_ticks, n_busy);
            a_add64(&P.g->hbm_frames, n_big);
            a_add64(&P.g->pushed_classes, pushed);
            a_add64(&P.g->sleep_ticks, n_sleep);
            a_add64(&P.g->node_classes, ncls);
            __hip_atomic_fetch_max(&P.g->max_stack, mu, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
    }
};

template <typename W, bool DIR>
__global__ void __launch_bounds__(256, 2) mcs_lane_kernel(SearchParams Pk) {
    extern __shared__ __align__(16) char smem[];
    __shared__ SearchParams P;
    if (threadIdx.x == 0)
        P = Pk;
    __syncthreads();
    const int wv = (int)threadIdx.x >> 6;
    if (Pk.single_wave && (blockIdx.x != 0 || wv != 0))
        return;
    LaneSearch<W, DIR> s(P, (lds_ptr<char>)smem + (size_t)sc(wv) * (size_t)Pk.lds_per_wave,
                         sc((int)(blockIdx.x * (blockDim.x >> 6)) + wv));
    s.main_loop();
}

}  // namespace mcs

// The kernel for rows of word_bytes (4, 8, 16 or 32), directed or not.
extern "C" void *mcs_internal_lane_kernel(int word_bytes, int directed) {
    using namespace mcs;
    switch (word_bytes) {
    case 4: return directed ? (void *)mcs_lane_kernel<uint32_t, true> : (void *)mcs_lane_kernel<uint32_t, false>;
    case 8: return directed ? (void *)mcs_lane_kernel<uint64_t, true> : (void *)mcs_lane_kernel<uint64_t, false>;
    case 16: return directed ? (void *)mcs_lane_kernel<u128, true> : (void *)mcs_lane_kernel<u128, false>;
    case 32: return directed ? (void *)mcs_lane_kernel<u256, true> : (void *)mcs_lane_kernel<u256, false>;
    }
    return nullptr;
}
