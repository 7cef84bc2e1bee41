// count.hip — gfx950 kernels that execute counting plans.
//
// Algorithm 2 (plan execution) run by wavefronts.  Each wave is a worker
// that takes tasks from two device queues: first-level sub-ranges of hub
// roots (split by the split kernel so that other waves can take them, the
// work-stealing of Algorithm 2's parallel loop), then chunks of ordinary
// roots.  A task is explored depth-first, one level buffer per plan level;
// each buffer holds a window of partial matches, and every expansion is
// flattened across the window so that the 64 lanes stay busy even when
// adjacency lists are short (power-law graphs have mostly short lists).
//
// Per element of a base list a lane checks, in order: injectivity against
// the bound nodes (visited marks), the degree thresholds, and membership in
// every other constraint list: one bit test when the list is long enough to
// have a dense row (an n-bit membership row built at graph load, the HBM
// analogue of staging a hub's list), else a binary search of the sorted
// uint32 list.  The survivors are compacted with a 64-bit ballot and a
// popcount.  The leaf group of a plan is counted, not enumerated (leaf_set): the
// heads of long lists' rows word by word (word_scan), the rest of long lists in
// chunks (chunk_scan), short lists flattened across the window, there against a
// bit map in LDS of a list that the window shares where it pays (use_filter).
// One leaf adds the set sizes up; several evaluate the planner's
// inclusion-exclusion terms over them in 128-bit integers.  Totals are
// unsigned 128-bit, kept as (lo, hi) uint64 pairs updated with 64-bit atomics
// and an explicit carry.
//
// Nothing here is a dense contraction, so no matrix cores are used; the
// kernels are bound by memory latency and bandwidth of list reads.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "donate.h"
#include "kernels.h"
#include "u128.h"

namespace xm {

static_assert(sizeof(PlanDesc) % 4 == 0, "plan descriptors are copied in 32-bit words");

constexpr uint32_t kSkip = 0xFFFFFFFFu;
constexpr uint32_t kIdlePolls = 1u << 13;  // polls a waiting wave makes for donated work
constexpr uint32_t kNapMax = 128;          // longest pause between two polls, in sleeps of 512 clocks (~27 us)
// Work donation: clocks a task runs before it looks whether other waves wait,
// and between such looks (~0.4 ms); partial matches of one parent in a donated
// range, at least; clocks a donated range should take; clocks a task runs
// before it donates single parents.  The costs are in the control words: a line
// serves ~70 accesses a us, so looks, donated tasks and waiters have to stay few.
// A tenth of the roots of R-MAT 16 took, with ranges of 2^18 / 2^20 / 2^21 clocks
// and 512 waiters, 730 / 60 / - ms, with 256 waiters and 2^21 40 ms, without
// ranges 48 ms; all idle waves waiting with long pauses 51 ms (while donors still
// polled until the queue was empty; now 31 ms.  With 512 waiters now: a 6-vertex
// pattern on 1/17 of R-MAT 14's roots 152 / 132 ms, stars on R-MAT 12 0.56 / 0.59).
constexpr uint32_t kDonateClocks = 1u << 20;
constexpr uint32_t kDonatePiece = 64;
constexpr uint32_t kDonateWork = 1u << 21;
constexpr uint32_t kDonateParents = 1u << 22;
constexpr uint32_t kComplete = 0x80000000u;
// Base lists at least this long are scanned by the whole wave on their own
// (wide_scan).  Measured at 32 / 64 / 128: unreduced motifs on R-MAT 16 192 /
// 174 / 181 ms, 96 plans on R-MAT 22 414 / 393 / 392 ms: one tile per scan is
// the shortest list that pays for reading the parent's probes.
constexpr uint32_t kWideMin = 64;
// Words a base element is worth in the dense head of a row.  A 16-byte row load
// takes 17 TD clocks for 256 words, a row test of an element up to one clock
// and, when it misses L2, a whole line.  Measured at 2 / 3 / 4 / 8 (none): 96
// plans on R-MAT 22 347 / 348 / 351 / 373 (382) ms, C5 + chord on R-MAT 20 72 /
// - / 72 / 75 (88), motifs on R-MAT 16 19.7 / 20.4 / 21.2 / 22.3 (21.3),
// unreduced 154 / 156 / 160 / 182 (155).
constexpr uint32_t kDenseWords = 2;

__device__ __forceinline__ uint32_t uni(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ uint32_t lane_id() {
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}
__device__ __forceinline__ uint32_t rank_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
// Make this wave's global and LDS writes visible to its other lanes.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
}

// Wave-wide inclusive scans (sum, max) over the 64 lanes with DPP row
// shifts and row broadcasts: 6 VALU steps, no LDS traffic.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ uint32_t scan_incl(uint32_t v, uint32_t) {
    v += dpp_<0x111, 0xf>(v);  // row_shr:1
    v += dpp_<0x112, 0xf>(v);  // row_shr:2
    v += dpp_<0x114, 0xf>(v);  // row_shr:4
    v += dpp_<0x118, 0xf>(v);  // row_shr:8
    v += dpp_<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    v += dpp_<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ __forceinline__ uint32_t scan_max(uint32_t v) {
    v = max(v, dpp_<0x111, 0xf>(v));
    v = max(v, dpp_<0x112, 0xf>(v));
    v = max(v, dpp_<0x114, 0xf>(v));
    v = max(v, dpp_<0x118, 0xf>(v));
    v = max(v, dpp_<0x142, 0xa>(v));
    v = max(v, dpp_<0x143, 0xc>(v));
    return v;
}

// Sorted-list membership: branchless search for the last element <= x.
template <class P>
__device__ __forceinline__ bool contains(P a, uint32_t len, uint32_t x) {
    if (len == 0) return false;
    uint32_t base = 0, n = len;
    while (n > 1) {
        uint32_t h = n >> 1;
        base = (a[base + h] <= x) ? base + h : base;
        n -= h;
    }
    return a[base] == x;
}

__device__ __forceinline__ const uint32_t* adj_of(const DevGraph& g, uint32_t dir) {
    return dir ? g.in_adj : g.out_adj;
}
__device__ __forceinline__ const uint32_t* off_of(const DevGraph& g, uint32_t dir) {
    return dir ? g.in_off : g.out_off;
}

// The probe of list (dir, node nd) at adjacency offset o with length l: the
// list itself, or its dense row (length kRowLen) when it has one.
__device__ __forceinline__ const uint32_t* probe_ref(const DevGraph& g, uint32_t dir, uint32_t nd, uint32_t o,
                                                     uint32_t& l) {
    if (l >= g.row_min) {
        const uint2 r = g.row_of[nd];
        const uint32_t row = dir ? r.y : r.x;
        if (row != kSkip) {
            l = kRowLen;
            return g.rows + (uint64_t)row * g.row_words;
        }
    }
    return adj_of(g, dir) + o;
}

// A list or row address put together from two words.  The address space is
// stated: the compiler cannot infer it from an integer, and a flat load
// would also go through the LDS path and its wait counter.
typedef const __attribute__((address_space(1))) uint32_t* gptr;
__device__ __forceinline__ gptr join_ptr(uint32_t lo, uint32_t hi) {
    return reinterpret_cast<gptr>(((uint64_t)hi << 32) | lo);
}

// Any address that may be read (a lane with nothing to probe reads it and
// ignores the value).
__device__ __forceinline__ const uint32_t* safe_ptr(const DevGraph& g) {
    return reinterpret_cast<const uint32_t*>(g.deg);
}

// Per-level constraint fields, loaded once into scalar registers.
struct LK {
    uint32_t n_cons, reuse, inj, deg_check, extra, dirm, dmin_out, dmin_in, gt, lt;
    uint64_t lvlb;
    __device__ __forceinline__ uint32_t lvl(uint32_t c) const { return (uint32_t)(lvlb >> (3 * c)) & 7u; }
    __device__ __forceinline__ uint32_t dir(uint32_t c) const { return (dirm >> c) & 1u; }
};
__device__ __forceinline__ LK load_lk(const LevelDesc& D, const KArgs& a) {
    LK k;
    k.n_cons = uni(D.n_cons);
    if (k.n_cons > a.maxc) {
        // the per-wave probe arrays hold maxc constraints: never index past them
        atomicOr(&a.ctl[kCtlBadPlan], 1u);
        k.n_cons = a.maxc;
    }
    k.reuse = uni(D.reuse);
    k.inj = uni(D.inj);
    k.deg_check = uni(D.deg_check);
    k.extra = uni(D.extra);
    k.dirm = uni(D.dir_mask);
    k.dmin_out = uni(D.dmin_out);
    k.dmin_in = uni(D.dmin_in);
    k.gt = uni(D.gt);
    k.lt = uni(D.lt);
    k.lvlb = ((uint64_t)uni((uint32_t)(D.lvl_bits >> 32)) << 32) | uni((uint32_t)D.lvl_bits);
    return k;
}

// Unsigned 128-bit atomic add into (lo, hi) with an overflow flag.
__device__ void add_u128(unsigned long long* c, unsigned long long lo, unsigned long long hi,
                         uint32_t* flag) {
    if (lo) {
        unsigned long long old = atomicAdd(c, lo);
        if (old + lo < old) {
            hi += 1;
            if (hi == 0) atomicOr(flag, 1u);
        }
    }
    if (hi) {
        unsigned long long old = atomicAdd(c + 1, hi);
        if (old + hi < old) atomicOr(flag, 1u);
    }
}

// Per-wave LDS carve-out.
struct Lds {
    uint32_t* bound;     // [kMaxK][64]
    uint32_t* anc;       // [kMaxK][64]
    uint32_t* base_lo;   // [64]: address of the parent's base list (low word)
    uint32_t* base_len;  // [64]
    uint32_t* base_hi;   // [64]: (high word)
    uint32_t* incl;      // [64]
    uint32_t* segcnt;    // [64]
    uint32_t* mark;      // [128]: tile parent marks
    uint32_t* slot_len;  // [maxc][64]: probe k of the parent: list length, kRowLen, or kSkip
    uint32_t* slot_lo;   // [maxc][64]: address of the list or of the dense row (low word)
    uint32_t* slot_hi;   // [maxc][64]: (high word)
    uint32_t* hist;      // [signature masks][64]
    uint32_t* filt;      // [filt_words]: bit map of a shared list, or embeddings to be listed
    uint32_t* st;        // wave state: cur[8], pofs[8], n[8], a donated id range: level, from, to;
                         // the filter's list: address (2 words), length; sequence
                         // number after the wave's last donated task
    uint32_t* mbuf;      // [kMergeChunk]: probe-list chunk of the cooperative merge
};

__device__ __forceinline__ Lds carve(uint32_t* w, uint32_t rows, uint32_t maxc, bool merge,
                                        uint32_t filt_words) {
    // the arrays of fixed size come first: their addresses are one register
    // plus constants
    Lds s;
    s.base_lo = w;
    s.base_len = w + 64;
    s.base_hi = w + 128;
    s.incl = w + 192;
    s.segcnt = w + 256;
    s.mark = w + 320;
    s.st = w + 448;
    s.bound = w + 480;
    s.anc = s.bound + rows * 64;
    s.slot_len = s.anc + rows * 64;
    s.slot_lo = s.slot_len + maxc * 64;
    s.slot_hi = s.slot_lo + maxc * 64;
    s.mbuf = s.slot_hi + maxc * 64;
    s.filt = s.mbuf + (merge ? kMergeChunk : 0);
    s.hist = s.filt + filt_words;
    return s;
}

struct Lvl {
    uint32_t* node;
    uint32_t* parent;  // level 0: first-level range start
    uint32_t* segb;
    uint32_t* segc;    // child count | kComplete
    uint32_t* aux;     // level 0: first-level range end
};

__device__ __forceinline__ Lvl lvl_arrays(uint32_t* scr, uint32_t cap, uint32_t l) {
    uint32_t* b = scr + (size_t)l * kLvlArrays * cap;
    return {b, b + cap, b + 2 * cap, b + 3 * cap, b + 4 * cap};
}

struct Ctx {
    const KArgs* a;
    const PlanDesc* P;
    uint32_t pi;
    Lds s;
    uint32_t* scr;
    uint32_t lane;
    unsigned long long acc_lo, acc_hi;  // per-lane 128-bit partial (leaf groups)
    bool ovf;                           // this lane's partial or a leaf-group term left the 128-bit range
    bool stop;                          // the cancel flag was seen: leave the task
    uint32_t polls;                     // leaf blocks since the last look at the cancel flag
    uint32_t begun, looked;             // clock of the task's start, and of its last look for waiting waves
};

// First-level base list length of root r for plan P (shortest constraint list).
__device__ __forceinline__ uint32_t level1_len(const DevGraph& g, const PlanDesc* P, uint32_t r) {
    const LevelDesc& D = P->lvl[1];
    uint32_t best = kSkip;
    for (uint32_t c = 0; c < D.n_cons; c++) {
        const uint32_t* off = off_of(g, D.cons_dir[c]);
        uint32_t l = off[r + 1] - off[r];
        best = l < best ? l : best;
    }
    return best;
}

// Number of elements <= x in the sorted list a[0, n).
__device__ __forceinline__ uint32_t count_le(const uint32_t* a, uint32_t n, uint32_t x) {
    uint32_t lo = 0;
    while (n > 0) {
        const uint32_t h = n >> 1;
        if (a[lo + h] <= x) {
            lo += h + 1;
            n -= h + 1;
        } else {
            n = h;
        }
    }
    return lo;
}

// Number of entries below x in the sorted array a[0, n).
__device__ __forceinline__ uint32_t count_lt(const uint32_t* a, uint32_t n, uint32_t x) {
    return x ? count_le(a, n, x - 1u) : 0u;
}

// Symmetry breaking: the part of the sorted list a[0, len) that lies above
// the largest (lt = 0) or below the smallest (lt = 1) bound image among the
// levels in gt (levels < lv) of this lane's partial match.
__device__ __forceinline__ void sym_trim(const Lds& s, uint32_t gt, uint32_t lt, uint32_t lv, uint32_t lane,
                                         const uint32_t*& a, uint32_t& len) {
    uint32_t lo = 0xFFFFFFFFu, hi = 0;
    for (uint32_t l = 0; l < lv; l++)
        if ((gt >> l) & 1u) {
            const uint32_t b = s.bound[l * 64 + lane];
            lo = b < lo ? b : lo;
            hi = b > hi ? b : hi;
        }
    if (lt) {
        len = lo ? count_le(a, len, lo - 1u) : 0u;
    } else {
        const uint32_t skip = count_le(a, len, hi);
        a += skip;
        len -= skip;
    }
}

// Phase A of a level: lane = one partial match (parent) of the window.  Walks
// the parent chain into LDS (bound nodes, ancestor indices), picks the base
// list and writes the probes (the other constraint lists, long ones as their
// dense rows) into the parent's probe slots.  Returns the base length; for a
// leaf pass brow becomes the dense row of the base list (kSkip: none), bskip
// the elements cut off its front, and flen the length of the shortest list of a
// constraint outside `shared` (kSkip: none).
template <bool IS_SIG>
__device__ __forceinline__ uint32_t phase_a(Ctx& C, const LK& D, uint32_t lv, uint32_t p, bool pv, bool walk,
                                            uint32_t shared, uint32_t& flen, uint32_t& brow, uint32_t& bskip) {
    const KArgs& a = *C.a;
    const DevGraph& g = a.g;
    const uint32_t lane = C.lane;
    uint32_t len = 0;
    brow = flen = kSkip;
    bskip = 0;
    if (!pv) {
        C.s.base_len[lane] = 0;
        return 0;
    }
    if (walk) {
        uint32_t idx = p;
        for (int l = (int)lv - 1; l >= 0; --l) {
            Lvl F = lvl_arrays(C.scr, a.cap, (uint32_t)l);
            C.s.bound[l * 64 + lane] = F.node[idx];
            C.s.anc[l * 64 + lane] = idx;
            if (l > 0) idx = F.parent[idx];
        }
    }
    auto put = [&](uint32_t k, const uint32_t* ptr, uint32_t l) {
        const uint64_t v = reinterpret_cast<uint64_t>(ptr);
        C.s.slot_len[k * 64 + lane] = l;
        C.s.slot_lo[k * 64 + lane] = (uint32_t)v;
        C.s.slot_hi[k * 64 + lane] = (uint32_t)(v >> 32);
    };
    const uint32_t* base = nullptr;
    uint32_t k = 0;
    bool fetched = false;
    if (D.reuse != kNoReuse) {
        uint32_t r = D.reuse;
        uint32_t ai = C.s.anc[(r - 1) * 64 + lane];
        Lvl F = lvl_arrays(C.scr, a.cap, r - 1);
        uint32_t sc = F.segc[ai];
        if (sc & kComplete) {
            base = lvl_arrays(C.scr, a.cap, r).node + F.segb[ai];
            len = sc & ~kComplete;
            for (uint32_t c = 0; c < D.n_cons; c++) {
                if (!((D.extra >> c) & 1u)) continue;
                const uint32_t nd = C.s.bound[D.lvl(c) * 64 + lane];
                const uint32_t* off = off_of(g, D.dir(c));
                const uint32_t o = off[nd];
                uint32_t l = off[nd + 1] - o;
                if (!((shared >> c) & 1u) && l < flen) flen = l;
                const uint32_t* ptr = probe_ref(g, D.dir(c), nd, o, l);
                put(k++, ptr, l);
            }
            fetched = true;
        }
    }
    if (!fetched) {
        // the shortest list is the base; the others are probed
        uint32_t best = kSkip, bc = 0, bo = 0;
        uint32_t dbest = kSkip, dc = 0, dof = 0, dlv = 0;  // shortest list at the deepest bound level
        for (uint32_t c = 0; c < D.n_cons; c++) {
            const uint32_t nd = C.s.bound[D.lvl(c) * 64 + lane];
            const uint32_t* off = off_of(g, D.dir(c));
            const uint32_t o = off[nd], l = off[nd + 1] - o;
            if (!((shared >> c) & 1u) && l < flen) flen = l;
            if (l < best) {
                best = l;
                bc = c;
                bo = o;
            }
            if (D.lvl(c) > dlv || (D.lvl(c) == dlv && l < dbest)) {
                dlv = D.lvl(c);
                dbest = l;
                dc = c;
                dof = o;
            }
        }
        // the first level keeps the shortest: root sub-ranges index into it
        if (kFreshBaseRatio && (IS_SIG || lv >= 2) && D.lvl(bc) < dlv &&
            (uint64_t)dbest <= (uint64_t)kFreshBaseRatio * best) {
            best = dbest;
            bc = dc;
            bo = dof;
        }
        for (uint32_t c = 0; c < D.n_cons; c++) {
            if (c == bc) continue;
            const uint32_t nd = C.s.bound[D.lvl(c) * 64 + lane];
            const uint32_t* off = off_of(g, D.dir(c));
            const uint32_t o = off[nd];
            uint32_t l = off[nd + 1] - o;
            const uint32_t* ptr = probe_ref(g, D.dir(c), nd, o, l);
            put(k++, ptr, l);
        }
        base = adj_of(g, D.dir(bc)) + bo;
        len = best;
        if (IS_SIG && len >= g.row_min) {
            const uint2 r = g.row_of[C.s.bound[D.lvl(bc) * 64 + lane]];
            brow = D.dir(bc) ? r.y : r.x;
        }
        if (!IS_SIG && lv == 1) {
            // a root carries its first-level range [lo, hi)
            Lvl F0 = lvl_arrays(C.scr, a.cap, 0);
            uint32_t lo = F0.parent[p], hi = F0.aux[p];
            hi = hi < len ? hi : len;
            lo = lo < hi ? lo : hi;
            base += lo;
            len = hi - lo;
        }
    }
    for (; k < D.n_cons; k++) put(k, safe_ptr(g), kSkip);
    // symmetry breaking: the base is sorted, so its candidates are a range
    if (D.gt) {
        const uint32_t* whole = base;
        sym_trim(C.s, D.gt, D.lt, lv, lane, base, len);
        bskip = (uint32_t)(base - whole);
    }
    const uint64_t bv = reinterpret_cast<uint64_t>(base);
    C.s.base_lo[lane] = (uint32_t)bv;
    C.s.base_hi[lane] = (uint32_t)(bv >> 32);
    C.s.base_len[lane] = len;
    return len;
}

// Probe slots a level uses: all but the base constraint, or (when reusing a
// complete candidate set) the extra constraints; lanes with fewer pad with
// kSkip.
__device__ __forceinline__ uint32_t n_slots(const LK& D) {
    return D.reuse == kNoReuse ? (D.n_cons ? D.n_cons - 1 : 0) : D.n_cons;
}

// Base element `local` of window parent j.
__device__ __forceinline__ uint32_t base_elem(const Ctx& C, uint32_t j, uint32_t local) {
    return join_ptr(C.s.base_lo[j], C.s.base_hi[j])[local];
}

// Window parents of the elements t0 + lane (tile a) and t0 + 64 + lane (tile
// b) of a flattened pass.  Lane j (a window parent) owns the elements
// [start, start + len); parents that own elements mark their first one, and a
// max-scan carries each mark forward.  `carry` is the parent of the last
// element of the previous step (0 before the first).
__device__ __forceinline__ void tile_parents(const Lds& s, uint32_t lane, uint32_t t0, uint32_t start, bool owns,
                                             uint32_t& carry, uint32_t& ja, uint32_t& jb) {
    s.mark[lane] = 0;
    s.mark[64 + lane] = 0;
    wave_sync();
    if (owns && start >= t0 && start - t0 < 128u) s.mark[start - t0] = lane + 1;
    wave_sync();
    const uint32_t ma = scan_max(s.mark[lane]);
    const uint32_t mb = scan_max(s.mark[64 + lane]);
    ja = ma ? ma - 1 : carry;
    const uint32_t last_a = uni(__shfl(ja, 63, 64));
    jb = mb ? mb - 1 : last_a;
    carry = uni(__shfl(jb, 63, 64));
}

// Two sorted-list searches per lane (one per element), both loads of a step
// issued together.  A lane without a search passes n = 0 and a readable
// pointer (its value is ignored).
__device__ __forceinline__ void search2(gptr A, uint32_t na, uint32_t xa, bool& fa, gptr B, uint32_t nb,
                                        uint32_t xb, bool& fb) {
    uint32_t ba = 0, bb = 0, ra = na, rb = nb;
    while (__ballot(ra > 1 || rb > 1)) {
        const uint32_t ha = ra >> 1, hb = rb >> 1;
        const uint32_t va = A[ba + ha], vb = B[bb + hb];
        ba = (va <= xa) ? ba + ha : ba;
        bb = (vb <= xb) ? bb + hb : bb;
        ra -= ha;
        rb -= hb;
    }
    const uint32_t ea = A[ba], eb = B[bb];
    fa = na > 0 && ea == xa;
    fb = nb > 0 && eb == xb;
}

// Membership of x in probe (ptr, len) for one lane: a dense-row bit or a
// sorted-list search (no test when len is kSkip: returns true).
__device__ __forceinline__ bool probe_one(gptr ptr, uint32_t len, uint32_t x) {
    if (len == kSkip) return true;
    if (len == kRowLen) return (ptr[x >> 5] >> (x & 31u)) & 1u;
    return contains(ptr, len, x);
}

// A bit map in LDS of one list that the partial matches of a window share (a
// constraint on a node bound at an earlier level).  Ids below lim have a bit of
// their own; the others share the map's second half by their low bits and are
// verified against the list (probe slot vk).  lim = 0xFFFFFFFF: every id of the
// graph has its own bit.  Lanes (window parents) in `lanes` use it.
struct Filter {
    uint64_t lanes;
    const uint32_t* bits;
    uint32_t lim, vk;
    __device__ __forceinline__ bool has(uint32_t x) const {
        const uint32_t i = x < lim ? x : (lim | (x & (lim - 1u)));
        return __builtin_amdgcn_ubfe(bits[i >> 5], i, 1u) != 0;
    }
};

// Candidate tests of two elements (xa of window parent ja, xb of jb) against
// level D: injectivity (levels in `inj`), degree thresholds, then each probe
// slot as a dense-row bit test or a sorted-list search.  oka / okb: in =
// element valid, out = element passes.
template <bool FILT>
__device__ __forceinline__ void check_pair(const Ctx& C, const LK& D, const Filter& flt, uint32_t inj, uint32_t lv,
                                           uint32_t ns, uint32_t ja, uint32_t xa, bool& oka, uint32_t jb,
                                           uint32_t xb, bool& okb) {
    const DevGraph& g = C.a->g;
    bool fa = false, fb = false;  // the filter decides the probe in slot vk
    if (FILT && flt.lanes) {
        fa = (flt.lanes >> ja) & 1u;
        fb = (flt.lanes >> jb) & 1u;
        const bool ha = flt.has(xa), hb = flt.has(xb);
        oka = oka && (ha || !fa);
        okb = okb && (hb || !fb);
        fa = fa && xa < flt.lim;
        fb = fb && xb < flt.lim;
    }
    for (uint32_t l = 0; l < lv; l++)
        if ((inj >> l) & 1u) {
            oka = oka && (xa != C.s.bound[l * 64 + ja]);
            okb = okb && (xb != C.s.bound[l * 64 + jb]);
        }
    if (D.deg_check) {
        // one byte per node: in degree order the frequent candidates (hubs)
        // share a few cache lines
        const uint32_t da = g.degc[oka ? xa : 0u], db = g.degc[okb ? xb : 0u];
        oka = oka && (da & 15u) >= D.dmin_out && (da >> 4) >= D.dmin_in;
        okb = okb && (db & 15u) >= D.dmin_out && (db >> 4) >= D.dmin_in;
    }
    const gptr safe = (gptr)safe_ptr(g);
    for (uint32_t k = 0; k < ns; k++) {
        uint32_t lA = C.s.slot_len[k * 64 + ja], lB = C.s.slot_len[k * 64 + jb];
        if (FILT && k == flt.vk) {
            lA = fa ? kSkip : lA;
            lB = fb ? kSkip : lB;
        }
        const gptr pA = join_ptr(C.s.slot_lo[k * 64 + ja], C.s.slot_hi[k * 64 + ja]);
        const gptr pB = join_ptr(C.s.slot_lo[k * 64 + jb], C.s.slot_hi[k * 64 + jb]);
        const bool rA = oka && lA == kRowLen, rB = okb && lB == kRowLen;
        if (__ballot(rA || rB)) {
            const uint32_t wa = (rA ? pA : safe)[rA ? (xa >> 5) : 0u];
            const uint32_t wb = (rB ? pB : safe)[rB ? (xb >> 5) : 0u];
            if (rA) oka = (wa >> (xa & 31u)) & 1u;
            if (rB) okb = (wb >> (xb & 31u)) & 1u;
        }
        // an empty list holds nothing
        if (lA == 0) oka = false;
        if (lB == 0) okb = false;
        const bool sa = oka && lA < kRowLen, sb = okb && lB < kRowLen;
        if (__ballot(sa || sb)) {
            bool fa, fb;
            search2(sa ? pA : safe, sa ? lA : 0u, xa, fa, sb ? pB : safe, sb ? lB : 0u, xb, fb);
            if (sa) oka = fa;
            if (sb) okb = fb;
        }
    }
}

// One step of a wide scan: U tiles of the base list from element i0 on, tested
// against the parent's probes.  Everything but the element is the same for all
// lanes: base, rows and lists sit in scalar registers.
template <int U, class F>
__device__ __forceinline__ void wide_step(const Ctx& C, const LK& D, uint32_t inj, uint32_t lv, uint32_t j,
                                          gptr base, uint32_t len, uint32_t i0, uint32_t nrow, gptr r0, gptr r1,
                                          uint32_t rest, F&& emit) {
    const DevGraph& g = C.a->g;
    uint32_t x[U];
    bool ok[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
        const uint32_t i = i0 + (uint32_t)u * 64u + C.lane;
        ok[u] = i < len;
        x[u] = base[ok[u] ? i : i0];
    }
    for (uint32_t l = 0; l < lv; l++)
        if ((inj >> l) & 1u) {
            const uint32_t b = uni(C.s.bound[l * 64 + j]);
#pragma unroll
            for (int u = 0; u < U; u++) ok[u] = ok[u] && x[u] != b;
        }
    if (D.deg_check) {
        uint32_t d[U];
#pragma unroll
        for (int u = 0; u < U; u++) d[u] = g.degc[ok[u] ? x[u] : 0u];
#pragma unroll
        for (int u = 0; u < U; u++) ok[u] = ok[u] && (d[u] & 15u) >= D.dmin_out && (d[u] >> 4) >= D.dmin_in;
    }
    // a lane that is out already reads the row's first word
    auto row_test = [&](gptr r) {
        uint32_t w[U];
#pragma unroll
        for (int u = 0; u < U; u++) w[u] = r[ok[u] ? x[u] >> 5 : 0u];
#pragma unroll
        for (int u = 0; u < U; u++) ok[u] = ok[u] && __builtin_amdgcn_ubfe(w[u], x[u], 1u) != 0;
    };
    if (nrow > 0) row_test(r0);
    if (nrow > 1) row_test(r1);
    for (uint32_t m = rest; m; m &= m - 1) {
        const uint32_t k = (uint32_t)__builtin_ctz(m);
        const uint32_t n = uni(C.s.slot_len[k * 64 + j]);
        const gptr p = join_ptr(uni(C.s.slot_lo[k * 64 + j]), uni(C.s.slot_hi[k * 64 + j]));
        if (n == kRowLen) {
            row_test(p);
            continue;
        }
        // a sorted list of the same length for every lane: the searches of all
        // tiles halve together
        uint32_t b[U];
#pragma unroll
        for (int u = 0; u < U; u++) b[u] = 0;
        for (uint32_t r = n; r > 1;) {
            const uint32_t h = r >> 1;
            uint32_t v[U];
#pragma unroll
            for (int u = 0; u < U; u++) v[u] = p[b[u] + h];
#pragma unroll
            for (int u = 0; u < U; u++) b[u] = v[u] <= x[u] ? b[u] + h : b[u];
            r -= h;
        }
        uint32_t v[U];
#pragma unroll
        for (int u = 0; u < U; u++) v[u] = p[b[u]];
#pragma unroll
        for (int u = 0; u < U; u++) ok[u] = ok[u] && v[u] == x[u];
    }
#pragma unroll
    for (int u = 0; u < U; u++) emit(x[u], ok[u]);
}

// Candidate tests of one window parent j whose base list is long, by the whole
// wave: the elements base[0, len) in order, 64 at a time; emit(x, ok) is called
// for each tile.  A flattened tile pays for its generality (which parent owns
// the element, its base and probe slots from LDS: ~70 VALU instructions per 64
// elements); here these are uniform and a tile against one row takes ~10.
// Measured, flattened only and with this: TT4 + pendant on R-MAT 18 313 and
// 134 ms, C5 + chord on R-MAT 20 (1/256 of the roots) 229 and 97 ms, 96 plans on
// R-MAT 22 614 and 385 ms, four unreduced motifs on R-MAT 16 162 and 157 ms (bound
// by the row gathers' misses in L2 either way).
template <bool FOUR, class F>
__device__ __forceinline__ void wide_scan(const Ctx& C, const LK& D, uint32_t inj, uint32_t lv, uint32_t ns,
                                          uint32_t j, gptr base, uint32_t len, F&& emit) {
    gptr r0 = base, r1 = base;
    uint32_t nrow = 0, rest = 0;
    for (uint32_t k = 0; k < ns; k++) {
        const uint32_t l = uni(C.s.slot_len[k * 64 + j]);
        if (l == kSkip) continue;
        if (l == 0) return;  // an empty list holds nothing
        if (l == kRowLen && nrow < 2) {
            const gptr p = join_ptr(uni(C.s.slot_lo[k * 64 + j]), uni(C.s.slot_hi[k * 64 + j]));
            if (nrow == 0) r0 = p;
            else r1 = p;
            nrow++;
        } else {
            rest |= 1u << k;
        }
    }
    uint32_t i0 = 0;
    if (FOUR)
        for (; i0 + 128 < len; i0 += 256) wide_step<4>(C, D, inj, lv, j, base, len, i0, nrow, r0, r1, rest, emit);
    for (; i0 < len; i0 += 128) wide_step<2>(C, D, inj, lv, j, base, len, i0, nrow, r0, r1, rest, emit);
}

// Whether bound node y of this lane's partial match lies in the lane's base
// list and passes all its probes: then a flattened pass without injectivity
// counted it once.  (at: the lane whose base list and probes they are.)
__device__ __forceinline__ bool bound_in_set(const Ctx& C, uint32_t ns, uint32_t y, uint32_t at) {
    const uint32_t lane = at;
    const uint32_t len = C.s.base_len[lane];
    if (!contains(join_ptr(C.s.base_lo[lane], C.s.base_hi[lane]), len, y)) return false;
    for (uint32_t k = 0; k < ns; k++)
        if (!probe_one(join_ptr(C.s.slot_lo[k * 64 + lane], C.s.slot_hi[k * 64 + lane]),
                       C.s.slot_len[k * 64 + lane], y))
            return false;
    return true;
}

// Elements of window parent j's long base list that pass all its probes (no
// injectivity: leaf passes settle that per partial match).
__device__ __forceinline__ uint32_t wide_count(const Ctx& C, const LK& D, uint32_t lv, uint32_t ns, uint32_t j) {
    uint32_t cnt = 0;
    wide_scan<true>(C, D, 0u, lv, ns, j, join_ptr(uni(C.s.base_lo[j]), uni(C.s.base_hi[j])), uni(C.s.base_len[j]),
              [&](uint32_t, bool ok) { cnt += (uint32_t)__popcll(__ballot(ok)); });
    return cnt;
}

// A window parent of a leaf pass as its lane sees it: base list, and up to two
// dense rows to test (when its probes are nothing else).
struct Par {
    uint32_t lo, hi, len;        // base list
    uint32_t n_rows;             // rows to test
    uint32_t r0lo, r0hi, r1lo, r1hi;
    bool rows_only;              // no sorted-list probe, at most two rows
};
__device__ __forceinline__ Par parent_view(const Ctx& C, uint32_t ns, uint32_t len) {
    const uint32_t lane = C.lane;
    Par p;
    p.lo = C.s.base_lo[lane];
    p.hi = C.s.base_hi[lane];
    p.len = len;
    p.n_rows = 0;
    p.r0lo = p.r0hi = p.r1lo = p.r1hi = 0;
    p.rows_only = true;
    for (uint32_t k = 0; k < ns; k++) {
        const uint32_t l = C.s.slot_len[k * 64 + lane];
        if (l == kSkip) continue;
        if (l == 0) p.len = 0;  // an empty list holds nothing
        if (l != kRowLen || p.n_rows == 2) {
            p.rows_only = false;
            continue;
        }
        const uint32_t lo = C.s.slot_lo[k * 64 + lane], hi = C.s.slot_hi[k * 64 + lane];
        if (p.n_rows == 0) {
            p.r0lo = p.r1lo = lo;
            p.r0hi = p.r1hi = hi;
        } else {
            p.r1lo = lo;
            p.r1hi = hi;
        }
        p.n_rows++;
    }
    return p;
}

__device__ __forceinline__ uint32_t from_lane(uint32_t v, uint32_t j) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)j);
}

// Count, for every lane (window parent) in `todo`, the base elements that are
// in its one or two rows; add(j, n) is called with the counts.  The parents'
// lists are cut into chunks of two tiles, and two chunks are in flight at a
// time, of one parent or of two, so short lists too keep four base loads and
// four row loads outstanding.  Everything about a chunk is scalar, read from
// its lane's registers: ~6 vector instructions a tile.  Measured against one
// parent at a time (wide_scan): TT4 + pendant on R-MAT 18 134 and 127 ms (best
// runs 129 and 103), four motifs on R-MAT 16 21.5 and 20.1, unreduced 158 and 154;
// loading ahead: 96 plans on R-MAT 22 348 and 328, C5 + chord on R-MAT 20 67 and
// 62, TT4 + pendant on R-MAT 18 99 and 90.
// AHEAD: the next pair's base loads are issued before the current pair's tests
// (in the kernels that have the registers for it).
template <bool AHEAD, class F>
__device__ __forceinline__ void chunk_scan(const Ctx& C, const Par& P, uint64_t todo, F&& add) {
    struct Chunk {
        gptr base, r0, r1;
        uint32_t j, n, rows;
    };
    const uint32_t lane = C.lane;
    uint32_t i0 = 0, left = 0;
    Chunk cur{};
    auto next = [&](Chunk& c) {
        if (i0 >= left) {
            if (!todo) {
                c = cur;
                c.n = 0;
                return;
            }
            cur.j = (uint32_t)__builtin_ctzll(todo);
            todo &= todo - 1;
            left = from_lane(P.len, cur.j);
            cur.base = join_ptr(from_lane(P.lo, cur.j), from_lane(P.hi, cur.j));
            cur.r0 = join_ptr(from_lane(P.r0lo, cur.j), from_lane(P.r0hi, cur.j));
            cur.rows = from_lane(P.n_rows, cur.j);
            cur.r1 = cur.r0;
            if (cur.rows > 1) cur.r1 = join_ptr(from_lane(P.r1lo, cur.j), from_lane(P.r1hi, cur.j));
            i0 = 0;
        }
        c = cur;
        c.base = cur.base + i0;
        c.n = left - i0 < 128u ? left - i0 : 128u;
        i0 += 128;
    };
    Chunk c[2];
    uint32_t x[4];
    auto load = [&](Chunk* k, uint32_t* y) {
        next(k[0]);
        next(k[1]);
#pragma unroll
        for (int u = 0; u < 4; u++) {
            // lanes past the end read the last element again
            const uint32_t n = k[u >> 1].n, i = (u & 1) * 64u + lane, last = n ? n - 1 : 0u;
            y[u] = k[u >> 1].base[i < last ? i : last];
        }
    };
    if (AHEAD) load(c, x);
    while (AHEAD ? c[0].n != 0 : (todo || i0 < left)) {
        Chunk nc[2];
        uint32_t y[4], w[4];
        uint64_t in[4];
        if (AHEAD) load(nc, y);
        else load(c, x);
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const uint32_t n = c[u >> 1].n, off = (u & 1) * 64u;
            in[u] = n >= off + 64u ? ~0ull : (n > off ? (1ull << (n - off)) - 1ull : 0ull);
        }
#pragma unroll
        for (int u = 0; u < 4; u++) w[u] = c[u >> 1].r0[x[u] >> 5];
#pragma unroll
        for (int u = 0; u < 4; u++) in[u] &= __ballot(__builtin_amdgcn_ubfe(w[u], x[u], 1u) != 0);
        if (c[0].rows > 1 || c[1].rows > 1) {
            // (a chunk with one row tests it again)
#pragma unroll
            for (int u = 0; u < 4; u++) w[u] = c[u >> 1].r1[(in[u] >> lane) & 1u ? x[u] >> 5 : 0u];
#pragma unroll
            for (int u = 0; u < 4; u++) in[u] &= __ballot(__builtin_amdgcn_ubfe(w[u], x[u], 1u) != 0);
        }
        add(c[0].j, (uint32_t)(__popcll(in[0]) + __popcll(in[1])));
        add(c[1].j, (uint32_t)(__popcll(in[2]) + __popcll(in[3])));
        if (AHEAD) {
            c[0] = nc[0];
            c[1] = nc[1];
#pragma unroll
            for (int u = 0; u < 4; u++) x[u] = y[u];
        }
    }
}

// The dense part of a parent's base list: the ids [xlo, xhi) in the words
// [w0, w1) (multiples of 4) of its row.
struct Dense {
    uint32_t lo, hi;  // the row
    uint32_t w0, w1, xlo, xhi;
};

// Splits parent P's base list (dense row brow, bskip elements cut off its
// front) into a dense part, taken from P, and the rest, which stays.  A row's
// head is dense where its list's ids are (row_pre: words and elements of the
// head); intersecting words there reads both rows in order, 16 bytes a lane,
// where the elements would each touch a sector of the probed row.
__device__ __forceinline__ Dense take_dense(const Ctx& C, const LK& D, uint32_t nb, uint32_t brow, uint32_t bskip,
                                            Par& P) {
    const DevGraph& g = C.a->g;
    Dense d{};
    if (brow == kSkip) return d;
    const uint2 pre = g.row_pre[brow];  // words, elements
    const uint64_t row = reinterpret_cast<uint64_t>(g.rows + (uint64_t)brow * g.row_words);
    d.lo = (uint32_t)row;
    d.hi = (uint32_t)(row >> 32);
    d.w1 = pre.x;
    d.xhi = pre.x * 32u;
    uint32_t take = pre.y > bskip ? pre.y - bskip : 0u;
    take = take < P.len ? take : P.len;
    if (D.gt) {
        uint32_t lo = 0xFFFFFFFFu, hi = 0;
        for (uint32_t l = 0; l < nb; l++)
            if ((D.gt >> l) & 1u) {
                const uint32_t b = C.s.bound[l * 64 + C.lane];
                lo = b < lo ? b : lo;
                hi = b > hi ? b : hi;
            }
        if (D.lt) {
            d.xhi = lo < d.xhi ? lo : d.xhi;
            d.w1 = (d.xhi + 127u) / 128u * 4u;
        } else {
            d.xlo = hi + 1u;
            d.w0 = d.xlo / 128u * 4u;
        }
    }
    if (d.w0 >= d.w1 || take * kDenseWords < d.w1 - d.w0) {
        d.w0 = d.w1 = 0;
        return d;
    }
    const uint64_t rest = (((uint64_t)P.hi << 32) | P.lo) + 4ull * take;
    P.lo = (uint32_t)rest;
    P.hi = (uint32_t)(rest >> 32);
    P.len -= take;
    return d;
}

// Count, for every lane in `todo`, the bits common to its dense part and its
// one or two rows.  Chunks of 256 words, two in flight; add(j, v) is called
// with each lane's share v of a chunk's count.
template <class F>
__device__ __forceinline__ void word_scan(const Ctx& C, const Par& P, const Dense& Dn, bool trim, uint64_t todo,
                                          F&& add) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));
    typedef const __attribute__((address_space(1))) u32x4* gptr4;
    struct Chunk {
        gptr base, r0, r1;
        uint32_t j, w, end, xlo, xhi, rows;
    };
    const uint32_t lane = C.lane;
    Chunk cur{};
    auto next = [&](Chunk& c) {
        if (cur.w >= cur.end) {
            if (!todo) {
                c = cur;
                return;
            }
            cur.j = (uint32_t)__builtin_ctzll(todo);
            todo &= todo - 1;
            cur.base = join_ptr(from_lane(Dn.lo, cur.j), from_lane(Dn.hi, cur.j));
            cur.w = from_lane(Dn.w0, cur.j);
            cur.end = from_lane(Dn.w1, cur.j);
            cur.r0 = join_ptr(from_lane(P.r0lo, cur.j), from_lane(P.r0hi, cur.j));
            cur.rows = from_lane(P.n_rows, cur.j);
            cur.r1 = cur.r0;
            if (cur.rows > 1) cur.r1 = join_ptr(from_lane(P.r1lo, cur.j), from_lane(P.r1hi, cur.j));
            if (trim) {
                cur.xlo = from_lane(Dn.xlo, cur.j);
                cur.xhi = from_lane(Dn.xhi, cur.j);
            }
        }
        c = cur;
        cur.w += 256;
    };
    while (todo || cur.w < cur.end) {
        Chunk c[2];
        next(c[0]);
        next(c[1]);
        u32x4 b[2], r[2];
        bool in[2];
        uint32_t w[2];
#pragma unroll
        for (int u = 0; u < 2; u++) {
            w[u] = c[u].w + 4 * lane;
            in[u] = w[u] < c[u].end;
            const uint32_t at = in[u] ? w[u] : 0u;
            b[u] = *(gptr4)(c[u].base + at);
            r[u] = *(gptr4)(c[u].r0 + at);
        }
        uint32_t n[2];
#pragma unroll
        for (int u = 0; u < 2; u++) b[u] &= r[u];
        if (c[0].rows > 1 || c[1].rows > 1) {
            // (a chunk with one row takes it again)
#pragma unroll
            for (int u = 0; u < 2; u++) b[u] &= *(gptr4)(c[u].r1 + (in[u] ? w[u] : 0u));
        }
        if (trim) {
            // keep the ids in [xlo, xhi)
#pragma unroll
            for (int u = 0; u < 2; u++)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const uint32_t x0 = (w[u] + (uint32_t)e) * 32u;
                    const uint32_t below = c[u].xhi > x0 ? c[u].xhi - x0 : 0u;     // ids of the word under xhi
                    const uint32_t under = c[u].xlo > x0 ? c[u].xlo - x0 : 0u;     // ids of the word under xlo
                    const uint32_t hm = below >= 32u ? ~0u : (1u << below) - 1u;
                    const uint32_t lm = under >= 32u ? ~0u : (1u << under) - 1u;
                    b[u][e] &= hm & ~lm;
                }
        }
#pragma unroll
        for (int u = 0; u < 2; u++) {
            n[u] = (uint32_t)(__popc(b[u].x) + __popc(b[u].y) + __popc(b[u].z) + __popc(b[u].w));
            n[u] = in[u] ? n[u] : 0u;
        }
        add(c[0].j, n[0]);
        add(c[1].j, n[1]);
    }
}

// Levels whose bound node is the same for all partial matches of the window
// (bit l: level l < nb).
__device__ __forceinline__ uint32_t same_levels(const Ctx& C, uint32_t nb, bool pv) {
    uint32_t m = 0;
    for (uint32_t l = 0; l < nb; l++) {
        const uint32_t v = C.s.bound[l * 64 + C.lane];
        if (!__ballot(pv && v != uni(v))) m |= 1u << l;  // (lane 0 always holds a partial match)
    }
    return m;
}

// Constraints of D on the levels in `same`.
__device__ __forceinline__ uint32_t shared_cons(const LK& D, uint32_t same) {
    uint32_t m = 0;
    for (uint32_t c = 0; c < D.n_cons; c++) m |= ((same >> D.lvl(c)) & 1u) << c;
    return m;
}

// After phase_a of a leaf pass: parents whose base is a short list of a
// constraint outside `shared` (flen elements) test it against a filter of the
// shortest shared list; such a lane gets the filtered list's probe in slot
// flt.vk.  The filter stays for later windows with the same list.
//
// A short list is tested in flattened tiles, where a search of the shared list
// costs a chain of ~log2(length) loads of 64 addresses; the filter is one LDS
// word.  Measured without and with it: three patterns on 30,011 nodes of degree
// ~20 7.9 and 6.5 ms.  Long lists are streamed against dense rows or searched as
// before: filtering them too, up to 2 / 4 / 8 times longer lists for the sake of
// it, took 357 / 411 / 413 ms on 96 plans of R-MAT 22 instead of 347.
__device__ __forceinline__ void use_filter(Ctx& C, const LK& D, uint32_t nb, uint32_t shared, uint32_t flen,
                                           uint32_t& len, Filter& flt) {
    const KArgs& a = *C.a;
    const DevGraph& g = a.g;
    const uint32_t lane = C.lane;
    const bool el = len > 0 && flen < kWideMin && flen <= len;
    const uint64_t em = __ballot(el);
    if (!em) return;
    uint32_t best = kSkip, bc = 0, bo = 0;
    for (uint32_t c = 0; c < D.n_cons; c++) {
        if (!((shared >> c) & 1u)) continue;
        const uint32_t nd = uni(C.s.bound[D.lvl(c) * 64]);
        const uint32_t* off = off_of(g, D.dir(c));
        const uint32_t o = uni(off[nd]), l = uni(off[nd + 1]) - o;
        if (l < best) {
            best = l;
            bc = c;
            bo = o;
        }
    }
    if (best == 0) return;
    const uint32_t total = uni(__shfl(scan_incl(el ? flen : 0u, lane), 63, 64));
    const uint64_t tag = reinterpret_cast<uint64_t>(adj_of(g, D.dir(bc)) + bo);
    const uint64_t old = ((uint64_t)uni(C.s.st[28]) << 32) | uni(C.s.st[27]);
    if (old != tag && total < 2u * best + 64u) return;  // not worth filling it
    const uint32_t bits = 32u * a.filt_words;
    flt.lanes = em;
    flt.bits = C.s.filt;
    flt.lim = g.n <= bits ? 0xFFFFFFFFu : bits / 2;
    flt.vk = D.n_cons - 2;
    if (old != tag) {
        // clear the old list's bits one by one if that is less than the map
        const uint32_t oldn = uni(C.s.st[29]);
        if (old && oldn <= 2 * a.filt_words) {
            const gptr L = (gptr)old;
            for (uint32_t i = lane; i < oldn; i += 64) {
                const uint32_t x = L[i];
                C.s.filt[(x < flt.lim ? x : (flt.lim | (x & (flt.lim - 1u)))) >> 5] = 0;
            }
        } else {
            uint4* z = reinterpret_cast<uint4*>(C.s.filt);
            for (uint32_t i = lane; i < a.filt_words / 4; i += 64) z[i] = make_uint4(0, 0, 0, 0);
        }
        if (lane == 0) {
            C.s.st[27] = (uint32_t)tag;
            C.s.st[28] = (uint32_t)(tag >> 32);
            C.s.st[29] = best;
        }
        wave_sync();
        const gptr L = (gptr)tag;
        for (uint32_t i = lane; i < best; i += 64) {
            const uint32_t x = L[i];
            const uint32_t h = x < flt.lim ? x : (flt.lim | (x & (flt.lim - 1u)));
            atomicOr(&C.s.filt[h >> 5], 1u << (h & 31u));
        }
    }
    if (el) {
        uint32_t fb = kSkip, fc = 0, fo = 0;
        for (uint32_t c = 0; c < D.n_cons; c++) {
            if ((shared >> c) & 1u) continue;
            const uint32_t nd = C.s.bound[D.lvl(c) * 64 + lane];
            const uint32_t* off = off_of(g, D.dir(c));
            const uint32_t o = off[nd], l = off[nd + 1] - o;
            if (l < fb) {
                fb = l;
                fc = c;
                fo = o;
            }
        }
        uint32_t k = 0;
        for (uint32_t c = 0; c < D.n_cons; c++) {
            if (c == fc) continue;
            const uint32_t nd = C.s.bound[D.lvl(c) * 64 + lane];
            const uint32_t* off = off_of(g, D.dir(c));
            const uint32_t o = off[nd];
            uint32_t l = off[nd + 1] - o;
            const uint64_t v = reinterpret_cast<uint64_t>(probe_ref(g, D.dir(c), nd, o, l));
            const uint32_t s = c == bc ? flt.vk : k++;
            C.s.slot_len[s * 64 + lane] = l;
            C.s.slot_lo[s * 64 + lane] = (uint32_t)v;
            C.s.slot_hi[s * 64 + lane] = (uint32_t)(v >> 32);
        }
        for (uint32_t s = D.n_cons - 1; s < n_slots(D); s++) C.s.slot_len[s * 64 + lane] = kSkip;
        const uint32_t* base = adj_of(g, D.dir(fc)) + fo;
        len = fb;
        if (D.gt) sym_trim(C.s, D.gt, D.lt, nb, lane, base, len);
        const uint64_t bv = reinterpret_cast<uint64_t>(base);
        C.s.base_lo[lane] = (uint32_t)bv;
        C.s.base_hi[lane] = (uint32_t)(bv >> 32);
        C.s.base_len[lane] = len;
    }
    wave_sync();
}

// Expand one window of level lv from the parents in level lv-1.  Returns the
// number of children written to level lv's buffer.
__device__ __forceinline__ uint32_t expand(Ctx& C, uint32_t lv) {
    const KArgs& a = *C.a;
    const LK D = load_lk(C.P->lvl[lv], a);
    const uint32_t lane = C.lane;
    uint32_t* st = C.s.st;
    const uint32_t nparents = uni(st[16 + lv - 1]);
    const uint32_t cur = uni(st[lv]);
    const uint32_t pofs = uni(st[8 + lv]);
    const uint32_t p = cur + lane;
    const bool pv = p < nparents;
    uint32_t flen, brow, bskip;
    uint32_t len = phase_a<false>(C, D, lv, p, pv, true, ~0u, flen, brow, bskip);
    bool cut = false;
    if (uni(st[24]) == lv && uni(st[26]) != kSkip && pv) {
        // a donated id range: its part of the sorted base list
        const uint64_t at = ((uint64_t)C.s.base_hi[lane] << 32) | C.s.base_lo[lane];
        const uint32_t* base = reinterpret_cast<const uint32_t*>(at);
        const uint32_t lo = count_lt(base, len, uni(st[25])), hi = count_lt(base, len, uni(st[26]));
        const uint64_t bv = reinterpret_cast<uint64_t>(base + lo);
        cut = hi - lo < len;
        len = hi - lo;
        C.s.base_lo[lane] = (uint32_t)bv;
        C.s.base_hi[lane] = (uint32_t)(bv >> 32);
        C.s.base_len[lane] = len;
    }
    if (pv && lane == 0) len -= pofs;
    uint32_t incl = scan_incl(len, lane);
    C.s.incl[lane] = incl;
    const bool seg = (C.P->seg_src >> lv) & 1u;
    if (seg) C.s.segcnt[lane] = 0;
    const uint32_t cap = a.cap;
    uint32_t np = uni((uint32_t)__popcll(__ballot(pv && incl <= cap)));
    bool partial = false;
    if (np == 0) {
        // the first parent alone exceeds the buffer: take a slice of it
        partial = true;
        np = 1;
        if (lane == 0) incl = len = cap;
        C.s.incl[0] = cap;
    }
    // lane j < np owns the elements [incl - len, incl)
    const bool owns = lane < np && len > 0;
    const uint32_t start = incl - len;
    wave_sync();
    Lvl Fo = lvl_arrays(C.scr, cap, lv);
    uint32_t nout = 0;
    const uint32_t ns = n_slots(D);
    // parents with a long base are scanned one by one, the runs between them
    // flattened; children are written in parent order either way
    const uint64_t wide = __ballot(lane < np && len >= kWideMin);
    for (uint32_t j0 = 0; j0 < np;) {
        const uint64_t ahead = wide >> j0;
        if (ahead & 1u) {
            const uint32_t before = nout;
            const uint32_t off = j0 == 0 ? pofs : 0u;
            const gptr base = join_ptr(uni(C.s.base_lo[j0]), uni(C.s.base_hi[j0])) + off;
            const uint32_t n = uni(__shfl(len, (int)j0, 64));
            wide_scan<false>(C, D, D.inj, lv, ns, j0, base, n, [&](uint32_t x, bool ok) {
                const uint64_t m = __ballot(ok);
                if (ok) {
                    const uint32_t pos = nout + rank_below(m);
                    Fo.node[pos] = x;
                    Fo.parent[pos] = cur + j0;
                }
                nout += (uint32_t)__popcll(m);
            });
            if (seg && lane == 0) C.s.segcnt[j0] = nout - before;
            j0++;
            continue;
        }
        // the run of short parents [j0, j1): elements [e0, e1)
        uint32_t j1 = ahead ? j0 + (uint32_t)__builtin_ctzll(ahead) : np;
        j1 = j1 < np ? j1 : np;
        const uint32_t e0 = uni(__shfl(start, (int)j0, 64)), e1 = uni(__shfl(incl, (int)j1 - 1, 64));
        uint32_t carry = j0;
        // two tiles per step: survivors of tile a are written before those of
        // tile b, so each parent's children stay contiguous and in order
        for (uint32_t t0 = e0; t0 < e1; t0 += 128) {
            const uint32_t ga = t0 + lane, gb = t0 + 64 + lane;
            uint32_t ja, jb;
            tile_parents(C.s, lane, t0, start, owns, carry, ja, jb);
            bool oka = ga < e1, okb = gb < e1;
            uint32_t xa = 0, xb = 0;
            const uint32_t la = ga - (ja ? C.s.incl[ja - 1] : 0u) + (ja == 0 ? pofs : 0u);
            const uint32_t lb = gb - (jb ? C.s.incl[jb - 1] : 0u) + (jb == 0 ? pofs : 0u);
            oka = oka && la < C.s.base_len[ja];
            okb = okb && lb < C.s.base_len[jb];
            if (oka) xa = base_elem(C, ja, la);
            if (okb) xb = base_elem(C, jb, lb);
            check_pair<false>(C, D, Filter{}, D.inj, lv, ns, ja, xa, oka, jb, xb, okb);
            const uint64_t ma = __ballot(oka);
            if (oka) {
                const uint32_t pos = nout + rank_below(ma);
                Fo.node[pos] = xa;
                Fo.parent[pos] = cur + ja;
                if (seg) atomicAdd(&C.s.segcnt[ja], 1u);
            }
            nout += (uint32_t)__popcll(ma);
            const uint64_t mb = __ballot(okb);
            if (okb) {
                const uint32_t pos = nout + rank_below(mb);
                Fo.node[pos] = xb;
                Fo.parent[pos] = cur + jb;
                if (seg) atomicAdd(&C.s.segcnt[jb], 1u);
            }
            nout += (uint32_t)__popcll(mb);
        }
        j0 = j1;
    }
    wave_sync();
    if (seg) {
        // children of each parent are contiguous in output order
        uint32_t cnt = (lane < np) ? C.s.segcnt[lane] : 0;
        uint32_t ex = scan_incl(cnt, lane) - cnt;
        if (lane < np) {
            Lvl Fi = lvl_arrays(C.scr, cap, lv - 1);
            bool complete = !(lane == 0 && (pofs > 0 || partial)) && !cut;
            if (lv == 1) {
                // a root split into first-level sub-ranges never has all its children here
                Lvl F0 = lvl_arrays(C.scr, cap, 0);
                complete = complete && F0.parent[cur + lane] == 0 && F0.aux[cur + lane] == kSkip;
            }
            Fi.segb[cur + lane] = ex;
            Fi.segc[cur + lane] = cnt | (complete ? kComplete : 0u);
        }
    }
    // advance the cursor of this level
    if (lane == 0) {
        if (partial) {
            st[8 + lv] = pofs + cap;
        } else {
            st[lv] = cur + np;
            st[8 + lv] = 0;
        }
        st[16 + lv] = nout;
    }
    wave_sync();
    return nout;
}

// |A intersect B| minus the listed bound nodes, for one partial match, by the
// whole wave: both sorted lists are walked in chunks of kMergeChunk elements
// (A in registers, B staged in LDS); each A element is looked up in the B
// chunk, and the chunk with the smaller maximum advances (both on a tie), so
// every matching pair is seen exactly once.  Reads are coalesced and no
// dependent global search is needed (merge path for balanced list sizes).
__device__ uint32_t merge_count(const Lds& s, gptr A, uint32_t na, gptr B, uint32_t nb, uint32_t inj, uint32_t nbound,
                                uint32_t j, uint32_t lane) {
    constexpr uint32_t U = kMergeChunk / 64;
    uint32_t ia = 0, ib = 0, cnt = 0;
    while (ia < na && ib < nb) {
        uint32_t av[U];
#pragma unroll
        for (uint32_t u = 0; u < U; u++) {
            uint32_t i = ia + u * 64 + lane;
            av[u] = i < na ? A[i] : 0xFFFFFFFFu;
            uint32_t k = ib + u * 64 + lane;
            s.mbuf[u * 64 + lane] = k < nb ? B[k] : 0xFFFFFFFFu;
        }
        const uint32_t alast = (ia + kMergeChunk < na ? ia + kMergeChunk : na) - 1;
        const uint32_t blast = (ib + kMergeChunk < nb ? ib + kMergeChunk : nb) - 1;
        const uint32_t amax = A[alast], bmax = B[blast];
        const uint32_t nbc = blast - ib + 1;
        wave_sync();
#pragma unroll
        for (uint32_t u = 0; u < U; u++) {
            uint32_t x = av[u];
            if (ia + u * 64 + lane < na) {
                uint32_t base = 0, n = nbc;
                while (n > 1) {
                    uint32_t h = n >> 1;
                    base = (s.mbuf[base + h] <= x) ? base + h : base;
                    n -= h;
                }
                bool ok = s.mbuf[base] == x;
                for (uint32_t t = 0; t < nbound; t++)
                    if ((inj >> t) & 1u) ok = ok && (x != s.bound[t * 64 + j]);
                cnt += ok ? 1u : 0u;
            }
        }
        if (amax <= bmax) ia += kMergeChunk;
        if (bmax <= amax) ib += kMergeChunk;
        wave_sync();
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) cnt += __shfl_xor(cnt, d, 64);
    return cnt;
}

// Survivors of this step's two tiles that belong to the parent owning the
// elements [start, start + len).
__device__ __forceinline__ uint32_t own_count(uint64_t ballot, uint32_t start, uint32_t len, uint32_t base) {
    const uint32_t lo = start > base ? start : base;
    const uint32_t end = start + len, top = base + 64;
    const uint32_t hi = end < top ? end : top;
    if (hi <= lo) return 0;
    const uint32_t a = lo - base, b = hi - base;
    const uint64_t m = (b == 64 ? ~0ull : ((1ull << b) - 1ull)) & ~((1ull << a) - 1ull);
    return (uint32_t)__popcll(ballot & m);
}

// Listing: the survivors of a tile pair are whole embeddings (bound levels
// 0..nb-1 of their parent plus the leaf).  They are collected in the wave's LDS
// (parent and leaf, kListRows of them), and one 64-bit atomic reserves the rows
// of a collection, written in pattern-vertex order while they fit the
// capacity.  With one atomic per tile pair the launch was as long as its atomics
// on that one word: 10.3 M rows of R-MAT 15's triangles 4.4 ms.
__device__ __forceinline__ void write_rows(const Ctx& C, uint32_t nb, uint32_t& held) {
    const KArgs& a = *C.a;
    if (held == 0) return;
    wave_sync();
    unsigned long long base = 0;
    if (C.lane == 0) base = atomicAdd(a.list_count, (unsigned long long)held);
    base = __shfl(base, 0, 64);
    const PlanDesc* P = C.P;
    const uint32_t k = P->k;
    for (uint32_t i = C.lane; i < held; i += 64) {
        const unsigned long long row = base + i;
        if (row >= a.list_cap) break;
        uint32_t* out = a.list + row * k;
        const uint32_t j = C.s.filt[kListRows + i];
        for (uint32_t l = 0; l < nb; l++) out[P->order[l]] = C.s.bound[l * 64 + j];
        out[P->order[nb]] = C.s.filt[i];
    }
    held = 0;
    wave_sync();
}
__device__ __forceinline__ void hold_rows(const Ctx& C, uint32_t nb, uint32_t& held, uint64_t m, uint32_t j, uint32_t x,
                                          bool ok) {
    if (ok) {
        const uint32_t at = held + rank_below(m);
        C.s.filt[at] = x;
        C.s.filt[kListRows + at] = j;
    }
    held += (uint32_t)__popcll(m);
    if (held + 64 > kListRows) write_rows(C, nb, held);
}

// Whether a task that has run for a while should look for waiting waves now.
__device__ __forceinline__ bool time_to_look(const Ctx& C, uint32_t& now) {
    now = (uint32_t)__builtin_readcyclecounter();
    return now - C.looked >= kDonateClocks;
}

// Work donation.  While some waves are idle (all queues drained), a wave that
// has spent at least kDonateClocks in one task hands off unstarted work as
// donated tasks, each a prefix phi(v_0..v_{l-1}) with a range of ids at level
// l, which another wave explores from level l.  It looks at the clock, not at
// windows done: the leaf pass of one window over hub lists can take
// milliseconds.  (Donating after 256 windows, and never within a leaf pass,
// left the ends of launches to a few waves.  Measured then and now: a tenth of
// the roots of R-MAT 16 48 and 39 ms, C5 + chord on R-MAT 20 73 and 68, TT4 +
// pendant on R-MAT 18 98-128 and 98-99.)  Slots are reserved with a CAS on the tail (never past
// the capacity) and published with a ready word.
// The queue is kept about as long as there are waiting waves: a backlog beyond
// that only adds tasks that are explored less efficiently than in a full window
// (with no such bound every running wave donated half of its work each time,
// 260,000 tasks a launch, and taking them took seconds).
//
// Tasks that may be donated now (0: none); `tail` becomes the queue's tail, and
// `head` its head or an earlier one.
__device__ __forceinline__ uint32_t donation_room(const Ctx& C, uint32_t& head, uint32_t& tail) {
    uint32_t v = 0;
    if (C.lane == 0) v = __atomic_load_n(&C.a->ctl[kCtlIdle], __ATOMIC_RELAXED);
    const uint32_t idle = uni(__shfl(v, 0, 64));
    head = tail = 0;
    if (idle == 0) return 0;
    if (C.lane < 2) v = __atomic_load_n(&C.a->ctl[C.lane ? kCtlDonTail : kCtlDonHead], __ATOMIC_RELAXED);
    tail = uni(__shfl(v, 1, 64));
    head = uni(__shfl(v, 0, 64));
    return idle > tail - head ? idle - (tail - head) : 0u;
}
// Reserve k slots behind the tail that donation_room saw.  One try: thousands of
// waves may look at the same time, and retrying against each other took longer
// than the work they had (a failed try comes back with the next look).
__device__ __forceinline__ uint32_t reserve_slots(Ctx& C, uint32_t k, uint32_t head, uint32_t tail) {
    const KArgs& a = *C.a;
    uint32_t base = kSkip;
    if (C.lane == 0 && don_fits(head, tail, k, a.don_cap) && atomicCAS(&a.ctl[kCtlDonTail], tail, tail + k) == tail)
        base = tail;
    base = uni(__shfl(base, 0, 64));
    if (base != kSkip && C.lane == 0) C.s.st[30] = base + k;
    return base;
}
// One donated task: level l below entry idx of level l-1, ids in [xlo, xhi).
__device__ __forceinline__ void donate(Ctx& C, uint32_t seq, uint32_t l, uint32_t idx, uint32_t xlo, uint32_t xhi) {
    const KArgs& a = *C.a;
    uint32_t* ent = a.don + (uint64_t)don_slot(seq, a.don_cap) * kDonWords;
    // Relaxed atomics go past the XCD's L2 by themselves; a release fence would
    // write that whole L2 back and the taker's acquire would empty its own (a
    // launch with 50,000 donated tasks spent most of a second on it).  The
    // entry's words have arrived once the stores are counted back.
    auto put = [&](uint32_t w, uint32_t v) { __atomic_store_n(&ent[w], v, __ATOMIC_RELAXED); };
    for (int j = (int)l - 1; j >= 0; --j) {
        Lvl F = lvl_arrays(C.scr, a.cap, (uint32_t)j);
        put(2 + (uint32_t)j, F.node[idx]);
        if (j > 0) idx = F.parent[idx];
    }
    put(kDonWords - 2, xlo);
    put(kDonWords - 1, xhi);
    put(0, C.pi | (l << 16));
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    put(1, don_published(seq, a.don_cap));
}

// At the shallowest level l >= 2 with at least two parents at level l-1 not yet
// expanded, the last half of them (at most 64) become donated tasks; the donor
// drops them from its window.
__device__ __forceinline__ void donate_parents(Ctx& C, uint32_t start, uint32_t lv) {
    uint32_t* st = C.s.st;
    uint32_t head, tail;
    const uint32_t room = donation_room(C, head, tail);
    if (room == 0) return;
    for (uint32_t l = (start > 2 ? start : 2); l <= lv; l++) {
        const uint32_t n = uni(st[16 + l - 1]);
        uint32_t first = uni(st[l]);
        if (l == lv && uni(st[8 + l]) > 0) first += 1;  // a parent in the middle of a slice stays
        if (first >= n || n - first < 2) continue;
        uint32_t k = (n - first) / 2;
        k = k < 64 ? k : 64;
        k = k < room ? k : room;
        const uint32_t base = reserve_slots(C, k, head, tail);
        if (base == kSkip) return;  // no room: keep the work
        if (C.lane < k) donate(C, base + C.lane, l, n - k + C.lane, 0, kSkip);
        if (C.lane == 0) st[16 + l - 1] = n - k;
        wave_sync();
        return;
    }
}

// Within the leaf pass over level lv's window: donate about the last half of
// the partial matches [from, n) that are not counted yet, as id ranges below
// their parents (level lv is expanded again there, for these ids only).
// each: clocks a partial match took so far; a range should take kDonateWork.
// Returns the new end of the window.  A window with too little left to cut is
// no look: the task's next one, between windows, may hand off parents.  (With
// every look of a leaf pass counted, tasks of windows of 0.5 to 1 ms handed off
// next to nothing: one task of R-MAT 15, 4-cycle unreduced 144 ms, TT4 + pendant
// 429; now 75 and 44.)
__device__ __forceinline__ uint32_t donate_leaves(Ctx& C, uint32_t lv, uint32_t from, uint32_t n, uint32_t now,
                                                  uint32_t each) {
    if (n < from + 2 * kDonatePiece) return n;
    const uint64_t pieces = (uint64_t)each * ((n - from) / 2) / kDonateWork;
    if (pieces == 0) return n;
    C.looked = now;
    uint32_t head, tail;
    uint32_t room = donation_room(C, head, tail);
    if (room == 0) return n;
    room = room < 64 ? room : 64;
    room = room < pieces ? room : (uint32_t)pieces;
    const KArgs& a = *C.a;
    const uint32_t lane = C.lane;
    Lvl F = lvl_arrays(C.scr, a.cap, lv);
    const uint32_t s = from + (n - from) / 2;
    const uint32_t pl = uni(F.parent[s]), ph = uni(F.parent[n - 1]);
    uint32_t q = ph, b = n, e = n;
    if (pl == ph) {
        // one parent: pieces of its children
        uint32_t sz = (n - s + room - 1) / room;
        sz = sz < kDonatePiece ? kDonatePiece : sz;
        b = s + lane * sz;
        e = b + sz;
        b = b < n ? b : n;
        e = e < n ? e : n;
    } else {
        // the children of each of the last parents, at most 64 of them
        const uint32_t np = ph - pl < room ? ph - pl : room;
        if (lane < np) {
            q = ph - np + 1 + lane;
            b = count_lt(F.parent, n, q);
            e = count_lt(F.parent, n, q + 1);
        }
    }
    const uint64_t m = __ballot(b < e);
    if (!m) return n;
    const uint32_t base = reserve_slots(C, (uint32_t)__popcll(m), head, tail);
    if (base == kSkip) return n;
    if (b < e) donate(C, base + rank_below(m), lv, q, F.node[b], F.node[e - 1] + 1u);
    wave_sync();
    return uni(__shfl(b, (int)__builtin_ctzll(m), 64));
}

// Size of descriptor D's candidate set (a leaf signature or a signature mask)
// for each partial match of the window, the bound nodes it may not hold taken
// off.  SUM: the sizes' sum (the same for every lane) instead, for plans with
// one leaf.  Listing and merging are in the roomy kernel with SUM only, which
// such launches always run: in the 80-VGPR kernel their code costs every launch
// registers (four motifs on R-MAT 16 20.1 ms with it).
template <bool SUM, bool ROOMY>
__device__ __forceinline__ unsigned long long leaf_set(Ctx& C, const LK& D, uint32_t nb, uint32_t p, bool pv,
                                                       uint32_t same) {
    const KArgs& a = *C.a;
    const uint32_t lane = C.lane;
    const bool listing = SUM && ROOMY && a.list != nullptr;
    const uint32_t shared = shared_cons(D, same);
    // When every constraint is on a node that the window shares (and so is the
    // reused set), all its partial matches have the same set: lane 0 measures
    // it for all, and only the bound nodes are looked up lane by lane.
    // Without and with it: C5 + chord on R-MAT 20 61 and 50 ms, 96 plans on R-MAT
    // 22 324 and 300 ms.
    const bool once = ROOMY && !listing && D.n_cons > 0 && shared == (1u << D.n_cons) - 1u && D.gt == 0 &&
                      (D.reuse == kNoReuse || (~same & ((1u << D.reuse) - 1u)) == 0);
    uint32_t flen, brow, bskip;
    uint32_t len = phase_a<true>(C, D, nb, p, pv && !(once && lane > 0), false, shared, flen, brow, bskip);
    const uint32_t ns = n_slots(D);
    Filter flt{};
    flt.vk = kSkip;
    if (ROOMY && shared && a.filt_words) use_filter(C, D, nb, shared, flen, len, flt);
    // one leaf whose set is a base list and one probe list: balanced big pairs
    // leave the flattened pass for the cooperative merge (a set measured once is
    // scanned: a merge settles one partial match's bound nodes only)
    bool big = false;
    if (SUM && ROOMY && a.merge_min != 0xFFFFFFFFu && pv && !listing && !once) {
        uint32_t nprobe = 0, pl = 0;
        for (uint32_t c = 0; c < ns; c++)
            if (C.s.slot_len[c * 64 + lane] != kSkip) {
                pl = C.s.slot_len[c * 64 + lane];
                nprobe++;
            }
        if (nprobe == 1 && pl != kRowLen) {
            const uint32_t mn = len < pl ? len : pl, mx = len < pl ? pl : len;
            big = mn >= a.merge_min && (uint64_t)mx <= (uint64_t)a.merge_ratio * mn;
        }
    }
    uint64_t bigmask = SUM && ROOMY ? __ballot(big) : 0ull;
    // long base lists leave the flattened pass too (listing stays flattened)
    Par P1 = parent_view(C, ns, len);
    const bool wd = len >= kWideMin && !big && !listing && !D.deg_check;
    const bool rows = wd && P1.rows_only && P1.n_rows > 0 && P1.len > 0;
    uint64_t wide = __ballot(wd && P1.len > 0 && !rows);
    Dense dn{};
    if (rows) dn = take_dense(C, D, nb, brow, bskip, P1);
    const uint64_t words = __ballot(dn.w1 > dn.w0), chunks = __ballot(rows && P1.len > 0);
    if (big || wd) len = 0;
    const uint32_t incl = scan_incl(len, lane);
    C.s.incl[lane] = incl;
    const uint32_t T = uni(__shfl(incl, 63, 64));
    const bool owns = len > 0;
    const uint32_t start = incl - len;
    wave_sync();
    unsigned long long lin = 0;
    uint32_t h = 0, carry = 0, held = 0;
    // two tiles per step
    for (uint32_t t0 = 0; t0 < T; t0 += 128) {
        const uint32_t ga = t0 + lane, gb = t0 + 64 + lane;
        uint32_t ja, jb;
        tile_parents(C.s, lane, t0, start, owns, carry, ja, jb);
        const uint32_t la = ga - (ja ? C.s.incl[ja - 1] : 0u);
        const uint32_t lb = gb - (jb ? C.s.incl[jb - 1] : 0u);
        bool oka = ga < T && la < C.s.base_len[ja];
        bool okb = gb < T && lb < C.s.base_len[jb];
        uint32_t xa = 0, xb = 0;
        if (oka) xa = base_elem(C, ja, la);
        if (okb) xb = base_elem(C, jb, lb);
        // injectivity is settled per partial match below (per element when
        // every embedding is written out)
        check_pair<ROOMY>(C, D, flt, listing ? D.inj : 0u, nb, ns, ja, xa, oka, jb, xb, okb);
        const uint64_t ma = __ballot(oka), mb = __ballot(okb);
        if (SUM) {
            lin += (unsigned long long)(__popcll(ma) + __popcll(mb));
            if (listing) {
                hold_rows(C, nb, held, ma, ja, xa, oka);
                hold_rows(C, nb, held, mb, jb, xb, okb);
            }
        } else if (owns) {
            h += own_count(ma, start, len, t0) + own_count(mb, start, len, t0 + 64);
        }
    }
    if (SUM && listing) write_rows(C, nb, held);
    auto add = [&](uint32_t j, uint32_t n) {
        if (SUM) lin += n;
        else h += lane == j ? n : 0u;
    };
    if (words) {
        uint32_t vacc = 0;  // SUM: this lane's share of all chunks
        word_scan(C, P1, dn, D.gt != 0, words, [&](uint32_t j, uint32_t v) {
            if (SUM) vacc += v;
            else add(j, uni(__shfl(scan_incl(v, lane), 63, 64)));
        });
        // (64 lists of the largest size stay below 2^32 elements)
        if (SUM) lin += uni(__shfl(scan_incl(vacc, lane), 63, 64));
    }
    if (chunks) chunk_scan<ROOMY>(C, P1, chunks, add);
    for (; wide; wide &= wide - 1) {
        const uint32_t j = (uint32_t)__builtin_ctzll(wide);
        add(j, wide_count(C, D, nb, ns, j));
    }
    if (once) {
        h = pv ? uni(h) : 0u;
        if (SUM) lin *= (unsigned long long)__popcll(__ballot(pv));
        wave_sync();
    }
    // the bound nodes the set may not contain were counted if present
    for (uint32_t b = 0; b < nb && !listing; b++) {
        if (!((D.inj >> b) & 1u)) continue;
        const bool hit = pv && !big && bound_in_set(C, ns, C.s.bound[b * 64 + lane], once ? 0u : lane);
        if (SUM) lin -= (unsigned long long)__popcll(__ballot(hit));
        else h -= hit ? 1u : 0u;
    }
    wave_sync();
    // balanced big pairs, one partial match at a time
    for (; SUM && ROOMY && bigmask; bigmask &= bigmask - 1) {
        const uint32_t j = (uint32_t)__builtin_ctzll(bigmask);
        const uint32_t blen = uni(C.s.base_len[j]);
        uint32_t pc = 0;
        for (uint32_t c = 0; c < ns; c++)
            if (C.s.slot_len[c * 64 + j] != kSkip) pc = c;
        pc = uni(pc);
        const uint32_t plen = uni(C.s.slot_len[pc * 64 + j]);
        const gptr A = join_ptr(uni(C.s.base_lo[j]), uni(C.s.base_hi[j]));
        const gptr B = join_ptr(uni(C.s.slot_lo[pc * 64 + j]), uni(C.s.slot_hi[pc * 64 + j]));
        lin += merge_count(C.s, A, blen, B, plen, D.inj, nb, j, lane);
    }
    return SUM ? lin : (unsigned long long)h;
}

// The same for a descriptor with one list L and no reuse: |L| (the part beyond
// the symmetry bound) minus the bound nodes found in it, per partial match.
__device__ __forceinline__ uint32_t leaf_list(const Ctx& C, const LK& D, uint32_t nb, bool pv) {
    if (!pv) return 0;
    const uint32_t lane = C.lane;
    const DevGraph& g = C.a->g;
    const uint32_t nd = C.s.bound[D.lvl(0) * 64 + lane];
    const uint32_t* off = off_of(g, D.dir(0));
    const uint32_t o = off[nd];
    uint32_t l = off[nd + 1] - o;
    const uint32_t* L = adj_of(g, D.dir(0)) + o;
    if (D.gt) sym_trim(C.s, D.gt, D.lt, nb, lane, L, l);
    uint32_t v = l;
    for (uint32_t b = 0; b < nb; b++)
        if (((D.inj >> b) & 1u) && contains(L, l, C.s.bound[b * 64 + lane])) v -= 1;
    return v;
}

// Leaf group of the 64 partial matches of a window, lane by lane: the plan's
// one signature (linear), or several: for every signature mask M the terms
// use, h[M] = |intersection over s in M of S_s| is measured, then the
// inclusion-exclusion terms over set partitions of the leaves are summed in
// 128-bit integers.
template <bool ROOMY>
__device__ __forceinline__ void leaf_masks(Ctx& C, uint32_t nb, uint32_t p, bool pv, uint32_t same) {
    const KArgs& a = *C.a;
    const PlanDesc* P = C.P;
    const uint32_t lane = C.lane;
    const bool linear = uni(P->linear) != 0;
    const uint32_t n_masks = linear ? 1u : uni(P->n_masks);
    for (uint32_t mi = 0; mi < n_masks; mi++) {
        const LK K = load_lk(linear ? P->sig[0] : P->mdesc[mi], a);
        const uint32_t h = K.n_cons == 1 && K.reuse == kNoReuse
                               ? leaf_list(C, K, nb, pv)
                               : (uint32_t)leaf_set<false, ROOMY>(C, K, nb, p, pv, same);
        if (linear) {
            if (u128_add(C.acc_lo, C.acc_hi, h, 0ull)) C.ovf = true;
            return;
        }
        // every mask whose test is this entry's takes its size
        for (uint32_t ms = uni(P->mask_set[mi]) & 0xFFFEu; ms; ms &= ms - 1)
            C.s.hist[(uint32_t)__builtin_ctz(ms) * 64 + lane] = h;
    }
    wave_sync();
    if (pv) {
        // inclusion-exclusion over set partitions of the leaves; a term whose
        // magnitude could pass 2^120 marks the plan as overflowed
        __int128 val = 0;
        bool big = false;
        const uint32_t n_terms = uni(P->n_terms);
        for (uint32_t t = 0; t < n_terms; t++) {
            const Term& tm = P->terms[t];
            uint32_t hv[kMaxBlocks];
            const uint32_t nb = tm.nb < kMaxBlocks ? tm.nb : kMaxBlocks;
            for (uint32_t b = 0; b < nb; b++) hv[b] = C.s.hist[(tm.mask[b] & 15u) * 64 + lane];
            val += ie_term(tm.coef, hv, nb, &big);
        }
        // the injective count of one partial match is never negative
        const unsigned __int128 v = (unsigned __int128)(val < 0 ? (__int128)0 : val);
        if (big || val < 0) C.ovf = true;
        if (u128_add(C.acc_lo, C.acc_hi, (unsigned long long)v, (unsigned long long)(v >> 64))) C.ovf = true;
    }
    wave_sync();
}

// Count the leaf group for every partial match in level `lv` (= e - 1).
template <bool NONLIN, bool ROOMY>
__device__ __forceinline__ void count_leaves(Ctx& C, uint32_t lv, uint32_t nprefix) {
    const KArgs& a = *C.a;
    const PlanDesc* P = C.P;
    const uint32_t lane = C.lane;
    const uint32_t nb = lv + 1;  // bound levels 0..lv
    const LK S0 = load_lk(P->sig[0], a);
    const uint32_t entered = (uint32_t)__builtin_readcyclecounter();
    for (uint32_t w0 = 0; w0 < nprefix; w0 += 64) {
        // a leaf pass over hub lists can run long: look at the cancel flag
        // every 8 blocks of 64 prefixes
        if (a.cancel && (++C.polls & 7u) == 0) {
            uint32_t stop = 0;
            if (lane == 0) stop = __atomic_load_n(a.cancel, __ATOMIC_RELAXED) != 0;
            if (uni(__shfl(stop, 0, 64))) {
                if (lane == 0) atomicOr(&a.ctl[kCtlCancelled], 1u);
                C.stop = true;
                return;
            }
        }
        uint32_t now;
        if (lv > 0 && w0 > 0 && time_to_look(C, now))
            nprefix = donate_leaves(C, lv, w0 + 64, nprefix, now, (now - entered) / w0);
        const uint32_t p = w0 + lane;
        const bool pv = p < nprefix;
        // walk the chain once: bound nodes of levels 0..lv
        if (pv) {
            uint32_t idx = p;
            for (int l = (int)lv; l >= 0; --l) {
                Lvl F = lvl_arrays(C.scr, a.cap, (uint32_t)l);
                C.s.bound[l * 64 + lane] = F.node[idx];
                C.s.anc[l * 64 + lane] = idx;
                if (l > 0) idx = F.parent[idx];
            }
        }
        const uint32_t same = ROOMY && !a.list ? same_levels(C, nb, pv) : 0u;
        if (NONLIN) {
            leaf_masks<ROOMY>(C, nb, p, pv, same);
        } else {
            unsigned long long v = 0;
            if ((!ROOMY || a.list == nullptr) && S0.n_cons == 1 && S0.reuse == kNoReuse) {
                v = leaf_list(C, S0, nb, pv);
            } else {
                v = leaf_set<true, ROOMY>(C, S0, nb, p, pv, same);
                v = lane == 0 ? v : 0ull;
            }
            if (u128_add(C.acc_lo, C.acc_hi, v, 0ull)) C.ovf = true;
        }
        wave_sync();
    }
}

__device__ __forceinline__ void flush(Ctx& C) {
    unsigned long long lo = C.acc_lo, hi = C.acc_hi;
    bool ovf = C.ovf;
    // wave reduction of 128-bit partials
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        unsigned long long olo = __shfl_xor(lo, d, 64);
        unsigned long long ohi = __shfl_xor(hi, d, 64);
        if (u128_add(lo, hi, olo, ohi)) ovf = true;
    }
    const bool any_ovf = __ballot(ovf) != 0;
    if (C.lane == 0 && (lo | hi))
        add_u128(C.a->partial + (blockIdx.x % C.a->copies) * C.a->copy_words + 2 * C.pi, lo, hi,
                 C.a->plan_flags + C.pi);
    if (C.lane == 0 && any_ovf) atomicOr(C.a->plan_flags + C.pi, 1u);
    C.acc_lo = C.acc_hi = 0;
    C.ovf = false;
}

// Depth-first exploration of the n0 partial matches held in level start-1
// (start = 1: roots in level 0).
template <bool NONLIN, bool ROOMY>
__device__ __forceinline__ void explore(Ctx& C, uint32_t n0, uint32_t start) {
    const uint32_t e = C.P->e;
    uint32_t* st = C.s.st;
    if (e == 1) {
        count_leaves<NONLIN, ROOMY>(C, 0, n0);
        return;
    }
    if (C.lane == 0) {
        st[16 + start - 1] = n0;
        st[start] = 0;
        st[8 + start] = 0;
    }
    wave_sync();
    C.begun = C.looked = (uint32_t)__builtin_readcyclecounter();
    uint32_t lv = start;
    uint32_t windows = 0;
    for (;;) {
        uint32_t nparents = uni(st[16 + lv - 1]);
        uint32_t cur = uni(st[lv]);
        if (cur >= nparents) {
            if (lv == start) break;
            lv -= 1;
            continue;
        }
        ++windows;
        // a long task still notices the cancel flag (counts are then partial)
        if (C.a->cancel && (windows & 15u) == 0) {
            uint32_t stop = 0;
            if (C.lane == 0) stop = __atomic_load_n(C.a->cancel, __ATOMIC_RELAXED) != 0;
            if (uni(__shfl(stop, 0, 64))) {
                if (C.lane == 0) atomicOr(&C.a->ctl[kCtlCancelled], 1u);
                break;
            }
        }
        uint32_t now;
        if (lv >= 2 && time_to_look(C, now)) {
            C.looked = now;
            if (now - C.begun >= kDonateParents) donate_parents(C, start, lv);
        }
        uint32_t nout = expand(C, lv);
        if (lv == e - 1) {
            if (nout) count_leaves<NONLIN, ROOMY>(C, lv, nout);
            if (C.stop) break;
        } else if (nout) {
            lv += 1;
            if (C.lane == 0) {
                st[lv] = 0;
                st[8 + lv] = 0;
            }
            wave_sync();
        }
    }
}

// Two register budgets.  MINB resident blocks per CU: kFullBlocksPerCu (6 waves
// per SIMD, 80 VGPRs, 90 of them spilled, 230-280 B of scratch a lane) for launches of more than
// kRoomyBlocksPerCu blocks per CU, and kRoomyBlocksPerCu (3 waves per SIMD, no
// scratch) for launches of at most that many.  The larger one
// at 8 / 7 / 6 blocks: four motifs on R-MAT 16 18.2 / 18.5 / 17.8 ms, unreduced
// 152 / 152 / 144 ms, a tenth of the roots 38.6 / 38.6 / 37.6 ms.
template <bool NONLIN, int MINB>
__global__ void __launch_bounds__(kBlockThreads, MINB) count_kernel(KArgs a) {
    constexpr bool ROOMY = MINB <= kRoomyBlocksPerCu;
    extern __shared__ uint32_t smem[];
    Ctx C;
    C.a = &a;
    C.lane = lane_id();
    // uniform over the wave, stated so: what is addressed from it stays in scalar
    // registers (without it the roomy kernels spill 15 and 18 of their 168 VGPRs,
    // with it none of 168 and 162)
    const uint32_t wid = uni(threadIdx.x >> 6);
    C.s = carve(smem + wid * a.lds_words, a.lds_rows, a.maxc, a.merge_min != 0xFFFFFFFFu,
                a.filt_words);
    const uint64_t gw = (uint64_t)blockIdx.x * kWavesPerBlock + wid;
    C.scr = a.scratch + gw * (uint64_t)a.wave_words;
    C.acc_lo = C.acc_hi = 0;
    C.ovf = false;
    C.pi = 0;
    C.P = a.plans;
    C.stop = false;
    C.polls = 0;
    C.begun = C.looked = 0;
    // this wave's home split queue: the XCD its block runs on (blocks go to
    // the 8 XCDs round-robin), so a hub's sub-range tasks share one L2
    const uint32_t home = blockIdx.x % kQueues;
    bool split_left = true;
    // 64-bit: the host keeps the product below 2^32 (root items are 32-bit)
    const uint64_t chunks_per_plan = ((uint64_t)a.n_src + a.chunk - 1) / a.chunk;
    const uint64_t total_chunks = chunks_per_plan * a.n_plans;
    if (C.lane < 4) C.s.st[27 + C.lane] = 0;  // no list is in the filter yet, nothing was donated
    Lvl F0 = lvl_arrays(C.scr, a.cap, 0);
    uint32_t taken = 0;
    // root items (item = chunk index x n_plans + plan) come from kQueues
    // cursors, so the grabs spread over several words and every cursor still
    // walks its items in order; a wave starts at its home cursor (its XCD's)
    // and moves on once one runs dry
    uint32_t rq = home, sq = home;
    bool roots_left = true;
    auto item_at = [&](uint32_t q, uint32_t c) -> uint64_t {
        if (a.n_plans > kQueues) {
            // chunk-major: cursor q walks the chunk indices q, q + kQueues, ...
            // with all plans of one index in a row, so the plans whose
            // chunks hold the same roots run on one XCD and share its L2
            const uint64_t ci = (uint64_t)q + (uint64_t)kQueues * (c / a.n_plans);
            return ci * a.n_plans + c % a.n_plans;
        }
        // plan-major: with few plans, cursor q keeps to the plans q mod
        // n_plans, so a wave's counts stay in its lanes between tasks
        return (uint64_t)q + (uint64_t)kQueues * c;
    };
    // A wave counts as active from its first task until the queues run dry
    // (and again while it runs a donated task), not per task.  The count is
    // spread over kActiveLines cache lines: atomics of all waves on one line
    // take ~14 ns each, which was most of a small launch (8,192 waves, four
    // updates each: 4 patterns on 2,000 nodes 545 us a launch).
    uint32_t* const active_line = a.ctl + kCtlActive0 + 32 * (blockIdx.x % kActiveLines);
    bool active = true;
    if (C.lane == 0) atomicAdd(active_line, 1u);
    for (;;) {
        // ---- take a task
        // (the lane number is made opaque: otherwise the per-lane addresses
        // below are computed ahead of the loop and kept, spilled, through explore)
        uint32_t ln = C.lane;
        asm volatile("" : "+v"(ln));
        uint32_t kind = 2, item = 0;
        bool stop = false;
        // the flag may sit in host memory: poll it on every 32nd task only
        if (a.cancel && (taken++ & 31u) == 0) {
            uint32_t c = 0;
            if (ln == 0) c = __atomic_load_n(a.cancel, __ATOMIC_RELAXED) != 0;
            stop = uni(__shfl(c, 0, 64)) != 0;
            if (stop && ln == 0) atomicOr(&a.ctl[kCtlCancelled], 1u);
        }
        // split queues: the home queue first, then the others (stealing); the
        // split kernel has finished, so an empty queue stays empty.  Each head
        // has a cache line of its own: with all heads on one line the atomics of
        // 230,000 tasks (four motifs, R-MAT 16) took 10 of a launch's 33 ms.
        while (!stop && split_left && kind == 2) {
            const uint32_t qcap = a.qbase[sq + 1] - a.qbase[sq];
            if (qcap) {
                uint32_t it = 0, cnt = 0;
                if (ln == 0) {
                    it = atomicAdd(&a.ctl[kCtlSplitHead0 + 32 * sq], 1u);
                    cnt = __atomic_load_n(&a.ctl[kCtlSplitCount0 + sq], __ATOMIC_RELAXED);
                }
                it = uni(__shfl(it, 0, 64));
                cnt = uni(__shfl(cnt, 0, 64));
                if (it < (cnt < qcap ? cnt : qcap)) {
                    kind = 0;
                    item = a.qbase[sq] + it;
                    break;
                }
            }
            // lane t reads the state of queue sq + 1 + t: one round trip shows
            // every queue, and a read does not serialise like a failing atomic
            bool left = false;
            if (ln < kQueues - 1) {
                const uint32_t q = (sq + 1 + ln) % kQueues;
                const uint32_t cap = a.qbase[q + 1] - a.qbase[q];
                if (cap) {
                    const uint32_t cnt = __atomic_load_n(&a.ctl[kCtlSplitCount0 + q], __ATOMIC_RELAXED);
                    left = __atomic_load_n(&a.ctl[kCtlSplitHead0 + 32 * q], __ATOMIC_RELAXED) < (cnt < cap ? cnt : cap);
                }
            }
            const uint64_t m = __ballot(left);
            if (m) sq = (sq + 1 + (uint32_t)__builtin_ctzll(m)) % kQueues;
            else split_left = false;
        }
        while (!stop && roots_left && kind == 2) {
            uint32_t c = 0;
            if (ln == 0) c = atomicAdd(&a.ctl[kCtlRootCursor0 + 32 * rq], 1u);
            const uint64_t it = item_at(rq, uni(__shfl(c, 0, 64)));
            if (it < total_chunks) {
                kind = 1;
                item = (uint32_t)it;
                break;
            }
            // as above: lane t reads cursor rq + 1 + t
            bool left = false;
            const uint32_t q = (rq + 1 + ln) % kQueues;
            if (ln < kQueues - 1)
                left = item_at(q, __atomic_load_n(&a.ctl[kCtlRootCursor0 + 32 * q], __ATOMIC_RELAXED)) < total_chunks;
            const uint64_t m = __ballot(left);
            if (m) rq = (rq + 1 + (uint32_t)__builtin_ctzll(m)) % kQueues;
            else roots_left = false;
        }
        if (kind == 2 && active) {
            if (ln == 0) atomicSub(active_line, 1u);
            active = false;
        }
        if (kind == 2 && !stop) {
            // queues drained: wait for donated work while any wave still holds a
            // task.  About kMaxWaiters waves wait (the others leave at once),
            // and they poll with growing pauses, so waiting waves do not crowd
            // the cache lines the working waves update.
            // No entry is left behind: a wave that donated leaves only when the
            // head has passed its last entry, whatever the number of waiters.
            // (With donors that stayed until the queue was empty, thousands of
            // them polled it: three unreduced plans on a hub root of R-MAT 15 322
            // ms, now 43.)
            uint32_t idle = 0;
            if (ln == 0) idle = __atomic_load_n(&a.ctl[kCtlIdle], __ATOMIC_RELAXED);
            const bool wait = uni(__shfl(idle, 0, 64)) < kMaxWaiters;
            const uint32_t given = uni(C.s.st[30]);
            if (wait || given) {
                // between the read and this add a few more waves than
                // kMaxWaiters may come in; they may wait as well
                if (wait && ln == 0) atomicAdd(&a.ctl[kCtlIdle], 1u);
                uint32_t nap = 1;
                for (uint32_t polls = 0; polls < kIdlePolls; polls++) {
                    // queue entries [head, tail).  A waiter tries an entry of its own
                    // choosing, so the claims spread over the entries (one CAS on
                    // the head by all waiters took ~7 us a task); now and then it is
                    // the head, which moves past entries that were read.
                    uint32_t h = 0, t = 0, got = kSkip;
                    if (ln == 0) {
                        h = __atomic_load_n(&a.ctl[kCtlDonHead], __ATOMIC_RELAXED);
                        t = __atomic_load_n(&a.ctl[kCtlDonTail], __ATOMIC_RELAXED);
                        if (h < t) {
                            const uint32_t r = (uint32_t)(gw * 2654435761u + polls * 40503u) >> 9;
                            const uint32_t s = (r & 3u) ? h + r % (t - h) : h;
                            uint32_t* const word = &a.don[(uint64_t)don_slot(s, a.don_cap) * kDonWords + 1];
                            const uint32_t pub = don_published(s, a.don_cap);
                            const uint32_t seen = __atomic_load_n(word, __ATOMIC_RELAXED);
                            if (seen == pub && atomicCAS(word, pub, pub + 1u) == pub) got = s;
                            for (uint32_t i = 0; s == h && h < t && i < 8; i++) {
                                if (__atomic_load_n(&a.don[(uint64_t)don_slot(h, a.don_cap) * kDonWords + 1],
                                                    __ATOMIC_RELAXED) != don_read(h, a.don_cap))
                                    break;
                                atomicCAS(&a.ctl[kCtlDonHead], h, h + 1);
                                h++;
                            }
                        }
                    }
                    got = uni(__shfl(got, 0, 64));
                    h = uni(__shfl(h, 0, 64));
                    t = uni(__shfl(t, 0, 64));
                    if (got != kSkip) {
                        kind = 3;
                        item = got;
                        break;
                    }
                    if (!wait && h >= given) break;
                    // a line of control words serves ~70 accesses a us: hundreds of
                    // waiters that look at once slow every other update down
                    if (h >= t) {
                        uint32_t act = 0;
                        if (ln < kActiveLines)
                            act = __atomic_load_n(&a.ctl[kCtlActive0 + 32 * ln], __ATOMIC_RELAXED);
                        if (!__ballot(act != 0)) break;
                        if (a.cancel && (polls & 63u) == 0) {
                            uint32_t c = 0;
                            if (ln == 0) c = __atomic_load_n(a.cancel, __ATOMIC_RELAXED) != 0;
                            if (uni(__shfl(c, 0, 64))) break;
                        }
                    }
                    // pauses double from ~0.2 us, so a launch ends within about
                    // twice its last task's remaining time or the longest pause
                    for (uint32_t z = 0; z < nap; z++) __builtin_amdgcn_s_sleep(8);
                    nap = nap < kNapMax ? nap * 2 : kNapMax;
                }
                if (wait && ln == 0) atomicSub(&a.ctl[kCtlIdle], 1u);
            }
        }
        if (kind == 3) {
            if (ln == 0) atomicAdd(active_line, 1u);
            active = true;
        }
        if (kind == 2) break;
        uint32_t n0 = 0, start = 1;
        // counts of consecutive tasks of one plan stay in the lanes'
        // accumulators: flush only when the plan changes (and at the end)
        auto set_plan = [&](uint32_t pi) {
            if (pi != C.pi) {
                flush(C);
                C.pi = pi;
            }
            C.P = a.plans + C.pi;
        };
        if (kind == 0) {
            uint4 it = a.split_items[item];
            set_plan(uni(it.x));
            if (C.lane == 0) {
                F0.node[0] = it.y;
                F0.parent[0] = it.z;
                F0.aux[0] = it.w;
            }
            n0 = 1;
        } else if (kind == 3) {
            // a donated prefix: bind levels 0..d-1 as single entries and explore from
            // level d, within the id range that came with it
            uint32_t* ent = a.don + (uint64_t)don_slot(item, a.don_cap) * kDonWords;
            asm volatile("" ::: "memory");  // (its words are read past L2, after the claim)
            const uint32_t head = uni(__atomic_load_n(&ent[0], __ATOMIC_RELAXED));
            set_plan(head & 0xFFFFu);
            start = head >> 16;
            if (C.lane < start) {
                Lvl F = lvl_arrays(C.scr, a.cap, C.lane);
                F.node[0] = __atomic_load_n(&ent[2 + C.lane], __ATOMIC_RELAXED);
                F.parent[0] = 0;
                F.segc[0] = 0;  // no complete child segments: reusers fetch their lists
                F.aux[0] = kSkip;
            }
            if (C.lane == 0) {
                C.s.st[25] = __atomic_load_n(&ent[kDonWords - 2], __ATOMIC_RELAXED);
                C.s.st[26] = __atomic_load_n(&ent[kDonWords - 1], __ATOMIC_RELAXED);
            }
            // every word has arrived: the slot is free for another task
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (C.lane == 0) __atomic_store_n(&ent[1], don_read(item, a.don_cap), __ATOMIC_RELAXED);
            n0 = 1;
        } else {
            // interleave plans so that all of them start on the low (hub) ids
            set_plan(uni(item % a.n_plans));
            const uint32_t ci = item / a.n_plans;
            // without a root list, a plan on a root share counts the ids
            // (j + 1) 2^s - 1 only: its chunks run over j, so that every lane
            // of a chunk gets a root of the share (n >> s of them)
            const uint32_t sh = C.P->root_share;
            const bool compact = a.roots == nullptr && sh > 0;
            const uint64_t n_p = compact ? ((uint64_t)a.n_src >> sh) : (uint64_t)a.n_src;
            const uint64_t cpp = compact ? (n_p + a.chunk - 1) / a.chunk : chunks_per_plan;
            // chunk ci takes the roots ci, ci + chunks, ci + 2 chunks, ...: long
            // lists cluster at low ids on power-law generators, and striding
            // spreads them over many tasks
            const uint64_t idx64 = (uint64_t)ci + (uint64_t)C.lane * cpp;
            const uint32_t idx = (uint32_t)(idx64 < n_p ? idx64 : n_p);
            bool ok = C.lane < a.chunk && ci < cpp && idx64 < n_p;
            uint32_t r = 0;
            if (ok) {
                r = compact ? (uint32_t)(((idx64 + 1) << sh) - 1) : (a.roots ? a.roots[idx] : idx);
                ok = r < a.g.n && in_root_share(r, sh);
            }
            if (ok) {
                uint2 d = a.g.deg[r];
                ok = d.x >= C.P->root_dout && d.y >= C.P->root_din;
            }
            if (ok && C.P->e >= 2) {
                uint32_t l = level1_len(a.g, C.P, r);
                // longer lists were queued as sub-ranges by the split kernel
                ok = l > 0 && l <= plan_item_size(l, C.P->e, a.split, a.split_work, a.cap);
            }
            uint64_t m = __ballot(ok);
            if (ok) {
                uint32_t pos = rank_below(m);
                F0.node[pos] = r;
                F0.parent[pos] = 0;
                F0.aux[pos] = kSkip;
            }
            n0 = (uint32_t)__popcll(m);
        }
        if (C.lane == 0) C.s.st[24] = kind == 3 ? start : 0u;
        wave_sync();
        if (n0) explore<NONLIN, ROOMY>(C, n0, start);
        if (C.stop) break;
    }
    // a wave that was counted as active must not stay so after a cancel
    if (C.lane == 0 && C.stop && active) atomicSub(active_line, 1u);
    flush(C);
}

// Hub roots whose first-level list is longer than `split` become several
// queued sub-range tasks.  Must agree with the root filter of count_kernel.
// A lane looks at one (root, plan); the wave writes the tasks of its lanes one
// after the other, 64 at a time (a root has up to kMaxPieces tasks: written by
// its own lane they took 170 us).
__global__ void split_kernel(KArgs a) {
    const uint32_t nsrc = a.roots ? a.n_src : a.n_hubs;
    const uint64_t total = (uint64_t)nsrc * a.n_plans;
    const uint32_t lane = lane_id();
    for (uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63u); i0 < total;
         i0 += (uint64_t)gridDim.x * blockDim.x) {
        // root-major: the tasks of all plans on one hub are pushed together,
        // so the waves of its XCD work on that hub's lists side by side
        const uint64_t i = i0 + lane;
        const uint32_t pi = (uint32_t)(i % a.n_plans);
        const uint32_t h = (uint32_t)(i / a.n_plans);
        const PlanDesc* P = a.plans + pi;
        uint32_t r = 0, len = 0, sz = 1, nit = 0, at = 0;
        if (i < total && P->e >= 2) {
            r = a.roots ? a.roots[h] : a.hubs[h];
            if (r < a.g.n && in_root_share(r, P->root_share)) {
                const uint2 d = a.g.deg[r];
                if (d.x >= P->root_dout && d.y >= P->root_din) {
                    len = level1_len(a.g, P, r);
                    sz = plan_item_size(len, P->e, a.split, a.split_work, a.cap);
                    nit = len > sz ? (len + sz - 1) / sz : 0;
                }
            }
        }
        if (nit) {
            // all tasks of one root go to one queue (one XCD's L2)
            const uint32_t qu = h % kQueues;
            const uint32_t qcap = a.qbase[qu + 1] - a.qbase[qu];
            const uint32_t base = atomicAdd(&a.ctl[kCtlSplitCount0 + qu], nit);
            at = a.qbase[qu] + base;
            if (base + nit > qcap) {
                atomicOr(&a.ctl[kCtlQueueFull], 1u);
                nit = 0;
            }
        }
        for (uint64_t m = __ballot(nit > 0); m; m &= m - 1) {
            const int j = __builtin_ctzll(m);
            const uint32_t n = uni(__shfl(nit, j, 64)), s = uni(__shfl(sz, j, 64)), l = uni(__shfl(len, j, 64));
            const uint32_t p = uni(__shfl(pi, j, 64)), root = uni(__shfl(r, j, 64)), to = uni(__shfl(at, j, 64));
            for (uint32_t q = lane; q < n; q += 64) {
                const uint32_t lo = q * s, hi = lo + s < l ? lo + s : l;
                a.split_items[to + q] = make_uint4(p, root, lo, hi);
            }
        }
    }
}

// Copy plan descriptors into the workspace table and clear control state.
__global__ void init_kernel(InitArgs a) {
    const uint32_t words = sizeof(PlanDesc) / 4;
    const uint32_t tid = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t nthr = gridDim.x * blockDim.x;
    for (uint32_t i = tid; i < a.count * words; i += nthr) {
        uint32_t pl = i / words, w = i % words;
        reinterpret_cast<uint32_t*>(a.table + a.first + pl)[w] =
            reinterpret_cast<const uint32_t*>(a.src[pl])[w];
    }
    if (a.zero_ctl) {
        for (uint32_t i = tid; i < kCtlWords; i += nthr) a.ctl[i] = 0;
        for (uint32_t i = tid; i < a.n_plans; i += nthr) a.plan_flags[i] = 0;
        for (uint32_t i = tid; i < a.partial_words; i += nthr) a.partial[i] = 0;
        // the workspace is reused across launches (and by the caller's
        // allocator): a slot is ready only once this launch publishes it
        for (uint32_t i = tid; i < a.don_cap; i += nthr) a.don[(uint64_t)i * kDonWords + 1] = 0;
        if (a.list_count && tid == 0) *a.list_count = 0;
    }
}

// Per-plan totals, and status from the flags the count kernel raised (one block).
__global__ void finalize_kernel(KArgs a) {
    // every donated task must have been taken (the head may stop short of the
    // last ones): one left behind would be missing from the counts
    const bool left = __syncthreads_or(don_left(a.don, kDonWords, a.don_cap, a.ctl[kCtlDonHead], a.ctl[kCtlDonTail],
                                                threadIdx.x, blockDim.x)) != 0;
    for (uint32_t i = threadIdx.x; i < a.n_plans; i += blockDim.x) {
        int32_t st = 0;
        if (a.ctl[kCtlBadPlan] || (left && !a.ctl[kCtlCancelled])) st = -1;
        else if (a.ctl[kCtlQueueFull]) st = -6;
        else if (a.ctl[kCtlCancelled]) st = -7;
        else if (a.plan_flags[i] & 1u) st = -5;
        // the copies' totals, added up
        unsigned long long lo = 0, hi = 0;
        bool big = false;
        for (uint32_t c = 0; c < a.copies; c++) {
            const unsigned long long* p = a.partial + (uint64_t)c * a.copy_words + 2 * i;
            if (u128_add(lo, hi, p[0], p[1])) big = true;
        }
        if (big && st == 0) st = -5;
        const uint32_t m = a.plans[i].sym_mult;
        // one embedding per orbit was counted: scale the 128-bit total
        if (m > 1 && st == 0 && u128_scale(lo, hi, m)) st = -5;
        a.counts[2 * i] = lo;
        a.counts[2 * i + 1] = hi;
        a.status[i] = st;
    }
}

// Workspace of xm_count_static: a fixed array in device memory, one copy per
// device, so that launches need no allocation.  Host code never uses this
// name as an address: the address comes from hipGetSymbolAddress.
static __device__ __align__(256) uint8_t g_static_scratch[kStaticScratchBytes];

hipError_t static_scratch_address(void** ptr) {
    return hipGetSymbolAddress(ptr, HIP_SYMBOL(g_static_scratch));
}

__global__ void desc_chunk_kernel(DescChunk c) {
    for (uint32_t i = threadIdx.x; i < c.n; i += blockDim.x) c.dst[i] = c.w[i];
}

hipError_t copy_desc(PlanDesc* dst, const PlanDesc& src, hipStream_t stream) {
    const uint32_t words = sizeof(PlanDesc) / 4;
    const uint32_t* s = reinterpret_cast<const uint32_t*>(&src);
    for (uint32_t o = 0; o < words; o += kDescChunkWords) {
        DescChunk c;
        c.dst = reinterpret_cast<uint32_t*>(dst) + o;
        c.n = words - o < kDescChunkWords ? words - o : kDescChunkWords;
        for (uint32_t i = 0; i < c.n; i++) c.w[i] = s[o + i];
        hipLaunchKernelGGL(desc_chunk_kernel, dim3(1), dim3(256), 0, stream, c);
    }
    return hipGetLastError();
}

int count_blocks_per_cu(bool nonlin, size_t lds_bytes) {
    int nb = 0;
    hipError_t e;
    if (nonlin)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, count_kernel<true, kFullBlocksPerCu>, kBlockThreads, lds_bytes);
    else
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, count_kernel<false, kFullBlocksPerCu>, kBlockThreads, lds_bytes);
    return e == hipSuccess ? nb : 0;
}

// One block per dense row: set the bit of every list element.
__global__ void rows_kernel(DevGraph g, const uint32_t* row_node, uint32_t n_out_rows, uint32_t n_rows,
                            uint32_t* rows) {
    for (uint32_t r = blockIdx.x; r < n_rows; r += gridDim.x) {
        const uint32_t dir = r >= n_out_rows ? 1u : 0u;
        const uint32_t v = row_node[r];
        const uint32_t* off = off_of(g, dir);
        const uint32_t* adj = adj_of(g, dir);
        uint32_t* row = rows + (uint64_t)r * g.row_words;
        for (uint32_t i = off[v] + threadIdx.x; i < off[v + 1]; i += blockDim.x) {
            const uint32_t x = adj[i];
            atomicOr(&row[x >> 5], 1u << (x & 31u));
        }
    }
}

// Head of each row where words beat elements: the number of words w (a power
// of two times 256, or the whole row) with the largest kDenseWords x elements - w.
__global__ void row_pre_kernel(DevGraph g, const uint32_t* row_node, uint32_t n_out_rows, uint32_t n_rows, uint2* pre) {
    const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n_rows) return;
    const uint32_t dir = r >= n_out_rows ? 1u : 0u, v = row_node[r];
    const uint32_t* off = off_of(g, dir);
    const uint32_t o = off[v], len = off[v + 1] - o;
    const uint32_t* list = adj_of(g, dir) + o;
    const uint32_t whole = g.row_words / 4 * 4;
    uint2 best = make_uint2(0, 0);
    int64_t gain = 0;
    for (uint64_t w = 256; whole > 0; w *= 2) {
        const uint32_t words = w < whole ? (uint32_t)w : whole;
        const uint32_t n = count_le(list, len, words * 32u - 1u);
        const int64_t gn = (int64_t)kDenseWords * n - words;
        if (gn > gain) {
            gain = gn;
            best = make_uint2(words, n);
        }
        if (w >= whole) break;
    }
    pre[r] = best;
}

hipError_t build_rows(const DevGraph& g, const uint32_t* row_node, uint32_t n_out_rows, uint32_t n_rows,
                      uint32_t* rows, uint2* row_pre, hipStream_t stream) {
    if (n_rows == 0) return hipSuccess;
    uint32_t blocks = n_rows < 65535u ? n_rows : 65535u;
    hipLaunchKernelGGL(rows_kernel, dim3(blocks), dim3(256), 0, stream, g, row_node, n_out_rows, n_rows, rows);
    hipLaunchKernelGGL(row_pre_kernel, dim3((n_rows + 255) / 256), dim3(256), 0, stream, g, row_node, n_out_rows,
                       n_rows, row_pre);
    return hipGetLastError();
}

hipError_t launch_count(const InitArgs* inits, int n_inits, const KArgs& a, uint32_t n_blocks,
                        hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop) {
    for (int i = 0; i < n_inits; i++) {
        hipLaunchKernelGGL(init_kernel, dim3(64), dim3(256), 0, stream, inits[i]);
    }
    uint32_t nsrc = a.roots ? a.n_src : a.n_hubs;
    uint64_t total = (uint64_t)nsrc * a.n_plans;
    uint32_t sb = (uint32_t)((total + 255) / 256);
    sb = sb < 1 ? 1 : (sb > 4096 ? 4096 : sb);
    hipLaunchKernelGGL(split_kernel, dim3(sb), dim3(256), 0, stream, a);
    size_t lds = (size_t)a.lds_words * 4 * kWavesPerBlock;
    if (ev_start) {
        hipError_t e = hipEventRecord(ev_start, stream);
        if (e != hipSuccess) return e;
    }
    // the whole kernel in registers when the launch asks for few enough waves
    // (listing and merging are in that kernel only)
    const bool roomy = n_blocks <= (uint64_t)a.n_cu * kRoomyBlocksPerCu || a.list || a.merge_min != 0xFFFFFFFFu;
    if (a.nonlinear && roomy)
        hipLaunchKernelGGL((count_kernel<true, kRoomyBlocksPerCu>), dim3(n_blocks), dim3(kBlockThreads), lds, stream, a);
    else if (a.nonlinear)
        hipLaunchKernelGGL((count_kernel<true, kFullBlocksPerCu>), dim3(n_blocks), dim3(kBlockThreads), lds, stream, a);
    else if (roomy)
        hipLaunchKernelGGL((count_kernel<false, kRoomyBlocksPerCu>), dim3(n_blocks), dim3(kBlockThreads), lds, stream, a);
    else
        hipLaunchKernelGGL((count_kernel<false, kFullBlocksPerCu>), dim3(n_blocks), dim3(kBlockThreads), lds, stream, a);
    if (ev_stop) {
        hipError_t e = hipEventRecord(ev_stop, stream);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(finalize_kernel, dim3(1), dim3(256), 0, stream, a);
    return hipGetLastError();
}

}  // namespace xm
