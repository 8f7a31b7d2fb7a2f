// The group-wise tree traversal shared by the force walk and its adjoint
// (Sec. III.A: one walk per group of targets; Sec. I.A: a cell is used whole
// when it passes the opening test with angle theta, otherwise it is opened).
//
// One 64-lane wavefront walks the tree for one target group:
//   * a stack of sibling ranges (first << 3 | count - 1); each pass pops up
//     to 128 cells, two per lane, from the top 64 ranges.  Children of
//     opened cells are pushed with shallower ranges below deeper ones, so
//     the stack holds at most 128 ranges per level (kStackMax).  Its top
//     entries live in an LDS ring of kRing entries, of which at most `ring`
//     (256, or 192 to exercise the spill path) are resident; the rest spill
//     to a per-wave area in device memory in blocks of 64 (a spill happens
//     only when a push would exceed `ring` resident entries, a refill only
//     when fewer than 64 are resident);
//   * each lane applies the opening test: distance d from the cell's centre
//     of mass to the group's box, accept the cell whole iff
//     d^2 >= (l / theta + delta)^2 (FP32, no contraction);
//   * accepted cells and the particles of opened leaves are compacted
//     (ballot + mbcnt) into two LDS index lists; no source data is read
//     during the traversal.  The caller's flush functions evaluate a list
//     when it fills, and once more at the end.
// Groups are taken from eight contiguous ranges (one per XCD, blockIdx % 8),
// so neighbouring groups share an L2; every wave leaves once all ranges are
// exhausted.
#pragma once

#include "bh_internal.h"
#include "wave.h"

namespace bh {

constexpr int kRing = 256;   // LDS window of the range stack (TreeView::ring <= kRing)
constexpr int kPcCap = 752;  // particle-cell index list
constexpr int kPcFlush = kPcCap - 128;  // a pass appends at most 128 cells
constexpr int kPpCap = 512;  // particle-particle index list
constexpr int kChunk = 64;   // sources staged per evaluation round
constexpr uint32_t kDealRanges = 96;  // stack ranges at which the waves of a split walk part

struct TravLds {
    uint32_t ring[kRing];
    uint32_t pcidx[kPcCap];
    uint32_t ppidx[kPpCap];
    uint32_t leaf[128];   // opened leaves: first particle less list position
    uint8_t starts[128];  // 1 where a popped range (an opened leaf's particles) begins
};

struct TreeView {
    const float4 *wA;   // com, r_open^2
    const uint2 *wN;    // (first, n | leaf bit)
    uint32_t ring;      // resident stack entries allowed: kRing, or 192 to exercise the spill path
    uint32_t *status;
    uint32_t *opened = nullptr;  // kLeafCells: opened internal cells are marked here
    // level starts and parents of the cells (null: not known, the walk starts at the root)
    const uint32_t *ls = nullptr, *parent = nullptr;
};

struct GroupBox {
    float cx, cy, cz, hx, hy, hz;
};

// Tight FP32 box of the gn targets (lane < gn holds one): centre (min+max)/2,
// half size (max-min)/2.
__device__ __forceinline__ GroupBox group_box(const float4 &me, bool own) {
    GroupBox b;
    float mn = wave_min(own ? me.x : INFINITY), mx = wave_max(own ? me.x : -INFINITY);
    b.cx = (mn + mx) * 0.5f; b.hx = (mx - mn) * 0.5f;
    mn = wave_min(own ? me.y : INFINITY); mx = wave_max(own ? me.y : -INFINITY);
    b.cy = (mn + mx) * 0.5f; b.hy = (mx - mn) * 0.5f;
    mn = wave_min(own ? me.z : INFINITY); mx = wave_max(own ? me.z : -INFINITY);
    b.cz = (mn + mx) * 0.5f; b.hz = (mx - mn) * 0.5f;
    return b;
}

// Split the group's gn targets over the 64 lanes: one phase with
// r = floor(64 / gn) slices, or two phases (Ta targets with ceil(64 / gn)
// slices, the remaining Tb with floor(64 / Tb)) when that needs fewer rounds.
__device__ __forceinline__ void plan_phases(uint32_t gn, uint32_t &T1, uint32_t &r1,
                                            uint32_t &T2, uint32_t &r2) {
    auto div = [](uint32_t a, uint32_t b) { return uniform(small_div(a, b)); };
    const uint32_t rs = div(64u, gn);
    const uint32_t cost1 = div(63u + rs, rs);
    const uint32_t ra = div(63u + gn, gn), Ta = div(64u, ra), Tb = gn - Ta;
    const uint32_t rb = Tb ? div(64u, Tb) : 0u;
    const uint32_t cost2 = div(63u + ra, ra) + (Tb ? div(63u + rb, rb) : 0u);
    if (Tb && cost2 < cost1) {
        T1 = Ta; r1 = ra; T2 = Tb; r2 = rb;
    } else {
        T1 = gn; r1 = rs; T2 = 0; r2 = 0;
    }
}

// Squared distance from a cell's centre of mass to the group's box (FP32,
// no contraction): the left side of the opening test.
__device__ __forceinline__ float box_d2(const float4 &A, const GroupBox &b) {
    const float dxm = fmaxf(fabsf(A.x - b.cx) - b.hx, 0.f);
    const float dym = fmaxf(fabsf(A.y - b.cy) - b.hy, 0.f);
    const float dzm = fmaxf(fabsf(A.z - b.cz) - b.hz, 0.f);
    float d2 = dxm * dxm + dym * dym;
    d2 = d2 + dzm * dzm;
    return d2;
}

// One of the 2^logw waves that walk the tree for one group.
struct Share {
    uint32_t w, logw;
};

// Split the waves' common entries: of the set flags of a (slot a of every
// lane, then b) entry k goes to wave (dealt + k) mod 2^logw.
__device__ __forceinline__ void deal(bool &a, bool &b, const Share &sh, uint32_t &dealt) {
    const uint64_t ma = ballot(a), mb = ballot(b);
    const uint32_t na = (uint32_t)__popcll(ma), wmask = (1u << sh.logw) - 1u;
    a &= ((dealt + count_below(ma)) & wmask) == sh.w;
    b &= ((dealt + na + count_below(mb)) & wmask) == sh.w;
    dealt += na + (uint32_t)__popcll(mb);
}

// A leaf of more than a chunk of particles (coincident ones: others hold at
// most 64) is not dealt to one wave: each takes its share of the particles, at
// least four.  Dealt whole it made one wave of every group do all the work of
// a coincident set, and those waves all in the same quarter of the CUs: force
// of 50000 coincident particles 4.69 ms (in shares 1.37; one wave per group
// 3.29), adjoint of 20000 9.73 (1.32; 6.41).
constexpr uint32_t kBigLeaf = kLeafBit | (uint32_t)kChunk;
__device__ __forceinline__ bool share_leaf(uint2 &N, const Share &sh) {
    const uint32_t c = N.y & ~kLeafBit, q = c >> sh.logw, r = c & ((1u << sh.logw) - 1u);
    N.x += q * sh.w + min(sh.w, r);
    N.y = (q + (sh.w < r ? 1u : 0u)) | kLeafBit;
    return true;
}

// Walk the tree for one group.  flush_pc(n) / flush_pp(n) evaluate the first
// n entries of L.pcidx / L.ppidx (called with n > 0, all lanes, after a
// barrier); both lists are empty when traverse returns.  Counts: accepted
// cells and particles of opened leaves.  kLeafCells: L.ppidx lists the
// opened leaf cells themselves instead of their particles (and the second
// count is of those leaves), and opened internal cells are marked in tv.opened.
//
// A pass pops up to 128 cells from the top 64 ranges: lane l takes cells l
// (slot a) and 64 + l (slot b) of their concatenation, so the pop, the scan
// and the barriers are shared by two opening tests and two cell loads are in
// flight per lane.  Pop order is slot a's cells, then slot b's; every list
// and the pushed children keep that order.
//
// A pass is a chain of some 350 instructions, an LDS scan and one round of
// loads (2000 to 4500 cycles, the most of a small set's walk), so it is written
// without branches around loads and tests, and an opened leaf's particles are
// listed by marks and a popcount.  Against branches, and a binary search per
// listed particle: 1000 particles 34.6 -> 32.8 us (walk), 65536 481 -> 449,
// 1M 4.57 -> 4.47 ms, 13M 56.9 -> 56.1.
//
// kSplit: 2^logw waves walk the tree for the same group, each calling
// traverse with its own share.  They run the same passes until the stack
// holds kDealRanges ranges, the accepted cells and opened leaves of those
// passes dealt out in list order (big leaves shared); then wave w keeps every 2^logw-th range and
// walks those subtrees alone.  Which wave takes what depends only on the tree
// and the group, so the sums do not depend on scheduling.  The more ranges are
// dealt out, the more alike the shares: 96 against 64 (that is all the smaller
// ring allows), walk in us: 16384 149 -> 144, 40000 228 -> 209, 65536 448 -> 393;
// 128 no better.
//
// kTop: where the level starts are known, the first pass takes all cells of
// the levels 0 to 2 (at most 73, each with its parent) instead of three passes
// of 1, 8 and 64: 1000 32.5 -> 31.2 us, 4099 61.7 -> 60.2.
template <bool kLeafCells = false, bool kSplit = false, bool kTop = false, class FlushPc,
          class FlushPp>
__device__ __forceinline__ void traverse(const TreeView &tv, const GroupBox &b, uint32_t lane,
                                         TravLds &L, uint32_t *spill, uint32_t &cnt_pc,
                                         uint32_t &cnt_pp, FlushPc &&flush_pc,
                                         FlushPp &&flush_pp,
                                         const Share sh = Share{0u, 0u}) {
    constexpr uint32_t rmask = (uint32_t)kRing - 1u;
    uint32_t pc_n = 0, pp_n = 0;
    uint32_t sp = 1, lo = 0;  // stack positions [lo, sp) are in the LDS ring
    cnt_pc = 0;
    cnt_pp = 0;
    bool common = kSplit;          // the waves still walk the same cells
    const uint32_t deal_at = min(kDealRanges, tv.ring - 128u);
    uint32_t dealt_pc = 0, dealt_pp = 0;  // entries dealt out so far
    bool top = kTop && tv.ls != nullptr;
    const uint32_t top_n = top ? uniform(tv.ls[3]) : 0u, top_push = top ? uniform(tv.ls[2]) : 0u;
    if (lane == 0) L.ring[0] = 0u;  // the root: first cell 0, one cell
    wave_sync();

    while (sp > 0) {
        uint32_t cell_a, cell_b, sp_new;
        bool have_a, have_b;
        uint32_t up_a = 0u, up_b = 0u;  // top: the cells' parents
        if (kTop && top) {
            have_a = lane < top_n;
            have_b = 64u + lane < top_n;
            cell_a = have_a ? lane : 0u;
            cell_b = have_b ? 64u + lane : 0u;
            up_a = tv.parent[cell_a];
            up_b = tv.parent[cell_b];
            sp_new = 0u;
        } else {
            // ---- refill the ring from the spill area when the top range is not resident
            const uint32_t avail = sp < 64u ? sp : 64u;
            if (sp - avail < lo) {
                lo -= 64u;
                L.ring[(lo + lane) & rmask] = spill[lo + lane];
                wave_sync();
            }
            // ---- pop up to 128 cells from the top ranges (range lane = stack top - lane)
            const uint32_t e = L.ring[(sp - 1 - lane) & rmask];
            const uint32_t ne = lane < avail ? (e & 7u) + 1u : 0u;
            const uint32_t incl = wave_incl_scan(ne, lane);
            const uint32_t excl = incl - ne;
            const uint32_t nfull = (uint32_t)__popcll(ballot(lane < avail && incl <= 128u));
            const uint32_t tall = read_lane(incl, avail - 1u);
            const uint32_t total = tall < 128u ? tall : 128u;
            L.starts[lane] = 0u;
            L.starts[64u + lane] = 0u;
            wave_sync();
            if (lane < avail && excl < 128u) L.starts[excl] = 1u;
            wave_sync();
            const uint64_t sa = ballot(L.starts[lane] != 0u);
            const uint64_t sb = ballot(L.starts[64u + lane] != 0u);
            // range of each slot's cell (cell 0 starts range 0: both indices are in 0..63)
            const uint32_t ja = (uint32_t)__popcll(sa & mask_le(lane)) - 1u;
            const uint32_t jb =
                (uint32_t)__popcll(sa) + (uint32_t)__popcll(sb & mask_le(lane)) - 1u;
            const uint32_t c0 = (e >> 3) - excl;  // a range's first cell less its slot
            const uint32_t ra = shfl(c0, ja), rb = shfl(c0, jb);
            have_a = lane < total;
            have_b = 64u + lane < total;
            cell_a = have_a ? ra + lane : 0u;
            cell_b = have_b ? rb + 64u + lane : 0u;
            sp_new = sp - nfull;
            if (nfull < avail && lane == nfull && excl < 128u) {
                const uint32_t taken = 128u - excl;  // the rest of this range stays on top
                L.ring[(sp_new - 1) & rmask] = (((e >> 3) + taken) << 3) | (ne - taken - 1u);
            }
        }

        // ---- opening test (idle slots read cell 0: all four loads are in flight
        // together, where branches around them made each wait for the last)
        uint2 Na = tv.wN[cell_a], Nb = tv.wN[cell_b];
        const float4 Aa = tv.wA[cell_a], Ab = tv.wA[cell_b];
        const bool far_a = box_d2(Aa, b) >= Aa.w, far_b = box_d2(Ab, b) >= Ab.w;
        const bool cut_a = (Na.y & kLeafBit) != 0u, cut_b = (Nb.y & kLeafBit) != 0u;
        bool push_a = true, push_b = true;
        if (kTop && top) {  // reached: the parent and its parent opened; pushed: the last level
            L.starts[lane] = (uint8_t)(!far_a & !cut_a);
            L.starts[64u + lane] = (uint8_t)(!far_b & !cut_b);
            wave_sync();
            const uint32_t root = L.starts[0];
            const bool in_a = L.starts[up_a & 127u] != 0u, in_b = L.starts[up_b & 127u] != 0u;
            wave_sync();
            have_a &= lane == 0u || (root != 0u && in_a);
            have_b &= root != 0u && in_b;
            push_a = cell_a >= top_push;
            push_b = cell_b >= top_push;
            top = false;
        }
        bool acc_a = have_a & far_a, acc_b = have_b & far_b;
        bool leaf_a = have_a & !far_a & cut_a, leaf_b = have_b & !far_b & cut_b;
        const bool open_a = have_a & !far_a & !cut_a & push_a;
        const bool open_b = have_b & !far_b & !cut_b & push_b;

        if (kSplit && common) {  // this wave's share of the entries, in list order
            deal(acc_a, acc_b, sh, dealt_pc);
            const bool all_a = leaf_a, all_b = leaf_b;
            deal(leaf_a, leaf_b, sh, dealt_pp);
            if (ballot(max(Na.y, Nb.y) > kBigLeaf) != 0ull) {
                if (all_a & (Na.y > kBigLeaf)) leaf_a = share_leaf(Na, sh);
                if (all_b & (Nb.y > kBigLeaf)) leaf_b = share_leaf(Nb, sh);
            }
        }

        // ---- accepted cells -> particle-cell index list
        const uint64_t ama = ballot(acc_a), amb = ballot(acc_b);
        const uint32_t na = (uint32_t)__popcll(ama);
        if (acc_a) L.pcidx[pc_n + count_below(ama)] = cell_a;
        if (acc_b) L.pcidx[pc_n + na + count_below(amb)] = cell_b;
        const uint32_t nacc = na + (uint32_t)__popcll(amb);
        pc_n += nacc;
        cnt_pc += nacc;

        // ---- opened internal cells -> their children ranges; the first popped
        // cell's children end on top, so deeper ranges stay above shallower ones
        const uint64_t oma = ballot(open_a), omb = ballot(open_b);
        const uint32_t nob = (uint32_t)__popcll(omb);
        const uint32_t npush = (uint32_t)__popcll(oma) + nob;
        const uint32_t last = sp_new + npush - 1u;  // the new top of the stack
        if (sp_new + npush > (uint32_t)kStackMax) {  // cannot happen: 128 ranges per level
            if (lane == 0) atomicOr(tv.status, kStOverflow);
            break;
        }
        while (sp_new + npush > lo + tv.ring) {
            // spill the 64 lowest resident entries (all below sp_new when ring >= 192)
            wave_sync();
            spill[lo + lane] = L.ring[(lo + lane) & rmask];
            lo += 64u;
            wave_sync();
        }
        if constexpr (kLeafCells) {
            if (open_a) tv.opened[cell_a] = 1u;
            if (open_b) tv.opened[cell_b] = 1u;
        }
        if (open_a) {
            L.ring[(last - count_below(oma)) & rmask] = (Na.x << 3) | (Na.y - 1u);
        }
        if (open_b) {
            L.ring[(sp_new + nob - 1u - count_below(omb)) & rmask] = (Nb.x << 3) | (Nb.y - 1u);
        }
        sp = sp_new + npush;
        if (kSplit && common && sp >= deal_at) {  // (at most tv.ring - 1 ranges, none spilled)
            wave_sync();
            const uint32_t j0 = sh.w + (lane << sh.logw), j1 = sh.w + ((64u + lane) << sh.logw);
            const uint32_t e0 = j0 < sp ? L.ring[j0] : 0u;
            const uint32_t e1 = j1 < sp ? L.ring[j1 & rmask] : 0u;
            wave_sync();
            L.ring[lane] = e0;
            if (j1 < sp) L.ring[64u + lane] = e1;
            sp = (sp - sh.w + (1u << sh.logw) - 1u) >> sh.logw;
            common = false;
        }

        // ---- opened leaves -> their cells (kLeafCells)
        if constexpr (kLeafCells) {
            if (pp_n + 128u > (uint32_t)kPpCap) {
                wave_sync();
                flush_pp(pp_n);
                pp_n = 0;
            }
            const uint64_t la = ballot(leaf_a), lb = ballot(leaf_b);
            const uint32_t nla = (uint32_t)__popcll(la);
            if (leaf_a) L.ppidx[pp_n + count_below(la)] = cell_a;
            if (leaf_b) L.ppidx[pp_n + nla + count_below(lb)] = cell_b;
            const uint32_t nl = nla + (uint32_t)__popcll(lb);
            pp_n += nl;
            cnt_pp += nl;
        }
        // ---- particles of opened leaves -> particle-particle index list, 64
        // entries at a time: the leaves that begin among them are marked, and an
        // entry's leaf is the last to begin at or before it (leaves in the order
        // of lanes, slot a first).  A leaf without particles is left out: it would
        // begin where the next one does.  Only a local essential tree has them
        // (cells its boxes accept, kept without what is below); a paired target
        // set, whose box reaches over two terminal cells, opens them.
        const bool pa = !kLeafCells & leaf_a & (Na.y != kLeafBit);
        const bool pb = !kLeafCells & leaf_b & (Nb.y != kLeafBit);
        const uint64_t la = ballot(pa), lb = ballot(pb);
        if ((la | lb) != 0ull) {
            const uint32_t ca = pa ? (Na.y & ~kLeafBit) : 0u;
            const uint32_t lc = ca + (pb ? (Nb.y & ~kLeafBit) : 0u);
            const uint32_t lincl = wave_incl_scan(lc, lane);
            const uint32_t np = read_lane(lincl, 63u);
            const uint32_t oa = lincl - lc, ob = oa + ca;
            const uint32_t k = count_below(la) + count_below(lb);
            if (pa) L.leaf[k] = Na.x - oa;
            if (pb) L.leaf[k + (pa ? 1u : 0u)] = Nb.x - ob;
            cnt_pp += np;
            uint32_t begun = 0;  // leaves that begin before entry `base`
            for (uint32_t base = 0; base < np;) {
                if (pp_n == (uint32_t)kPpCap) {
                    wave_sync();
                    flush_pp(pp_n);
                    pp_n = 0;
                }
                const uint32_t room = min((uint32_t)kPpCap - pp_n, 64u);
                const uint32_t take = min(room, np - base);
                L.starts[lane] = 0u;
                wave_sync();
                if (pa & (oa - base < take)) L.starts[oa - base] = 1u;
                if (pb & (ob - base < take)) L.starts[ob - base] = 1u;
                wave_sync();
                const uint64_t m = ballot(L.starts[lane] != 0u);
                const uint32_t s = begun + (uint32_t)__popcll(m & mask_le(lane)) - 1u;
                if (lane < take) L.ppidx[pp_n + lane] = L.leaf[s] + base + lane;
                begun += (uint32_t)__popcll(m);
                pp_n += take;
                base += take;
                wave_sync();
            }
        }
        wave_sync();
        if (pc_n > (uint32_t)kPcFlush) {
            flush_pc(pc_n);
            pc_n = 0;
        }
    }
    wave_sync();
    if (pc_n) flush_pc(pc_n);
    if (pp_n) flush_pp(pp_n);
    wave_sync();
}

// Persistent group loop: tasks (group, wave of the group) in eight contiguous
// ranges of groups, one per XCD (blockIdx % 8); fn(g, w) handles group g as
// wave w of 2^logw (waves of one group do not wait for each other).  A
// block's first task is its place among the blocks of its range, the next
// ones come from the range's counter; a block whose range is exhausted reads
// all eight counters at once and goes on with a range that has tasks left, so
// a launch of more blocks than tasks touches no counter but by that one load.
// Each counter has a cache line of its own: eight in one line, each block
// adding to all of them before it left, kept a grid of 4096 waves at 0.3 ms
// however few the groups.
template <class Fn>
__device__ __forceinline__ void for_each_group(uint32_t ng, uint32_t *work, uint32_t lane,
                                               uint32_t logw, Fn &&fn) {
    const uint32_t q = lane & 7u;  // lane's range, for the look at all of them
    const uint32_t qn = (uint32_t)((((uint64_t)ng * (q + 1)) >> 3) - (((uint64_t)ng * q) >> 3))
                        << logw;
    const uint32_t qb = (gridDim.x + 7u - q) >> 3;  // blocks that start in it
    uint32_t part = blockIdx.x & 7u, t = blockIdx.x >> 3;
    for (;;) {
        const uint32_t r0 = (uint32_t)(((uint64_t)ng * part) >> 3);
        const uint32_t size = read_lane(qn, part), given = read_lane(qb, part);
        while (t < size) {
            fn(r0 + (t >> logw), t & ((1u << logw) - 1u));
            if (lane == 0) t = given + atomicAdd(&work[part * kWorkStride], 1u);
            t = uniform(t);
        }
        const uint32_t seen = __hip_atomic_load(&work[q * kWorkStride], __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t left = (uint32_t)ballot(lane < 8u && qb + seen < qn);
        if (left == 0u) return;
        const uint32_t turn = ((left | (left << 8)) >> part) & 0xffu;  // ranges from part on
        part = (part + (uint32_t)__builtin_ctz(turn)) & 7u;
        const uint32_t first = read_lane(qb, part);
        if (lane == 0) t = first + atomicAdd(&work[part * kWorkStride], 1u);
        t = uniform(t);
    }
}

}  // namespace bh
