// Internal declarations of the gfx950 tree-code library: the context that
// owns every device buffer, and the host-side launchers each .hip file
// provides.  Every kernel is enqueued on the caller's stream; nothing here
// synchronises except where a launcher says so.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

#include "bh.h"

namespace bh {

constexpr int kKeyBits = 21;            // bits per axis of a Morton key
constexpr int kLevels = 22;             // levels 0..21
constexpr int kLsSize = 24;             // level_start entries (23 used)
constexpr int kGrid = 1024;             // grid of the strided kernels over the cells (boxes, flags, radii, centres)
constexpr int kTreeTile = 1024;         // particles per block of the octree build
constexpr uint32_t kScanTiles = 64;  // tiles whose counts every block of k_tree_write adds up
constexpr int kSpanTiles = 128;         // tiles per block of the moment pass over tile ends
constexpr uint32_t kLeafBit = 0x80000000u;
constexpr uint32_t kNone = 0xffffffffu;
constexpr int kWorkStride = 32;         // a cache line per work counter of the walk
constexpr int kStackMax = 2689;         // walk stack bound: 21 levels x 128 ranges + root
// Adjoint: the cells of the top levels (the first kHotCells in level order) are hit by far
// more groups than the rest, so their accumulators come in kHotCopies copies (4 per XCD).
// A copy's stride (in doubles) is one 128-byte line more than a multiple of a
// power of two, so that a cell's copies fall on different L2 channels.
constexpr uint32_t kHotCells = 65536;
constexpr uint32_t kHotCopies = 32;
constexpr uint64_t kHotCopy = 10ull * kHotCells + 16;
constexpr int kDiagN = 9;               // diagnostics: M, KE, PE, p xyz, L xyz
constexpr int kDiagBlocks = 1024;       // blocks of the diagnostics reduction

// device status word bits
constexpr uint32_t kStNonFinite = 1u;
constexpr uint32_t kStMass = 2u;
constexpr uint32_t kStOverflow = 4u;
constexpr uint32_t kStIndex = 8u;       // a target index outside [0, n)
constexpr uint32_t kStOutside = 16u;    // a particle outside the caller-given key box

// Particle state in sorted (Morton) order, structure of arrays.
struct State {
    float *x, *y, *z, *m, *vx, *vy, *vz;
    uint32_t *cid;  // caller index of each sorted slot
    double *x64, *y64, *z64;  // FP64 master positions (pos_fp64 contexts), else null
};

// Particles to be sorted, read in place: the context's own state, the caller's
// arrays (positions and velocities [n][3]) or a snapshot.
struct Source {
    const float *x = nullptr, *y = nullptr, *z = nullptr;     // every ps-th value
    const float *vx = nullptr, *vy = nullptr, *vz = nullptr;  // every vs-th; null: zero
    const float *m = nullptr;
    uint32_t ps = 1, vs = 1;
    const uint32_t *cid = nullptr;  // null: the index
    const double *x64 = nullptr, *y64 = nullptr, *z64 = nullptr;  // null: the FP32 positions
    bool check = false;  // latch bad masses and velocities (the caller's data)
};
inline Source source_of(const State &s) {
    Source r;
    r.x = s.x; r.y = s.y; r.z = s.z; r.m = s.m;
    r.vx = s.vx; r.vy = s.vy; r.vz = s.vz;
    r.cid = s.cid;
    r.x64 = s.x64; r.y64 = s.y64; r.z64 = s.z64;
    return r;
}

// Octree cells, breadth-first order (level, then key).
struct Cells {
    uint64_t *prefix;  // key >> 3 (21 - level)
    uint32_t *level, *begin, *count, *child0, *nchild, *parent;
    uint32_t *ls;      // [kLsSize] level_start on the device
    uint16_t *lev;     // [n_max] levels of the cells that start at / hold each particle
    uint32_t *tcnt;    // [kLevels + 1][tiles] cells of each level (and groups) starting before a tile
    uint32_t *ttot;    // [kLevels + 1] their totals; then, for at most kScanTiles tiles, those counts
                       // (tcnt holds each tile's own)
    // FP64 moments of the upward pass
    double *M, *S, *com, *Q;  // [c], [c][3], [c][3], [c][6]; com = S / M, filled for export
    // records read by the walk
    float4 *wA;  // com (FP32) and r_open^2 of the last theta
    uint2 *wN;   // internal: (child0, nchild); leaf: (begin, count | kLeafBit)
    float4 *P0;  // particle-cell record: com x, y, z, M
    float4 *P1;  // -3 Qxx, -3 Qyy, -3 Qzz, -3 Qxy
    float4 *P2;  // -3 Qxz, -3 Qyz, trace(Q) / 2, -3 trace(Q) / 2
    float2 *size;  // cell size l, |com - geometric centre|
};

struct Groups {
    uint32_t *flag, *scan;  // [n] first groups of paired target sets and their exclusive scan
    uint32_t *begin;        // [n + 1]
    uint32_t *count_dev;    // [1] number of groups
    float4 *box;            // [2 * n] centre, half size
    uint32_t *npp, *npc;    // [n]
};

// Boundary tree of a domain (Sec. III.B.2): the cells reached from the root
// through cells of more than ncrit particles, down to level `level`;
// terminal cells (level `level`, at most ncrit particles, or leaves) cover
// every particle once.
struct Boundary {
    bool valid = false;
    int level = -1;
    uint32_t nterm = 0;
    uint32_t ncell = 0;        // cells of the tree
    float margin = 0.f;        // widening of the terminal boxes
    uint32_t *flag = nullptr;  // [cap_cells + 1] bit 0: in the boundary tree, bit 1: terminal
    uint32_t *scan = nullptr;  // [cap_cells + 1] exclusive scan of the terminal bits
    uint32_t *ids = nullptr;   // [cap_cells] terminal cells in cell order
    float4 *box = nullptr;     // [2 cap_cells] centre, half size (widened) of each
    float4 *cmin = nullptr, *cmax = nullptr;  // [cap_cells] FP32 particle box of every cell
    uint32_t *lvl = nullptr;   // [kLevels] boundary cells per level
    uint32_t *part = nullptr;  // scan partials
};

// Local essential trees of remote domains merged under virtual cells
// (Sec. III.B.2), plus the scratch of their construction.
struct Let {
    bool valid = false;
    float theta = 0.f;
    int nsrc = 0;
    uint32_t ncell = 0, npart = 0;
    int64_t cell_cap = 0, part_cap = 0;
    float4 *wA = nullptr, *P0 = nullptr, *P1 = nullptr, *P2 = nullptr, *xyzm = nullptr;
    uint2 *wN = nullptr;
    uint32_t *origin = nullptr;  // [cell_cap][2] (source, source cell); kNone for virtual
    // scratch of the construction, over all sources one after another: per cell
    // accepted and opened marks, per particle marks, per source a word (zeroed
    // together), then kept cells and particles and their exclusive scan
    uint32_t *marks = nullptr, *keep = nullptr, *spart = nullptr, *info = nullptr;
    int64_t marks_cap = 0, keep_cap = 0, spart_cap = 0, info_cap = 0;
};

// Device buffers of the domain cut: group-start costs and the cuts.
struct Cut {
    uint64_t *S = nullptr;  // [n + 1]
    int64_t *cuts = nullptr;  // [p + 1]
    int64_t S_cap = 0, cuts_cap = 0;
};

struct Sort {
    uint64_t *key[2];
    uint32_t *idx[2];
    uint32_t *counts;      // [256 * tiles]
    uint32_t *scan_part;   // partials of the generic scan
    int64_t counts_len, scan_part_len;
};

}  // namespace bh

struct bh_ctx {
    int64_t nmax = 0, cap_cells = 0, n = 0;
    bh_params p{};
    int device = 0;
    int cus = 0;

    bh::State st[2]{};
    int cur = 0;
    float4 *acc = nullptr;  // sorted acceleration + potential
    float4 *xyzm = nullptr; // sorted position + mass, one record per particle
    float4 *pacc = nullptr;     // split walks: partial sums, one row of n per wave of a group
    uint2 *pcnt = nullptr;      // their interaction counts per group
    uint32_t *spill = nullptr;  // walk stack spill area, kStackMax per wave
    float *box = nullptr;   // [8]: lo xyz, side, scale
    float *box_part = nullptr;
    uint32_t *status = nullptr;
    bool clear_status = false;  // a build starts with clear status words (tree_force_static)
    uint32_t *work = nullptr;                // [2][8][kWorkStride] walk work counters, one per line
    unsigned long long *totals = nullptr;    // [4] n_pp, n_pc, leaves
    bh::Sort sort{};
    bh::Cells cells{};
    bh::Groups groups{};

    // adjoint buffers (contexts created with adjoint = 1)
    // per-XCD copies (8): [8][cap_cells][10] dL/dM, dL/dcom xyz, dL/dQ xx yy zz xy xz yz;
    // [8][n_max][4] dL/dx xyz, dL/dm of sorted particles; the first kHotCells cells
    // accumulate in kHotCopies copies of kHotCopy doubles instead
    double *lcell = nullptr;
    double *gsrc = nullptr;
    double *lhot = nullptr;
    float4 *usort = nullptr;   // [n] cotangent of the accelerations, sorted order
    uint32_t *leafof = nullptr;  // [n] leaf cell of each sorted particle
    double *cic = nullptr;       // [65536] accumulator of the surface-density grid
    uint32_t *inv = nullptr;     // [n] sorted slot of each caller index (direct sum)
    double *diag = nullptr;      // [kDiagBlocks + 1][kDiagN] diagnostics partials, result
    uint8_t *seg = nullptr;      // recomputed states of an adjoint segment (grown on demand)
    int64_t seg_cap = 0;         // bytes of seg

    bh::Boundary bnd{};
    bh::Let let{};
    bh::Cut cut{};

    bool built = false, have_acc = false;
    bool counts_valid = false;  // npp / npc / totals describe a walk of the current groups
    bool fixed_box = false;     // keys relative to a caller-given box (bh_set_box)
    float box_lo[3] = {0.f, 0.f, 0.f}, box_side = 1.f;
    float acc_theta = 0.f, acc_eps = 0.f;
    int walk_grid = 0;
    bool walk_small_stack = false;  // test hook: at most 192 resident stack entries
    uint32_t pair_groups = 0;       // sibling groups of together <= this many walk as one (0: off)

    // events: build start, after sort, after octree+groups, after moments,
    // walk start, walk end, step start, step end, adjoint walk start, end
    hipEvent_t ev[10]{};
    bool ev_rec[10]{};
    std::string last_error;
};

namespace bh {

// walk_vjp.hip: coef * u^T d(acc)/d(x, m) accumulated into caller-order
// g_pos [n][3] / g_mass [n] (either may be null); u is caller order [n][3]
void launch_walk_vjp(bh_ctx *c, float theta, float eps, const float *u, float coef, float *g_pos,
                     float *g_mass, hipStream_t st);
void launch_axpy3(const float *x, float *y, float a, uint32_t n, hipStream_t st);

// loss.hip: cloud-in-cell surface density on a polar grid and its adjoint
void launch_cic(const float *pos, const float *mass, const uint8_t *sel, uint32_t n, float rmin,
                float rmax, int nr, int nphi, double *scratch, float *density, hipStream_t st);
void launch_cic_vjp(const float *pos, const float *mass, const uint8_t *sel, uint32_t n,
                    float rmin, float rmax, int nr, int nphi, const float *gden, float *g_pos,
                    float *g_mass, hipStream_t st);

// direct.hip: FP64 direct sum at caller-index targets tgt [nt] (device)
// into acc [nt][3] / pot [nt] (device, FP64)
// (targets outside [0, n) are skipped and latch kStIndex)
void launch_direct(bh_ctx *c, const int64_t *tgt, uint32_t nt, float eps, double *acc,
                   double *pot, hipStream_t st);

// keys_sort.hip
// bounding box (-> box), keys of s, their sort (-> key[0]), and the particles
// in that order (-> st[cur ^ 1], xyzm; cur is flipped)
void launch_sort(bh_ctx *c, const Source &s, uint32_t n, hipStream_t st);
int64_t sort_counts_len(int64_t nmax);
int64_t scan_part_len(int64_t n);

// scan.hip: exclusive scan of n u32 (in may equal out); part >= scan_part_len(n)
void launch_exclusive_scan(const uint32_t *in, uint32_t *out, uint32_t n, uint32_t *part,
                           hipStream_t st);

// build.hip
void launch_build(bh_ctx *c, uint32_t n, hipStream_t st);  // cells and groups

// moments.hip
// Squared opening radius (fl32(l / theta) + delta)^2 in FP32.
__device__ __forceinline__ float open_radius2(float2 size, float theta) {
    const float r = size.x / theta + size.y;
    return r * r;
}

// The walk's counters and totals, by one block.
__device__ __forceinline__ void zero_walk(uint32_t *work, unsigned long long *totals) {
    if (work && threadIdx.x < 16u) work[threadIdx.x * kWorkStride] = 0u;
    if (totals && threadIdx.x < 2u) totals[threadIdx.x] = 0ull;
}

// theta > 0: also what launch_walk_prep does for the context's own walk
void launch_moments(bh_ctx *c, uint32_t n, float theta, hipStream_t st);
void launch_com(bh_ctx *c, hipStream_t st);
// opening radii of c's cells for theta; also the work counters of walker (which
// is about to walk; null: none) to zero, and its interaction totals if totals
void launch_walk_prep(bh_ctx *c, float theta, bh_ctx *walker, bool totals, hipStream_t st);

// let.hip: boundary trees and local essential trees (Sec. III.B.2); nc is
// the cell count of the tree the launcher reads (cell_count)
void launch_bnd_flags(bh_ctx *c, hipStream_t st);                // -> bnd.flag bit 0, bnd.lvl
void launch_bnd_terminal(bh_ctx *c, int level, hipStream_t st);  // -> flag bit 1, scan input
void launch_bnd_boxes(bh_ctx *c, uint32_t nc, uint32_t nterm, hipStream_t st);  // -> ids, box
constexpr int kLetMaxSrc = 64;
// All of the LETs of tgt: opening radii of the sources for theta, marks, the
// kept cells and particles below the nv virtual cells (of the level sizes lv);
// then per source (boundary tree sufficed, cells, particles) and the totals of
// both to let.info [3 nsrc + 2].
void launch_let(bh_ctx *tgt, bh_ctx *const *srcs, int nsrc, float theta, const int64_t lv[4],
                int nlv, uint32_t nv, hipStream_t st);
uint32_t cell_count(const bh_ctx *c, hipStream_t st);  // synchronises st, reads the count

// walk.hip
// The cells and particles a walk reads: a context's own tree, another
// domain's tree, or a merged local essential tree.
struct SrcView {
    const float4 *wA;   // com, r_open^2 (prepared for the walk's theta)
    const uint2 *wN;    // internal: (child0, nchild); leaf: (first, count | kLeafBit)
    const float4 *P0, *P1, *P2;
    const float4 *xyzm;  // particles the leaves index
};
SrcView own_view(const bh_ctx *c);
// What becomes of the forces beside c->acc: written to caller-order outputs
// (row rows[i] of caller index i, or row i), and a kick v += a kick_h.
struct WalkOut {
    float *acc = nullptr, *pot = nullptr;
    const uint32_t *rows = nullptr;
    bool kick = false;
    float kick_h = 0.f;
    bool totals = true;  // sum up the interactions (the last walk of an evaluation)
};
// c's groups walk the tree v; remote: no self pairs (v is not c's own tree);
// accum: forces and counts add to c->acc, npp, npc.  The own tree's walk and a
// remote one have work counters of their own (both reset by launch_walk_prep).
void launch_walk_view(bh_ctx *c, const SrcView &v, float eps, bool remote, bool accum,
                      const WalkOut &out, hipStream_t st);
int walk_blocks_per_cu();
// Waves that share a group's walk: 2^logw for a group of more than t1 targets,
// half as many for one of more than t2, a quarter as many for a smaller one.
//
// A set of up to a million particles has few groups for each wave slot of the
// chip, and the longest walks set the time: those of the groups with the most
// targets (a wave evaluates its lists in about as many rounds as the group has
// targets; at 16384 the mean walk of a quarter of a group took 64 us, that of
// 54 to 64 targets 150 to 174).  Splitting costs throughput (every wave repeats
// the top of the walk, lists are shorter), so fewer waves share as the groups
// become more.  Walk in us, all groups alike (the best number of waves) / this
// rule, disk + halo at theta 0.4: n = 1000 31 / 32 (Plummer); 4099 74 / 63
// (Plummer); 16384 194 / 175; 40000 388 / 307; 65536 472 / 387; 131072 834 / 677;
// 1M 4637 / 4390 and 4768 with no split.  The lines, us by the rule below / above:
//   8192 (4 or 2 waves for groups of up to 16 targets), forces at theta 0.4, 0.6,
//   0.8: 4099 (Plummer) 71 / 76, 64 / 69, 61 / 62; 8192 111 / 118, 96 / 94, 88 / 84
//   (disk + halo 123 / 130, 99 / 104, 89 / 87); 10000 125 / 135, 104 / 102, 89 / 88
//   (134 / 131, 108 / 100, 94 / 86); 12000 146 / 145, 123 / 115, 108 / 100.
//   20480 (up to 8 or 4): 16384 (Plummer, theta 0.5) 147 / 162, 24576 (0.6) 171 /
//   153, 32768 (Plummer) 228 / 187.
//   262144 (up to 4 or 2): 200000 933 / 1016, 262144 1208 / 1264 and (0.6) 630 /
//   600, 500000 2281 / 2163 and 1199 / 1079.
//   2^20 (up to 2 or 1), forces of a disk + halo at 0.4, 0.6, 0.8: 300000 1360 /
//   1508, 690 / 735, 419 / 420; 700000 3015 / 3222, 1440 / 1462, 818 / 790; 1M 4252 /
//   4478, 1992 / 1987, 1140 / 1071; 1.2M 5074 / 5284, 2385 / 2383, 1346 / 1270; 2M
//   8537 / 8652, 3985 / 3940, 2183 / 2084; 3M 12937 / 12835, 6327 / 5982, 3487 /
//   3194.  The longer walks of a small theta gain by two waves and the short
//   ones of a large theta lose; the rule does not look at theta, and at a million
//   the three come out even.
struct Split {
    uint32_t logw, t1, t2;
};
__host__ __device__ inline uint32_t group_logw(const Split &s, uint32_t gn) {
    return s.logw - (gn <= s.t1 ? 1u : 0u) - (gn <= s.t2 ? 1u : 0u);
}
constexpr int64_t kSplit8 = 20480, kSplit4 = 262144, kSplit2 = 1048576;
inline Split walk_split(int64_t n) {
    if (n <= 8192) return {3u, 32u, 0u};
    if (n <= kSplit8) return {3u, 32u, 16u};
    if (n <= kSplit4) return {2u, 32u, 16u};
    if (n <= kSplit2) return {1u, 40u, 0u};
    return {0u, 0u, 0u};
}
// entries (one row of n per wave) of the partial sums of a context of n_max
inline int64_t split_rows(int64_t n_max) {
    const int64_t a = 8 * (n_max < kSplit8 ? n_max : kSplit8),
                  b = n_max > kSplit8 ? 4 * (n_max < kSplit4 ? n_max : kSplit4) : 0,
                  c = n_max > kSplit4 ? 2 * (n_max < kSplit2 ? n_max : kSplit2) : 0;
    return a > b ? (a > c ? a : c) : (b > c ? b : c);
}

// integrate.hip
void launch_save(const State &s, uint32_t n, char *dst, hipStream_t st);
void launch_kick_drift(bh_ctx *c, float h, float dt, uint32_t n, hipStream_t st);
void launch_unsort_add(bh_ctx *c, float *acc, float *pot, uint32_t n, hipStream_t st);
void launch_state_out(bh_ctx *c, float *pos, float *vel, uint32_t n, hipStream_t st);
void launch_range_out(bh_ctx *c, uint32_t lo, uint32_t cnt, float *pos, float *vel, float *mass,
                      uint32_t *ids, hipStream_t st);
void launch_totals(bh_ctx *c, uint32_t n, hipStream_t st);
void launch_count_leaves(bh_ctx *c, hipStream_t st);
void launch_diagnostics(bh_ctx *c, hipStream_t st);  // result at diag + kDiagBlocks * kDiagN
void launch_fill_u32(uint32_t *p, uint32_t v, uint64_t n, hipStream_t st);
void launch_cut(bh_ctx *c, int32_t p, int64_t C, uint64_t *S, int64_t *cuts, hipStream_t st);

inline uint32_t cdiv(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }

// Record timing event k of the context on st (contexts without events, such
// as the one tree_force_static assembles over its static buffer, skip it).
inline void record_event(bh_ctx *c, int k, hipStream_t st) {
    if (!c->ev[k]) return;
    (void)hipEventRecord(c->ev[k], st);
    c->ev_rec[k] = true;
}

// levels of a particle, packed: lo (5 bits), hi (5 bits), its group cell's
// level (5 bits), first of a group
__device__ __forceinline__ uint32_t lv_lo(uint32_t v) { return v & 31u; }
__device__ __forceinline__ uint32_t lv_hi(uint32_t v) { return (v >> 5) & 31u; }
__device__ __forceinline__ uint32_t lv_glev(uint32_t v) { return (v >> 10) & 31u; }
__device__ __forceinline__ bool lv_group(uint32_t v) { return (v >> 15) & 1u; }

// Peano-Hilbert curve (the curve of Sec. III.B.1), after J. Skilling,
// "Programming the Hilbert curve", AIP Conf. Proc. 707, 381 (2004): integer
// coordinates of b bits per axis are turned in place into the curve's
// transposed index, whose bits interleaved like a Morton key (X[0] the high
// bit of each digit) are the position along the curve; ph_decode inverts it.
// The top 3l bits of a key are the l-bit key of the coordinates' top l bits,
// so each octree cell is one key range, as with Morton keys.
__device__ __forceinline__ void ph_encode(uint32_t X[3], int b) {
    if (b < 1) return;
    const uint32_t top = 1u << (b - 1);
    for (uint32_t Q = top; Q > 1u; Q >>= 1) {
        const uint32_t P = Q - 1u;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const uint32_t sw = (X[0] ^ X[i]) & P;
            const bool inv = (X[i] & Q) != 0u;
            X[0] ^= inv ? P : sw;      // invert the low bits of X[0], or swap them
            if (!inv) X[i] ^= sw;      //   with those of X[i]
        }
    }
    X[1] ^= X[0];
    X[2] ^= X[1];
    uint32_t t = 0;
    for (uint32_t Q = top; Q > 1u; Q >>= 1)
        if (X[2] & Q) t ^= Q - 1u;
    X[0] ^= t;
    X[1] ^= t;
    X[2] ^= t;
}

__device__ __forceinline__ void ph_decode(uint32_t X[3], int b) {
    if (b < 1) return;
    const uint32_t end = 2u << (b - 1);
    const uint32_t t = X[2] >> 1;
    X[2] ^= X[1];
    X[1] ^= X[0];
    X[0] ^= t;
    for (uint32_t Q = 2; Q != end; Q <<= 1) {
        const uint32_t P = Q - 1u;
#pragma unroll
        for (int i = 2; i >= 0; --i) {
            const uint32_t sw = (X[0] ^ X[i]) & P;
            const bool inv = (X[i] & Q) != 0u;
            X[0] ^= inv ? P : sw;
            if (!inv) X[i] ^= sw;
        }
    }
}

}  // namespace bh
