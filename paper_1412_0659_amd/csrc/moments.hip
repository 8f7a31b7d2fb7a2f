// Upward pass: mass, centre of mass and quadrupole of every cell in FP64
// (Sec. I.A: multipole moments computed once the tree is built; Sec. VI.A
// Eq. (1): the quadrupole is the 3x3 second moment of the cell's mass about
// its centre of mass; Table II "Tree-properties").
//
//   leaf:   M = sum m, S = sum m x, com = S / M, Q = sum m s s^T, s = x - com
//   parent: M = sum M_c, S = sum S_c, com = S / M,
//           Q = sum (Q_c + M_c d d^T), d = com_c - com   (parallel axis)
//
// Each cell is one thread summing in a fixed order (a leaf over its
// particles in sorted order, a parent over its children in child order),
// with contraction off, so the result does not depend on the launch.  The
// FP64 record of a cell is M, S and Q (80 bytes); com = S / M is recomputed
// where needed.  The walk reads FP32 copies, written as soon as the moments
// are known: com and the opening radius r_open = l / theta + |com - geometric
// centre| (l = cell size) for the opening test, and (com, M, -3 Q, tr Q / 2,
// -3 tr Q / 2) for the particle-cell terms.
//
// The cells that start and end inside one tile of kTreeTile particles are
// summed by the tile's block (k_moments_tile): its leaves first, all levels
// at once, then its parents from the deepest level up, each level's moments
// kept in LDS for the next.  A cell across a tile's end is the last one of
// its level to start in the tile, so at most one per tile and level is left
// over; those inside a span of kSpanTiles tiles are summed by one block per
// span (k_moments_span, eight lanes per tile end, level by level), the rest by
// one block (k_moments_top, eight lanes per span end): three launches for any
// number of particles and levels (one to kTreeTile particles, two to a span).
//
// Bound: memory, 16 B per particle and 200 B per cell; on small sets the
// chain of levels (0.6 us a level in a tile, 2.5 us in the spans).  Measured:
// 0.36 ms at 13M, 0.092 ms at 1M, where one launch per level took 0.42 and
// 0.135 ms (22 launches on a new particle set); 16384: 42 against 95 us, 1000:
// 16 against 67.  A tile's parents by one lane each took 25 us at 1000 and 51 at
// 16384 with the spans (a chain of 400 instructions a level against 120), with
// eight lanes per parent split by child instead of by quantity the tile's LDS
// would hold three blocks a CU instead of four.  Across tile ends, one lane per
// parent (its 27 FP64 divisions in a row) took 54 and 135 us in the spans and
// the top at 13M; sums by shuffles 101 and 191; LDS sums one read at a time with
// all records written inside the chain of levels 52 and 67, 15 us more at 100003
// than now.
#include "bh_internal.h"
#include "wave.h"

namespace bh {

// A leaf's particles are read kBatch at a time (the loads of a batch issue
// together), once for the mass and centre and once more, from the cache, for
// the quadrupole: holding 16 particles in registers instead halved the waves
// in flight.
constexpr uint32_t kBatch = 8;

struct MomArgs {
    Cells c;
    const float4 *xyzm;  // sorted particles as (x, y, z, m) records
    const float *box;  // lo xyz, side
    int curve;
    // theta > 0: the opening radii for a walk at theta, and its counters zeroed
    float theta;
    uint32_t *work;
    unsigned long long *totals;
};

struct Mom {
    double M, s0, s1, s2, q0, q1, q2, q3, q4, q5;
};

__device__ __forceinline__ void leaf_sums(const MomArgs &a, uint32_t b, uint32_t cnt, Mom &r,
                                          double &c0, double &c1, double &c2) {
    r = Mom{0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    float4 p[kBatch];
#pragma unroll 1
    for (uint32_t o = 0; o < cnt; o += kBatch) {
#pragma unroll
        for (uint32_t k = 0; k < kBatch; ++k) p[k] = a.xyzm[o + k < cnt ? b + o + k : b];
#pragma unroll
        for (uint32_t k = 0; k < kBatch; ++k) {
            if (o + k < cnt) {
                const double mj = p[k].w;
                r.M = r.M + mj;
                r.s0 = r.s0 + mj * (double)p[k].x;
                r.s1 = r.s1 + mj * (double)p[k].y;
                r.s2 = r.s2 + mj * (double)p[k].z;
            }
        }
    }
    c0 = r.s0 / r.M; c1 = r.s1 / r.M; c2 = r.s2 / r.M;
#pragma unroll 1
    for (uint32_t o = 0; o < cnt; o += kBatch) {
        if (cnt > kBatch) {
#pragma unroll
            for (uint32_t k = 0; k < kBatch; ++k) p[k] = a.xyzm[o + k < cnt ? b + o + k : b];
        }
#pragma unroll
        for (uint32_t k = 0; k < kBatch; ++k) {
            if (o + k < cnt) {
                const double mj = p[k].w;
                const double d0 = (double)p[k].x - c0, d1 = (double)p[k].y - c1,
                             d2 = (double)p[k].z - c2;
                r.q0 = r.q0 + (mj * d0) * d0;
                r.q1 = r.q1 + (mj * d1) * d1;
                r.q2 = r.q2 + (mj * d2) * d2;
                r.q3 = r.q3 + (mj * d0) * d1;
                r.q4 = r.q4 + (mj * d0) * d2;
                r.q5 = r.q5 + (mj * d1) * d2;
            }
        }
    }
}

// A parent from its children in memory, in child order; a child's centre of
// mass is its S / M, the same division that made it.
__device__ __forceinline__ void parent_sums(const Cells &c, uint32_t k0, uint32_t nch, Mom &r,
                                            double &c0, double &c1, double &c2) {
    r = Mom{0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (size_t j = k0; j < (size_t)k0 + nch; ++j) {
        r.M = r.M + c.M[j];
        r.s0 = r.s0 + c.S[3 * j];
        r.s1 = r.s1 + c.S[3 * j + 1];
        r.s2 = r.s2 + c.S[3 * j + 2];
    }
    c0 = r.s0 / r.M; c1 = r.s1 / r.M; c2 = r.s2 / r.M;
#pragma unroll 1
    for (size_t j = k0; j < (size_t)k0 + nch; ++j) {
        const double mk = c.M[j];
        const double d0 = c.S[3 * j] / mk - c0, d1 = c.S[3 * j + 1] / mk - c1,
                     d2 = c.S[3 * j + 2] / mk - c2;
        const double *Q = c.Q + 6 * j;
        r.q0 = r.q0 + (Q[0] + (mk * d0) * d0);
        r.q1 = r.q1 + (Q[1] + (mk * d1) * d1);
        r.q2 = r.q2 + (Q[2] + (mk * d2) * d2);
        r.q3 = r.q3 + (Q[3] + (mk * d0) * d1);
        r.q4 = r.q4 + (Q[4] + (mk * d0) * d2);
        r.q5 = r.q5 + (Q[5] + (mk * d1) * d2);
    }
}

// every third bit of v (bits 0, 3, 6, ...) gathered into the low 21 bits
__device__ __forceinline__ uint32_t every_third_bit(uint64_t v) {
    v &= 0x1249249249249249ull;
    v = (v ^ (v >> 2)) & 0x10C30C30C30C30C3ull;
    v = (v ^ (v >> 4)) & 0x100F00F00F00F00Full;
    v = (v ^ (v >> 8)) & 0x001F0000FF0000FFull;
    v = (v ^ (v >> 16)) & 0x001F00000000FFFFull;
    v = (v ^ (v >> 32)) & 0x00000000001FFFFFull;
    return (uint32_t)v;
}

// corner coordinates of a cell from its key prefix (x the high bit of each
// 3-bit digit, the first digit the most significant)
__device__ __forceinline__ void cell_coords(uint64_t prefix, uint32_t p[3]) {
    p[0] = every_third_bit(prefix >> 2);
    p[1] = every_third_bit(prefix >> 1);
    p[2] = every_third_bit(prefix);
}

// Write cell i's moments and walk records; the build left the ends of its
// particles and children, made counts here.
__device__ __forceinline__ void cell_out(const MomArgs &a, uint32_t i, uint32_t lev,
                                         uint64_t prefix, uint32_t b0, uint32_t n0, uint32_t k0,
                                         uint32_t nch, const Mom &r, double c0, double c1,
                                         double c2) {
    const Cells &c = a.c;
    c.count[i] = n0;
    c.nchild[i] = nch;
    c.M[i] = r.M;
    c.S[3 * i] = r.s0; c.S[3 * i + 1] = r.s1; c.S[3 * i + 2] = r.s2;
    double2 *q = reinterpret_cast<double2 *>(c.Q) + 3 * (size_t)i;
    q[0] = make_double2(r.q0, r.q1);
    q[1] = make_double2(r.q2, r.q3);
    q[2] = make_double2(r.q4, r.q5);

    // walk records: com (FP32), opening-radius terms, particle-cell record
    const double lo0 = a.box[0], lo1 = a.box[1], lo2 = a.box[2], side = a.box[3];
    uint32_t p[3];
    cell_coords(prefix, p);          // the digits, deinterleaved
    if (a.curve == 1) ph_decode(p, (int)lev);  // Peano-Hilbert prefix -> octant
    const double lc = side * (1.0 / (double)(1u << lev));
    const double e0 = c0 - (lo0 + ((double)p[0] + 0.5) * lc);
    const double e1 = c1 - (lo1 + ((double)p[1] + 0.5) * lc);
    const double e2 = c2 - (lo2 + ((double)p[2] + 0.5) * lc);
    const double dl = __dsqrt_rn((e0 * e0 + e1 * e1) + e2 * e2);
    const double tr = (r.q0 + r.q1) + r.q2;
    const float2 size = make_float2((float)lc, (float)dl);
    c.wA[i] = make_float4((float)c0, (float)c1, (float)c2,
                          a.theta > 0.f ? open_radius2(size, a.theta) : 0.f);
    c.P0[i] = make_float4((float)c0, (float)c1, (float)c2, (float)r.M);
    c.P1[i] = make_float4((float)(-3.0 * r.q0), (float)(-3.0 * r.q1), (float)(-3.0 * r.q2),
                          (float)(-3.0 * r.q3));
    c.P2[i] = make_float4((float)(-3.0 * r.q4), (float)(-3.0 * r.q5), (float)(0.5 * tr),
                          (float)(-1.5 * tr));
    c.wN[i] = nch ? make_uint2(k0, nch) : make_uint2(b0, n0 | kLeafBit);
    c.size[i] = size;
}

// Cell i of level lev on its own, a parent's children read from memory.
__device__ __forceinline__ void cell_pass(const MomArgs &a, uint32_t i, uint32_t lev) {
    const Cells &c = a.c;
    // the topology in one round of loads (child0 is only used by parents)
    const uint32_t kend = c.nchild[i], b0 = c.begin[i], n0 = c.count[i] - b0, k0 = c.child0[i];
    const uint64_t prefix = c.prefix[i];
    const uint32_t nch = kend ? kend - k0 : 0u;
    Mom r;
    double c0, c1, c2;
    if (nch == 0) leaf_sums(a, b0, n0, r, c0, c1, c2);
    else parent_sums(c, k0, nch, r, c0, c1, c2);
    cell_out(a, i, lev, prefix, b0, n0, k0, nch, r, c0, c1, c2);
}

// The cells of level l that start before tile t (the total for t = tiles).
__device__ __forceinline__ uint32_t starts_before(const Cells &c, uint32_t ntiles, uint32_t l,
                                                  uint32_t t) {
    const uint32_t *pre = ntiles <= kScanTiles ? c.ttot + kLevels + 1 : c.tcnt;
    return t < ntiles ? pre[(size_t)l * ntiles + t] : c.ttot[l];
}

// The levels l < levels_across(i) are those whose cells hold both particle
// i - 1 and i.
__device__ __forceinline__ uint32_t levels_across(const Cells &c, uint32_t i) {
    return min(lv_hi(c.lev[i - 1u]) + 1u, lv_lo(c.lev[i]));
}

// v of the lane that kCtrl names in each quad
template <int kCtrl>
__device__ __forceinline__ double quad_lane(double v) {
    const int2 i = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(
        double, make_int2(__builtin_amdgcn_update_dpp(0, i.x, kCtrl, 0xf, 0xf, false),
                          __builtin_amdgcn_update_dpp(0, i.y, kCtrl, 0xf, 0xf, false)));
}

constexpr int kMomCells = 368;  // cells of a tile whose moments fit in LDS (235 on average)

// (sixteen waves a CU either way)
template <int kMomThreads>
__global__ __launch_bounds__(kMomThreads, 1024 / kMomThreads) void k_moments_tile(MomArgs a, uint32_t n,
                                                              uint32_t ntiles) {
    // M, S xyz, com xyz, Q xx yy zz xy xz yz of the tile's cells
    __shared__ double mo[13][kMomCells];
    __shared__ uint32_t first[kLevels], ofs[kLevels + 1], inside[kLevels];
    // the parents of level l: par[ofs[l] ..], npar[l] of them, each its cell, its
    // first child and the number of its children
    __shared__ uint32_t par[kMomCells], npar[kLevels];
    static_assert(kMomCells <= 512, "nine bits for a cell");
    const Cells &c = a.c;
    const uint32_t lane = lane_id();
    if (a.theta > 0.f && blockIdx.x == 0) zero_walk(a.work, a.totals);
    if (threadIdx.x < 64) {
        const uint32_t l = min(lane, (uint32_t)kLevels - 1u);
        const uint32_t s0 = starts_before(c, ntiles, l, blockIdx.x),
                       s1 = starts_before(c, ntiles, l, blockIdx.x + 1u);
        const uint32_t cnt = lane < kLevels ? s1 - s0 : 0u;
        const uint32_t end = (blockIdx.x + 1u) * kTreeTile;
        const uint32_t across = end < n ? levels_across(c, end) : 0u;
        const uint32_t inc = wave_incl_scan(cnt, lane);
        if (lane <= kLevels) ofs[lane] = inc - cnt;
        if (lane < kLevels) {
            first[lane] = c.ls[lane] + s0;
            // the last cell to start is left out where it holds the tile's end
            inside[lane] = cnt && lane < across ? cnt - 1u : cnt;
            npar[lane] = 0u;
        }
    }
    __syncthreads();
    const uint32_t total = ofs[kLevels];
    if (total > (uint32_t)kMomCells) {  // (tiny leaves, chains of coincident particles)
        for (int l = kLevels - 1; l >= 0; --l) {
            const uint32_t m = inside[l];
            for (uint32_t q = threadIdx.x; q < m; q += kMomThreads)
                cell_pass(a, first[l] + q, (uint32_t)l);
            if (m) __syncthreads();  // the next level up reads these cells
        }
        return;
    }
    auto keep = [&](uint32_t q, const Mom &r, double c0, double c1, double c2) {
        mo[0][q] = r.M;
        mo[1][q] = r.s0; mo[2][q] = r.s1; mo[3][q] = r.s2;
        mo[4][q] = c0; mo[5][q] = c1; mo[6][q] = c2;
        mo[7][q] = r.q0; mo[8][q] = r.q1; mo[9][q] = r.q2;
        mo[10][q] = r.q3; mo[11][q] = r.q4; mo[12][q] = r.q5;
    };
    // ---- this thread's cells: topology, and the moments of the leaves
    constexpr int kOwn = (kMomCells + kMomThreads - 1) / kMomThreads;
    uint32_t lev[kOwn], ci[kOwn], b0[kOwn], n0[kOwn], k0[kOwn], nch[kOwn];
    uint64_t prefix[kOwn];
#pragma unroll
    for (int s = 0; s < kOwn; ++s) {
        const uint32_t q = threadIdx.x + s * kMomThreads;
        lev[s] = kNone;  // no cell
        if (q >= total) continue;
        uint32_t l = 0;
#pragma unroll
        for (int k = 1; k < kLevels; ++k) l += q >= ofs[k] ? 1u : 0u;
        if (q - ofs[l] >= inside[l]) continue;
        lev[s] = l;
        const uint32_t i = first[l] + (q - ofs[l]);
        ci[s] = i;
        const uint32_t kend = c.nchild[i];
        b0[s] = c.begin[i];
        n0[s] = c.count[i] - b0[s];
        k0[s] = c.child0[i];
        prefix[s] = c.prefix[i];
        nch[s] = kend ? kend - k0[s] : 0u;
        if (nch[s])
            par[ofs[l] + atomicAdd(&npar[l], 1u)] =
                q | (ofs[l + 1u] + (k0[s] - first[l + 1u])) << 9 | nch[s] << 18;
    }
#pragma unroll
    for (int s = 0; s < kOwn; ++s) {
        if (lev[s] == kNone || nch[s] != 0u) continue;
        Mom r;
        double c0, c1, c2;
        leaf_sums(a, b0[s], n0[s], r, c0, c1, c2);
        keep(threadIdx.x + s * kMomThreads, r, c0, c1, c2);
    }
    // ---- the parents, from the deepest level up, by eight lanes each: lane k
    // sums quantity k mod 4 of (M, S), then entry k of Q, over the children in
    // child order
    const uint32_t k = lane & 7u, k4 = lane & 3u;
    const uint32_t ra = k < 3u ? k : (k == 5u ? 1u : 0u), rb = k < 3u ? k : (k == 3u ? 1u : 2u);
    __syncthreads();
    for (uint32_t l = kLevels - 1; l-- > 0u;) {
        const uint32_t np = npar[l];
        if (np == 0u) continue;
        for (uint32_t u = threadIdx.x >> 3; u < np; u += kMomThreads / 8) {
            const uint32_t e = par[ofs[l] + u], q = e & 511u, q0 = (e >> 9) & 511u, m = e >> 18;
            double x[8], v = 0.0;
#pragma unroll
            for (uint32_t j = 0; j < 8u; ++j) x[j] = mo[k4][q0 + (j < m ? j : 0u)];
#pragma unroll
            for (uint32_t j = 0; j < 8u; ++j) v = j < m ? v + x[j] : v;
            const double com = v / quad_lane<0x00>(v);
            const double c0 = quad_lane<0x55>(com), c1 = quad_lane<0xaa>(com),
                         c2 = quad_lane<0xff>(com);
            const double ca = ra == 0u ? c0 : (ra == 1u ? c1 : c2),
                         cb = rb == 0u ? c0 : (rb == 1u ? c1 : c2);
            if (k < 4u) mo[k][q] = v;
            if (k > 0u && k < 4u) mo[3u + k][q] = com;
            if (k < 6u) {
                double w = 0.0;
#pragma unroll 4
                for (uint32_t j = 0; j < 8u; ++j) {
                    const uint32_t i = q0 + (j < m ? j : 0u);
                    const double t = mo[7u + k][i] +
                                     (mo[0][i] * (mo[4u + ra][i] - ca)) * (mo[4u + rb][i] - cb);
                    w = j < m ? w + t : w;
                }
                mo[7u + k][q] = w;
            }
        }
        __syncthreads();
    }
    // ---- all of them written
#pragma unroll
    for (int s = 0; s < kOwn; ++s) {
        if (lev[s] == kNone) continue;
        const uint32_t q = threadIdx.x + s * kMomThreads;
        const Mom r{mo[0][q], mo[1][q], mo[2][q], mo[3][q], mo[7][q],
                    mo[8][q], mo[9][q], mo[10][q], mo[11][q], mo[12][q]};
        cell_out(a, ci[s], lev[s], prefix[s], b0[s], n0[s], k0[s], nch[s], r, mo[4][q], mo[5][q],
                 mo[6][q]);
    }
}

struct Across {
    uint32_t i, k0, nch;  // i = kNone: none
};

constexpr int kAcrossThreads = 1024;
constexpr int kAcrossUnits = kAcrossThreads / 8;
constexpr int kAcrossRow = kAcrossThreads + 2;  // (the eight lanes' rows in different banks)
static_assert(kAcrossUnits >= kSpanTiles, "a span's tiles in one round");

// row[b] = the sum of row[b .. b + n - 1], n <= 8, in that order (the eight
// reads go out together)
__device__ __forceinline__ void ordered_sum(double *row, uint32_t b, uint32_t n) {
    double x[8], v = 0.0;
#pragma unroll
    for (uint32_t j = 0; j < 8u; ++j) x[j] = row[b + j];
#pragma unroll
    for (uint32_t j = 0; j < 8u; ++j) v = j < n ? v + x[j] : v;
    row[b] = v;
}

// The moments of a parent across an end, by eight lanes of a wave (have:
// these eight have one): lane k reads child k, then each sum over the children
// runs in child order in one lane, through the LDS rows ch.
__device__ __forceinline__ void group_parent(const Cells &c, bool have, const Across &o,
                                             double (*ch)[kAcrossRow]) {
    const uint32_t t = threadIdx.x, k = t & 7u, b = t & ~7u;
    const double2 *Q2 = reinterpret_cast<const double2 *>(c.Q);
    const uint32_t nch = have ? o.nch : 0u;
    double cm = 0.0, s0 = 0.0, s1 = 0.0, s2 = 0.0;
    double2 qa = make_double2(0.0, 0.0), qb = qa, qc = qa;
    if (k < nch) {
        const size_t j = (size_t)o.k0 + k;
        cm = c.M[j];
        s0 = c.S[3 * j]; s1 = c.S[3 * j + 1]; s2 = c.S[3 * j + 2];
        qa = Q2[3 * j]; qb = Q2[3 * j + 1]; qc = Q2[3 * j + 2];
    }
    ch[0][t] = cm; ch[1][t] = s0; ch[2][t] = s1; ch[3][t] = s2;
    wave_sync();
    if (k < 4u) ordered_sum(ch[k], b, nch);
    wave_sync();
    const double M = ch[0][b];
    const double c0 = ch[1][b] / M, c1 = ch[2][b] / M, c2 = ch[3][b] / M;
    const double d0 = s0 / cm - c0, d1 = s1 / cm - c1, d2 = s2 / cm - c2;
    ch[4][t] = qa.x + (cm * d0) * d0;
    ch[5][t] = qa.y + (cm * d1) * d1;
    ch[6][t] = qb.x + (cm * d2) * d2;
    ch[7][t] = qb.y + (cm * d0) * d1;
    ch[8][t] = qc.x + (cm * d0) * d2;
    ch[9][t] = qc.y + (cm * d1) * d2;
    wave_sync();
    if (k < 6u) ordered_sum(ch[4u + k], b, nch);
    wave_sync();
    if (have) {  // what the next level reads
        const size_t i = o.i;
        if (k == 0u) c.M[i] = ch[0][b];
        if (k < 3u) c.S[3 * i + k] = ch[1u + k][b];
        if (k < 6u) c.Q[6 * i + k] = ch[4u + k][b];
    }
    wave_sync();
}

// The cells across the ends of consecutive units of `tiles` tiles (unit u
// ends at particle (u + 1) tiles kTreeTile): those that end by `limit`, of the
// units u0 .. u0 + units - 1.  Eight lanes per unit; first each lane looks up
// the cells of its unit on every eighth level (and finishes a leaf, of which
// there is at most one), then level by level from the deepest the eight sum
// the unit's parent.
__device__ __forceinline__ void across_pass(const MomArgs &a, uint32_t ntiles, uint32_t u0,
                                            uint32_t units, uint32_t tiles, uint32_t limit) {
    __shared__ double ch[10][kAcrossRow];
    __shared__ uint32_t levels;  // bit l: some unit has a parent on level l
    constexpr int kOwn = (kLevels + 7) / 8;
    static_assert(kOwn == 3, "levels a lane looks up");
    const Cells &c = a.c;
    const uint32_t len = tiles * kTreeTile;
    const uint32_t uu = threadIdx.x >> 3, k = threadIdx.x & 7u;
    if (units <= (uint32_t)kAcrossUnits) {
        if (threadIdx.x == 0) levels = 0u;
        __syncthreads();
        const uint32_t across = uu < units ? levels_across(c, (u0 + uu + 1u) * len) : 0u;
        uint32_t leaf = kNone, leaf_level = 0;
        // (an array per field, so that they stay in registers)
        uint32_t wi[kOwn], wb[kOwn], wn[kOwn], wk[kOwn], wc[kOwn], wp0[kOwn], wp1[kOwn];
#pragma unroll
        for (int s = 0; s < kOwn; ++s) {
            const uint32_t l = k + 8u * (uint32_t)s;
            wi[s] = kNone;
            wb[s] = wn[s] = wk[s] = wc[s] = wp0[s] = wp1[s] = 0u;
            if (l >= across) continue;
            const uint32_t s1 = starts_before(c, ntiles, l, (u0 + uu + 1u) * tiles);
            if (s1 == starts_before(c, ntiles, l, (u0 + uu) * tiles)) continue;
            const uint32_t i = c.ls[l] + s1 - 1u;
            const uint32_t end = c.count[i];  // (still the end of its particles)
            const uint32_t kend = c.nchild[i], k0 = c.child0[i], b0 = c.begin[i];
            const uint64_t pre = c.prefix[i];
            if (end > limit) continue;
            if (kend == 0u) {
                leaf = i;
                leaf_level = l;
                continue;
            }
            wi[s] = i;
            wb[s] = b0; wn[s] = end - b0;
            wk[s] = k0; wc[s] = kend - k0;
            wp0[s] = (uint32_t)pre; wp1[s] = (uint32_t)(pre >> 32);
            atomicOr(&levels, 1u << l);
        }
        if (leaf != kNone) cell_pass(a, leaf, leaf_level);
        __syncthreads();
        uint32_t todo = levels;
        while (todo) {
            const uint32_t l = 31u - (uint32_t)__clz((int)todo);
            todo &= ~(1u << l);
            const int src = (int)((lane_id() & ~7u) + (l & 7u));
            auto pick = [&](uint32_t v0, uint32_t v1, uint32_t v2) {
                return shfl(l < 8u ? v0 : (l < 16u ? v1 : v2), src);
            };
            Across o{pick(wi[0], wi[1], wi[2]), 0u, 0u};
            if (ballot(o.i != kNone) != 0ull) {
                o.k0 = pick(wk[0], wk[1], wk[2]); o.nch = pick(wc[0], wc[1], wc[2]);
                group_parent(c, o.i != kNone, o, ch);
            }
            __syncthreads();  // the next level up reads these cells
        }
        // the rest of their records, off the chain of levels
#pragma unroll
        for (int s = 0; s < kOwn; ++s) {
            const size_t i = wi[s];
            if (wi[s] == kNone) continue;
            const Mom r{c.M[i],     c.S[3 * i],     c.S[3 * i + 1], c.S[3 * i + 2], c.Q[6 * i],
                        c.Q[6 * i + 1], c.Q[6 * i + 2], c.Q[6 * i + 3], c.Q[6 * i + 4],
                        c.Q[6 * i + 5]};
            cell_out(a, wi[s], k + 8u * (uint32_t)s, ((uint64_t)wp1[s] << 32) | wp0[s], wb[s],
                     wn[s], wk[s], wc[s], r, r.s0 / r.M, r.s1 / r.M, r.s2 / r.M);
        }
        return;
    }
    // more units than lanes (sets of more than 16 million particles): every
    // level over all of them before the next
    for (int l = kLevels - 1; l >= 0; --l) {
        for (uint32_t u = threadIdx.x; u < units; u += (uint32_t)kAcrossThreads) {
            if ((uint32_t)l >= levels_across(c, (u0 + u + 1u) * len)) continue;
            const uint32_t s1 = starts_before(c, ntiles, (uint32_t)l, (u0 + u + 1u) * tiles);
            if (s1 == starts_before(c, ntiles, (uint32_t)l, (u0 + u) * tiles)) continue;
            const uint32_t i = c.ls[l] + s1 - 1u;
            if (c.count[i] <= limit) cell_pass(a, i, (uint32_t)l);
        }
        __syncthreads();
    }
}

// The cells across a tile's end that end inside its span of kSpanTiles tiles.
__global__ __launch_bounds__(kAcrossThreads) void k_moments_span(MomArgs a, uint32_t ntiles) {
    const uint32_t u0 = blockIdx.x * kSpanTiles;
    const uint32_t ends = min((uint32_t)kSpanTiles, ntiles - 1u - u0);  // tile ends below n
    across_pass(a, ntiles, u0, ends, 1u, (blockIdx.x + 1u) * (kSpanTiles * kTreeTile));
}

// The cells across a span's end, by one block.
__global__ __launch_bounds__(kAcrossThreads) void k_moments_top(MomArgs a, uint32_t n,
                                                                uint32_t ntiles,
                                                                uint32_t nspans) {
    across_pass(a, ntiles, 0u, nspans - 1u, kSpanTiles, n);
}

void launch_moments(bh_ctx *ctx, uint32_t n, float theta, hipStream_t st) {
    MomArgs a;
    a.c = ctx->cells;
    a.xyzm = ctx->xyzm;
    a.box = ctx->box;
    a.curve = (int)ctx->p.curve;
    a.theta = theta;
    a.work = ctx->work;
    a.totals = ctx->totals;
    const uint32_t nt = cdiv(n, kTreeTile), ns = cdiv(nt, kSpanTiles);
    // Threads of a tile: one cell each while there is about a tile for each CU,
    // else more tiles a CU.  The launches by 256 / 512, in us: 1000 18.5 / 16.3;
    // 16384 44 / 42; 100003 59 / 57; 1M 92 / 99; 13M 364 / 422.
    if (n <= 262144u) hipLaunchKernelGGL(k_moments_tile<512>, dim3(nt), dim3(512), 0, st, a, n, nt);
    else hipLaunchKernelGGL(k_moments_tile<256>, dim3(nt), dim3(256), 0, st, a, n, nt);
    if (nt > 1) hipLaunchKernelGGL(k_moments_span, dim3(ns), dim3(kAcrossThreads), 0, st, a, nt);
    if (ns > 1) hipLaunchKernelGGL(k_moments_top, dim3(1), dim3(kAcrossThreads), 0, st, a, n, nt, ns);
}

// com = S / M of every cell (FP64), for export
__global__ __launch_bounds__(256) void k_com(Cells c) {
    const uint32_t nc = c.ls[kLevels];
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < nc; i += gridDim.x * 256) {
        const double mm = c.M[i];
        c.com[3 * i] = c.S[3 * i] / mm;
        c.com[3 * i + 1] = c.S[3 * i + 1] / mm;
        c.com[3 * i + 2] = c.S[3 * i + 2] / mm;
    }
}

void launch_com(bh_ctx *ctx, hipStream_t st) {
    hipLaunchKernelGGL(k_com, dim3(kGrid * 2), dim3(256), 0, st, ctx->cells);
}

// The opening radii of a walk at theta, stored in wA.w; the first block also
// zeroes the walk's counters.
__global__ __launch_bounds__(256) void k_walk_prep(Cells c, float theta, uint32_t *work,
                                                   unsigned long long *totals) {
    if (blockIdx.x == 0) zero_walk(work, totals);
    const uint32_t nc = c.ls[kLevels];
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < nc; i += gridDim.x * 256)
        c.wA[i].w = open_radius2(c.size[i], theta);
}

void launch_walk_prep(bh_ctx *ctx, float theta, bh_ctx *walker, bool totals, hipStream_t st) {
    // (a cell per particle at most in sets worth more than a few blocks)
    const uint32_t nb = cdiv((uint64_t)ctx->n, 256);
    hipLaunchKernelGGL(k_walk_prep, dim3(nb < kGrid * 2u ? nb : kGrid * 2u), dim3(256), 0, st,
                       ctx->cells, theta, walker ? walker->work : nullptr,
                       walker && totals ? walker->totals : nullptr);
}

}  // namespace bh
