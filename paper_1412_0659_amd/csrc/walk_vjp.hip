// Adjoint of the tree force with the walk's decisions held fixed: given a
// cotangent u_i of every acceleration a_i, accumulate u^T da/dx and
// u^T da/dm.  The force is Sec. VI.A Eq. (2) (with r^2 -> r^2 + eps^2) over
// the interaction lists of the walk; cells enter through their moments
// (Sec. I.A, Eq. (1)), so the adjoint has three parts:
//   * targets:  d a_i / d x_i = -sum J  (J = dF/dd, d = source - x_i);
//   * sources:  particle j gets +J^T u_i and d F/d m_j . u_i; cell c gets
//               dL/dcom += J^T u_i, dL/dM += dF/dM . u_i, dL/dQ += dF/dQ . u_i;
//   * moments:  each particle k receives, from every cell holding it, with
//               s = x_k - com:  dcom/dx_k = m_k / M, dQ/dx_k = m_k (e s^T + s e^T),
//               dM/dm_k = 1, dcom/dm_k = s / M, dQ/dm_k = s s^T (the centre of
//               mass dependence of Q cancels because sum m s = 0).
// The walk (walk_common.h) is repeated exactly, so the lists are those of the
// force evaluation.  Both lists are taken in chunks of 64 sources, lane =
// source, looping over the group's targets; each pair's J^T u is added to the
// source's running sums and, summed over the lanes, subtracted from the
// target's.  That second sum runs on the matrix cores: a 16 x 16 x 4 FP32
// product of a matrix whose row t % 16 is one and the other rows zero with the
// 64 lanes' values adds four lanes' sum to each of 16 columns of the target's
// row (exact products, FP32 sums), so a trip issues three of them instead of 21
// dependent DPP adds and three lane reads; the columns are added once per list
// flush.  A value that is not finite would reach the other rows as 0 x inf:
// such a flush is seen by its sums and its target side taken again with the
// lane sums.
//
// Source terms reach FP64 accumulators with one atomic per value, source and
// group.  They come in kXcd copies, one per XCD: a wave adds into the copy of
// the XCD it runs on (read from the hardware XCC id), so no cache line is
// updated from two XCDs.  The cells of the top levels are accepted by far more
// groups than deeper ones (a few cache lines of them take a quarter of all the
// atomics), so the first kHotCells cells get kHotCopies copies, kHotCopies /
// kXcd per XCD chosen by the workgroup.  The copies are summed after the walk.
// A cell's (particle's) values lie together, and a chunk's sums are turned
// through LDS so that the lanes of one atomic instruction add to consecutive
// addresses: the cells of a list come in runs of siblings, and 64 cells of ten
// values are 40 to 60 cache lines instead of ten times the 15 or so runs.
//
// Sums: a source's over the group's targets and a target's over one flush of a
// list are FP32 (the latter in 16 columns); flushes, lists and waves meet in
// FP64.  (One FP32 sum over all flushes lost 1e-3 to 0.5 of the cells' part of
// a target next to a pair 0.02 to 0.005 apart; the three wider sums cost 1 to 3%
// on sets of up to 4096, nothing from 16384.)  B' below, the quadrupole with its
// trace folded in, is rounded to FP32 once more than the two terms it stands
// for.  Against FP64 on the same lists (300 to 40000 particles, theta 0.3 to
// 0.8) the positions' gradient is 0.20 to 0.94 times as far off as with lane
// sums and the trace apart, the masses' as far.
//
// Bound: the L2's atomics, which go at 2.35e10 requests of 64 bytes per second
// (1.9e11 adds where eight lanes fill a request): at 1M (theta 0.4) 2.34e9 adds
// leave in 3.46e8 requests, 14.7 ms at that rate.  The walk takes 16.9 ms, 15.9
// with the pairs left out and 14.2 with the adds left out (84 VALU instructions
// and a reciprocal root per particle-cell pair).  It took 23.0 ms with lane sums
// by DPP, accumulators field by field and particle pairs evaluated once per
// side; 19.4 with a source's sums added once per 32 targets.
#include <algorithm>

#include "walk_common.h"

namespace bh {

constexpr uint32_t kXcd = 8;
constexpr uint32_t kCellAdj = 10;  // a cell's adjoints: M, com xyz, Q xx yy zz xy xz yz

// XCD (XCC) that runs the calling wave.
__device__ __forceinline__ uint32_t xcc_id() {
    uint32_t v;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(v));
    return v & (kXcd - 1u);
}

// FP64 add executed in the L2 of the calling XCD (no return value).
__device__ __forceinline__ void add_l2(double *p, double v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

struct VjpArgs {
    const float4 *xyzm;   // sorted positions + mass
    const float4 *u;      // sorted cotangents of the accelerations
    const float4 *wA;
    const uint2 *wN;
    const float4 *P0, *P1, *P2;
    const uint32_t *gbeg, *ngroups;
    uint32_t *work, *spill, *status;
    uint32_t ring;
    Split split;
    // copy 0 of kXcd accumulators; copy k at + k * lstride / gstride: cell
    // adjoint q of cell c at lcell[kCellAdj * c + q], particle adjoint q of
    // particle j at gsrc[4 * j + q]
    double *lcell, *gsrc;
    uint64_t lstride, gstride;
    // kHotCopies copies of the first kHotCells cells' adjoints, copy k at
    // lhot + k * kHotCopy
    double *lhot;
    float eps2;
};

__device__ __forceinline__ float rsqv(float v) { return __builtin_amdgcn_rsqf(v); }

// Adjoint of one particle-cell term.  A = (com, M); B = (xx, yy, zz, xy) and
// C = (xz, yz, e) of the trace-free B' = -3 Q + tr(Q) I with e = tr(Q) eps^2,
// in which the force is F = M d r^-3 + q r^-5 - 5/2 s d r^-7, q = B'd, s = d.q +
// e (Eq. (2) with the trace taken into the quadrupole term).  Returns
//   w = J^T u = u (M r^-3 - 5/2 s r^-7) + B'u r^-5 - 5 ud r^-7 q
//       + d [ud (-3 M r^-5 + 35/2 s r^-9) - 5 uq r^-7],
// ud = u.d, uq = u.q, and adds the cell-side terms to running sums:
// dF/dM . u = ud r^-3 to sM.  dF/dQ . u for the six stored entries: with v =
// r^-5 u - 5/2 ud r^-7 d,
//   diagonal  -3 v_a d_a - 3/2 ud r^-5,   off-diagonal  -3 (v_a d_b + v_b d_a);
// sQ collects the v-terms unscaled (diagonal v_a d_a, off-diagonal
// v_a d_b + v_b d_a) and st the ud r^-5, so that the factors -3 and -3/2 are
// applied once per sum (pc_adj_finish).
struct CellSums {
    float w[3], M, Q[6], t;
};

__device__ __forceinline__ void pc_adj(const float *T, const float *U, const float4 &A,
                                       const float4 &B, const float4 &C, float eps2, float w[3],
                                       CellSums &c) {
    const float dx = A.x - T[0], dy = A.y - T[1], dz = A.z - T[2];
    const float r2 = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, eps2)));
    const float ri = rsqv(r2);
    const float ri2 = ri * ri, ri3 = ri * ri2, ri5 = ri3 * ri2, ri7 = ri5 * ri2;
    const float ud = fmaf(U[0], dx, fmaf(U[1], dy, U[2] * dz));
    const float qx = fmaf(B.x, dx, fmaf(B.w, dy, C.x * dz));
    const float qy = fmaf(B.w, dx, fmaf(B.y, dy, C.y * dz));
    const float qz = fmaf(C.x, dx, fmaf(C.y, dy, B.z * dz));
    const float bux = fmaf(B.x, U[0], fmaf(B.w, U[1], C.x * U[2]));
    const float buy = fmaf(B.w, U[0], fmaf(B.y, U[1], C.y * U[2]));
    const float buz = fmaf(C.x, U[0], fmaf(C.y, U[1], B.z * U[2]));
    const float s7 = fmaf(dx, qx, fmaf(dy, qy, fmaf(dz, qz, C.z))) * ri7;
    const float uq = fmaf(U[0], qx, fmaf(U[1], qy, U[2] * qz));
    const float m3 = A.w * ri3;
    const float cu = fmaf(-2.5f, s7, m3);
    const float cb = -5.f * (ud * ri7);
    const float cd = fmaf(ud, fmaf(-3.f, m3, 17.5f * s7) * ri2, -5.f * (uq * ri7));
    w[0] = fmaf(cu, U[0], fmaf(cd, dx, fmaf(bux, ri5, cb * qx)));
    w[1] = fmaf(cu, U[1], fmaf(cd, dy, fmaf(buy, ri5, cb * qy)));
    w[2] = fmaf(cu, U[2], fmaf(cd, dz, fmaf(buz, ri5, cb * qz)));
    c.w[0] += w[0]; c.w[1] += w[1]; c.w[2] += w[2];
    c.M = fmaf(ud, ri3, c.M);
    c.t = fmaf(ud, ri5, c.t);
    const float h = 0.5f * cb;
    const float vx = fmaf(h, dx, ri5 * U[0]), vy = fmaf(h, dy, ri5 * U[1]),
                vz = fmaf(h, dz, ri5 * U[2]);
    c.Q[0] = fmaf(vx, dx, c.Q[0]);
    c.Q[1] = fmaf(vy, dy, c.Q[1]);
    c.Q[2] = fmaf(vz, dz, c.Q[2]);
    c.Q[3] = fmaf(vx, dy, fmaf(vy, dx, c.Q[3]));
    c.Q[4] = fmaf(vx, dz, fmaf(vz, dx, c.Q[4]));
    c.Q[5] = fmaf(vy, dz, fmaf(vz, dy, c.Q[5]));
}

// dL/dQ of the six stored entries from the sums of pc_adj.
__device__ __forceinline__ void pc_adj_finish(float *sQ, float st) {
    const float t = -1.5f * st;
    sQ[0] = fmaf(-3.f, sQ[0], t);
    sQ[1] = fmaf(-3.f, sQ[1], t);
    sQ[2] = fmaf(-3.f, sQ[2], t);
    sQ[3] *= -3.f;
    sQ[4] *= -3.f;
    sQ[5] *= -3.f;
}

// Adjoint of one particle-particle term: F = m d r^-3, J = m (I r^-3 - 3 d d^T r^-5).
template <bool kEps0>
__device__ __forceinline__ void pp_adj(const float *T, const float *U, const float4 &P,
                                       float eps2, float w[3], float &gm) {
    const float dx = P.x - T[0], dy = P.y - T[1], dz = P.z - T[2];
    const float r2 = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, eps2)));
    float ri = rsqv(r2);
    if (kEps0) ri = r2 > 0.f ? ri : 0.f;
    const float ri2 = ri * ri, ri3 = ri * ri2, ri5 = ri3 * ri2;
    const float ud = fmaf(U[0], dx, fmaf(U[1], dy, U[2] * dz));
    const float c1 = P.w * ri3, c2 = -3.f * P.w * ud * ri5;
    w[0] = fmaf(c1, U[0], c2 * dx);
    w[1] = fmaf(c1, U[1], c2 * dy);
    w[2] = fmaf(c1, U[2], c2 * dz);
    gm = ud * ri3;
}

// Sum of v over the 64 lanes, returned uniform: DPP inclusive scan (row
// shifts, then row broadcasts), lane 63's value read into a scalar.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ float dpp_add(float s) {
    return s + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s), kCtrl, kRowMask,
                                                          0xf, false));
}
__device__ __forceinline__ float wave_total(float v) {
    v = dpp_add<0x111, 0xf>(v);  // row_shr:1
    v = dpp_add<0x112, 0xf>(v);  // row_shr:2
    v = dpp_add<0x114, 0xf>(v);  // row_shr:4
    v = dpp_add<0x118, 0xf>(v);  // row_shr:8
    v = dpp_add<0x142, 0xa>(v);  // row_bcast:15 -> rows 1, 3
    v = dpp_add<0x143, 0xc>(v);  // row_bcast:31 -> rows 2, 3
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

constexpr uint32_t kTile = 16;            // targets of one accumulator tile
constexpr uint32_t kTiles = 2;            // tiles taken at once
constexpr uint32_t kTurn = 32 * kCellAdj; // values turned through LDS at once

struct VjpLds {
    float4 tp[64];  // the group's targets: position, u_x
    float2 tu[64];  // u_y, u_z
    union {
        float turn[kTurn];              // sums of a chunk on their way to the atomics
        float4 tsum[kTile * kTiles];    // target sums of a flush
    };
    TravLds T;
};

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Target sums of up to kTiles x kTile targets: d[tile][k] is component k, row
// t of a tile in lanes 16 (t / 4) .. + 15, register t % 4.
struct TargetSums {
    f32x4 d[kTiles][3];
};

// w of target `row` of the tile (sel: one in the lanes of that row, else zero)
__device__ __forceinline__ void add_target(f32x4 d[3], float sel, const float w[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) d[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(sel, w[k], d[k], 0, 0, 0);
}

// sel of the next row: its lanes rotated by one inside each row of 16
__device__ __forceinline__ float next_row(float sel) {
    return __int_as_float(
        __builtin_amdgcn_update_dpp(0, __float_as_int(sel), 0x121, 0xf, 0xf, false));
}

// Whether every sum is finite.
__device__ __forceinline__ bool sums_finite(const TargetSums &s) {
    float z = 0.f;
#pragma unroll
    for (uint32_t i = 0; i < kTiles; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int r = 0; r < 4; ++r) z = fmaf(s.d[i][k][r], 0.f, z);
    return ballot(!(z == 0.f)) == 0ull;
}

// Sum over the 16 lanes of a DPP row, in its last lane.
__device__ __forceinline__ float row_total(float v) {
    v = dpp_add<0x111, 0xf>(v);
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    return dpp_add<0x118, 0xf>(v);
}

// Take the sums from lane tb + t's target terms g, t < kTiles kTile.
__device__ __forceinline__ void take_targets(const TargetSums &s, VjpLds &L, uint32_t lane,
                                             uint32_t tb, double g[3]) {
#pragma unroll
    for (uint32_t i = 0; i < kTiles; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float x = row_total(s.d[i][0][r]), y = row_total(s.d[i][1][r]),
                        z = row_total(s.d[i][2][r]);
            if ((lane & 15u) == 15u)
                L.tsum[i * kTile + (lane >> 4) * 4u + (uint32_t)r] = make_float4(x, y, z, 0.f);
        }
    wave_sync();
    if (lane - tb < kTiles * kTile) {
        const float4 o = L.tsum[lane - tb];
        g[0] -= o.x; g[1] -= o.y; g[2] -= o.z;
    }
    wave_sync();
}

template <bool kEps0>
__device__ void vjp_group(const VjpArgs &a, uint32_t g, uint32_t w, uint32_t lane, VjpLds &L,
                          uint32_t *spill) {
    const uint32_t gb = a.gbeg[g];
    const uint32_t gn = a.gbeg[g + 1] - gb;
    if (gn == 0u || gn > 64u) {
        if (lane == 0) atomicOr(a.status, kStOverflow);
        return;
    }
    const uint32_t logw = group_logw(a.split, gn);
    if (w >> logw) return;  // fewer waves share this group
    const uint32_t xcd = xcc_id();
    double *const lcx = a.lcell + xcd * a.lstride;
    double *const gsx = a.gsrc + xcd * a.gstride;
    const uint32_t hk = xcd + kXcd * ((blockIdx.x / kXcd) % (kHotCopies / kXcd));
    double *const lhx = a.lhot + hk * kHotCopy;
    const bool own = lane < gn;
    const uint32_t ti = gb + (own ? lane : 0u);
    const float4 me = a.xyzm[ti];
    const GroupBox b = group_box(me, own);
    const float4 mu = a.u[ti];
    L.tp[lane] = make_float4(me.x, me.y, me.z, mu.x);
    L.tu[lane] = make_float2(mu.y, mu.z);
    double gt[3] = {0.0, 0.0, 0.0};  // target terms of lane t's target

    // one trip: target t's position and cotangent
    auto target = [&](uint32_t t, float T[3], float U[3]) {
        const float4 p = L.tp[t];
        const float2 q = L.tu[t];
        T[0] = p.x; T[1] = p.y; T[2] = p.z;
        U[0] = p.w; U[1] = q.x; U[2] = q.y;
    };
    // all trips of targets [tb, tb + kTiles kTile): pair(t, w) evaluates one
    auto trips = [&](uint32_t tb, TargetSums &ts, auto &&pair) {
#pragma unroll
        for (uint32_t i = 0; i < kTiles; ++i) {
            const uint32_t t0 = tb + i * kTile, t1 = gn < t0 + kTile ? gn : t0 + kTile;
            float sel = (lane & 15u) == 0u ? 1.f : 0.f;
            for (uint32_t t = t0; t < t1; ++t) {
                float wv[3];
                pair(t, wv);
                add_target(ts.d[i], sel, wv);
                sel = next_row(sel);
            }
        }
    };
    // the target side of a flush whose sums are not all finite, by lane sums
    auto lane_sums = [&](uint32_t tb, auto &&pair) {
        for (uint32_t t = tb; t < gn && t < tb + kTiles * kTile; ++t) {
            float wv[3];
            pair(t, wv);
            const float x = wave_total(wv[0]), y = wave_total(wv[1]), z = wave_total(wv[2]);
            if (lane == t) {
                gt[0] -= x; gt[1] -= y; gt[2] -= z;
            }
        }
    };

    // More targets than the tiles hold at once: their sums are taken after each
    // chunk, so that a source's sums still leave once (else once per list).
    const bool wide = gn > kTiles * kTile;

    // particle-cell list; lanes past it hold a null cell (zero mass and
    // moments, far away)
    auto flush_pc = [&](uint32_t n) {
        float4 A, B, C;
        auto load = [&](uint32_t base) {
            A = make_float4(1e18f, 1e18f, 1e18f, 0.f);
            B = C = make_float4(0.f, 0.f, 0.f, 0.f);
            if (base + lane < n) {
                const uint32_t c = L.T.pcidx[base + lane];
                A = a.P0[c];
                B = a.P1[c];
                C = a.P2[c];
                const float tr = 2.f * C.z;  // the trace into the quadrupole
                B.x += tr; B.y += tr; B.z += tr;
                C.z = tr * a.eps2;
            }
        };
        CellSums cs;
        auto pair = [&](uint32_t t, float wv[3]) {
            float T[3], U[3];
            target(t, T, U);
            pc_adj(T, U, A, B, C, a.eps2, wv, cs);
        };
        TargetSums ts{};
        for (uint32_t base = 0; base < n; base += kChunk) {
            const uint32_t m = n - base < (uint32_t)kChunk ? n - base : (uint32_t)kChunk;
            load(base);
            cs = CellSums{};
            for (uint32_t tb = 0; tb < gn; tb += kTiles * kTile) {
                if (wide) ts = TargetSums{};
                trips(tb, ts, pair);
                if (!wide) continue;
                const CellSums keep = cs;
                if (sums_finite(ts)) take_targets(ts, L, lane, tb, gt);
                else lane_sums(tb, pair);
                cs = keep;
            }
            pc_adj_finish(cs.Q, cs.t);
            const float v[kCellAdj] = {cs.M,    cs.w[0], cs.w[1], cs.w[2], cs.Q[0],
                                       cs.Q[1], cs.Q[2], cs.Q[3], cs.Q[4], cs.Q[5]};
            for (uint32_t half = 0; half < m; half += 32u) {
                wave_sync();
                if ((lane & 32u) == half) {
#pragma unroll
                    for (uint32_t q = 0; q < kCellAdj; ++q)
                        L.turn[(lane & 31u) * kCellAdj + q] = v[q];
                }
                wave_sync();
#pragma unroll
                for (uint32_t r = 0; r < kTurn / 64u; ++r) {
                    const uint32_t f = r * 64u + lane, k = f / kCellAdj, q = f - k * kCellAdj;
                    if (half + k < m) {
                        const uint32_t c = L.T.pcidx[base + half + k];
                        double *lc = c < kHotCells ? lhx : lcx;
                        add_l2(lc + (size_t)c * kCellAdj + q, (double)L.turn[f]);
                    }
                }
            }
            wave_sync();
        }
        if (wide) return;
        if (sums_finite(ts)) {
            take_targets(ts, L, lane, 0u, gt);
        } else {
            for (uint32_t base = 0; base < n; base += kChunk) {
                load(base);
                lane_sums(0u, pair);
            }
        }
        wave_sync();
    };
    // particle-particle list; the self pair contributes nothing
    auto flush_pp = [&](uint32_t n) {
        float4 P;
        uint32_t j;
        auto load = [&](uint32_t base) {
            P = make_float4(1e18f, 1e18f, 1e18f, 0.f);
            j = kNone;
            if (base + lane < n) {
                j = L.T.ppidx[base + lane];
                P = a.xyzm[j];
            }
        };
        float4 s;  // the source's sums
        auto pair = [&](uint32_t t, float wv[3]) {
            float T[3], U[3], gm;
            target(t, T, U);
            pp_adj<kEps0>(T, U, P, a.eps2, wv, gm);
            if (gb + t == j) wv[0] = wv[1] = wv[2] = gm = 0.f;
            s.x += wv[0]; s.y += wv[1]; s.z += wv[2]; s.w += gm;
        };
        TargetSums ts{};
        for (uint32_t base = 0; base < n; base += kChunk) {
            const uint32_t m = n - base < (uint32_t)kChunk ? n - base : (uint32_t)kChunk;
            load(base);
            s = make_float4(0.f, 0.f, 0.f, 0.f);
            for (uint32_t tb = 0; tb < gn; tb += kTiles * kTile) {
                if (wide) ts = TargetSums{};
                trips(tb, ts, pair);
                if (!wide) continue;
                const float4 keep = s;
                if (sums_finite(ts)) take_targets(ts, L, lane, tb, gt);
                else lane_sums(tb, pair);
                s = keep;
            }
            wave_sync();
            reinterpret_cast<float4 *>(L.turn)[lane] = s;
            wave_sync();
#pragma unroll
            for (uint32_t r = 0; r < 4u; ++r) {
                const uint32_t f = r * 64u + lane, k = f >> 2;
                if (k < m) add_l2(gsx + 4ull * L.T.ppidx[base + k] + (f & 3u), (double)L.turn[f]);
            }
            wave_sync();
        }
        if (wide) return;
        if (sums_finite(ts)) {
            take_targets(ts, L, lane, 0u, gt);
        } else {
            for (uint32_t base = 0; base < n; base += kChunk) {
                load(base);
                lane_sums(0u, pair);
            }
        }
        wave_sync();
    };

    uint32_t cnt_pc, cnt_pp;
    const TreeView tv{a.wA, a.wN, a.ring, a.status};
    traverse<false, true>(tv, b, lane, L.T, spill, cnt_pc, cnt_pp, flush_pc, flush_pp,
                            Share{w, logw});
    if (own) {
        double *gs = gsx + 4ull * ti;
#pragma unroll
        for (int k = 0; k < 3; ++k) add_l2(gs + k, gt[k]);
    }
    wave_sync();
}

template <bool kEps0>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_walk_vjp(VjpArgs a) {
    __shared__ VjpLds L;
    const uint32_t lane = threadIdx.x;
    uint32_t *spill = a.spill + (size_t)blockIdx.x * kStackMax;
    for_each_group(*a.ngroups, a.work, lane, a.split.logw, [&](uint32_t g, uint32_t w) {
        vjp_group<kEps0>(a, g, w, lane, L, spill);
    });
}

// ---- moments part, combination and unsorting --------------------------------

// What the walk needs, in one launch (six of 4 to 5 us each on small sets):
// opening radii and work counters, the accumulators' zeros, the leaf of every
// particle, the cotangents in sorted order.
__global__ __launch_bounds__(256) void k_vjp_prep(Cells c, float theta, uint32_t *work,
                                                  const float *__restrict__ u,
                                                  const uint32_t *__restrict__ cid, uint32_t n,
                                                  float4 *__restrict__ us, uint32_t *leafof,
                                                  double *lcell, uint64_t lstride, double *gsrc,
                                                  uint64_t gstride, double *lhot) {
    if (blockIdx.x == 0) zero_walk(work, nullptr);
    const uint32_t nc = c.ls[kLevels];
    const uint64_t t = (uint64_t)blockIdx.x * 256 + threadIdx.x, step = (uint64_t)gridDim.x * 256;
    for (uint64_t i = t; i < nc; i += step) {
        c.wA[i].w = open_radius2(c.size[i], theta);
        if (c.nchild[i] != 0) continue;
        const uint32_t b = c.begin[i], e = b + c.count[i];
        for (uint32_t j = b; j < e; ++j) leafof[j] = (uint32_t)i;
    }
    for (uint64_t i = t; i < n; i += step) {
        const size_t p = cid[i];
        us[i] = make_float4(u[3 * p], u[3 * p + 1], u[3 * p + 2], 0.f);
    }
    // (cells in the hot copies leave their others unused)
    const uint64_t all = (uint64_t)nc * kCellAdj, hot = (uint64_t)min(nc, kHotCells) * kCellAdj;
    for (uint64_t i = t; i < hot; i += step)
#pragma unroll 8
        for (uint32_t k = 0; k < kHotCopies; ++k) lhot[i + k * kHotCopy] = 0.0;
    for (uint64_t i = hot + t; i < all; i += step)
#pragma unroll
        for (uint32_t k = 0; k < kXcd; ++k) lcell[i + k * lstride] = 0.0;
    for (uint64_t i = t; i < 4ull * n; i += step)
#pragma unroll
        for (uint32_t k = 0; k < kXcd; ++k) gsrc[i + k * gstride] = 0.0;
}

// Fold the copies of the cells' adjoints into copy 0 of lcell.
__global__ __launch_bounds__(256) void k_fold_cells(const uint32_t *ls, double *lcell,
                                                    uint64_t lstride,
                                                    const double *__restrict__ lhot) {
    const uint64_t total = (uint64_t)ls[kLevels] * kCellAdj;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < total;
         i += (uint64_t)gridDim.x * 256) {
        double v = 0.0;
        if (i < (uint64_t)kHotCells * kCellAdj) {
#pragma unroll 8
            for (uint32_t k = 0; k < kHotCopies; ++k) v += lhot[i + k * kHotCopy];
        } else {
#pragma unroll
            for (uint32_t k = 0; k < kXcd; ++k) v += lcell[i + k * lstride];
        }
        lcell[i] = v;
    }
}

// Each particle adds the adjoints of the cells holding it (its leaf and the
// leaf's ancestors), then the total is scaled and added to the caller-order
// outputs.
__global__ __launch_bounds__(256) void k_moments_vjp(Cells c, const float4 *__restrict__ xyzm,
                                                     const uint32_t *__restrict__ leafof,
                                                     const uint32_t *__restrict__ cid,
                                                     const double *__restrict__ lcell,
                                                     const double *__restrict__ gsrc,
                                                     uint64_t gstride, uint32_t n, float coef,
                                                     float *g_pos,
                                                     float *g_mass) {
    const uint32_t k = blockIdx.x * 256 + threadIdx.x;
    if (k >= n) return;
    const float4 p = xyzm[k];
    const double xk = p.x, yk = p.y, zk = p.z, mk = p.w;
    double gx = 0.0, gy = 0.0, gz = 0.0, gm = 0.0;
#pragma unroll
    for (uint32_t x = 0; x < kXcd; ++x) {
        const double2 *g = reinterpret_cast<const double2 *>(gsrc + x * gstride + 4ull * k);
        const double2 a = g[0], b = g[1];
        gx += a.x; gy += a.y; gz += b.x; gm += b.y;
    }
    for (uint32_t cc = leafof[k]; cc != kNone; cc = c.parent[cc]) {
        const double *l = lcell + (size_t)cc * kCellAdj;
        const double lM = l[0], lx = l[1], ly = l[2], lz = l[3];
        const double qxx = l[4], qyy = l[5], qzz = l[6], qxy = l[7], qxz = l[8], qyz = l[9];
        const double M = c.M[cc];
        const double sx = xk - c.S[3 * (size_t)cc] / M, sy = yk - c.S[3 * (size_t)cc + 1] / M,
                     sz = zk - c.S[3 * (size_t)cc + 2] / M;
        const double Lx = 2.0 * qxx * sx + qxy * sy + qxz * sz;
        const double Ly = qxy * sx + 2.0 * qyy * sy + qyz * sz;
        const double Lz = qxz * sx + qyz * sy + 2.0 * qzz * sz;
        const double f = mk / M;
        gx += f * lx + mk * Lx;
        gy += f * ly + mk * Ly;
        gz += f * lz + mk * Lz;
        const double sLs = qxx * sx * sx + qyy * sy * sy + qzz * sz * sz + qxy * sx * sy +
                           qxz * sx * sz + qyz * sy * sz;
        gm += lM + (lx * sx + ly * sy + lz * sz) / M + sLs;
    }
    const size_t o = cid[k];
    if (g_pos) {
        g_pos[3 * o] += (float)(coef * gx);
        g_pos[3 * o + 1] += (float)(coef * gy);
        g_pos[3 * o + 2] += (float)(coef * gz);
    }
    if (g_mass) g_mass[o] += (float)(coef * gm);
}

// Waves per group of the adjoint walk, as in the force walk; its sums leave by
// atomics, which a split does not multiply, so a small set is split further.
// Disk + halo at theta 0.4 / 0.6, walk in us, all groups alike (the best number
// of waves) / this rule: n = 1000 51 / 51 (Plummer); 4096 156 / 128; 16384 511 /
// 468; 65536 1650 / 1484 and 759 / 676; 131072 - and 1452 / 1276; 262144 4881 /
// 4610 (one wave 6001); 500000 - and 4401 / 4082; 1M 17816 / 16990; 2M 34749 /
// 34514 and 16322 / 16167; 7M equal.  The lines: 16 waves at 1000 take 57, at
// 65536 1566 and 802; four at 500000 4348.
static Split vjp_split(int64_t n) {
    if (n <= 2048) return {3u, 0u, 0u};
    if (n <= 32768) return {4u, 32u, 16u};
    if (n <= 360448) return {2u, 32u, 16u};
    return {1u, 40u, 0u};
}

void launch_walk_vjp(bh_ctx *c, float theta, float eps, const float *u, float coef, float *g_pos,
                     float *g_mass, hipStream_t st) {
    const uint32_t n = (uint32_t)c->n;
    const uint32_t nb = cdiv(n, 256);
    const uint64_t lstride = kCellAdj * (uint64_t)c->cap_cells, gstride = 4ull * (uint64_t)c->nmax;
    const uint32_t *ls = c->cells.ls;
    const uint32_t grid = std::min<uint32_t>(cdiv(4ull * n, 256), 4096u);
    hipLaunchKernelGGL(k_vjp_prep, dim3(grid), dim3(256), 0, st, c->cells, theta, c->work, u,
                       (const uint32_t *)c->st[c->cur].cid, n, c->usort, c->leafof, c->lcell,
                       lstride, c->gsrc, gstride, c->lhot);
    VjpArgs a;
    a.xyzm = c->xyzm; a.u = c->usort;
    a.wA = c->cells.wA; a.wN = c->cells.wN;
    a.P0 = c->cells.P0; a.P1 = c->cells.P1; a.P2 = c->cells.P2;
    a.gbeg = c->groups.begin; a.ngroups = c->groups.count_dev;
    a.work = c->work; a.spill = c->spill; a.status = c->status;
    a.ring = c->walk_small_stack ? 192u : (uint32_t)kRing;
    a.lcell = c->lcell; a.gsrc = c->gsrc; a.lhot = c->lhot;
    a.lstride = lstride; a.gstride = gstride;
    a.eps2 = eps * eps;
    record_event(c, 8, st);
    a.split = vjp_split(c->n);
    const dim3 walks(c->walk_grid);
    if (eps == 0.f) hipLaunchKernelGGL(k_walk_vjp<true>, walks, dim3(64), 0, st, a);
    else hipLaunchKernelGGL(k_walk_vjp<false>, walks, dim3(64), 0, st, a);
    record_event(c, 9, st);
    hipLaunchKernelGGL(k_fold_cells, dim3(std::min<uint32_t>(cdiv(4ull * n, 256), 2048u)),
                       dim3(256), 0, st, ls, c->lcell, lstride, (const double *)c->lhot);
    hipLaunchKernelGGL(k_moments_vjp, dim3(nb), dim3(256), 0, st, c->cells,
                       (const float4 *)c->xyzm, (const uint32_t *)c->leafof,
                       (const uint32_t *)c->st[c->cur].cid, (const double *)c->lcell,
                       (const double *)c->gsrc, gstride, n, coef, g_pos, g_mass);
}

// y += a x over n [3]-vectors (the drift's transpose in the adjoint step)
__global__ __launch_bounds__(256) void k_axpy3(const float *__restrict__ x, float *y, float a,
                                               uint32_t n3) {
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < n3) y[i] = fmaf(a, x[i], y[i]);
}

void launch_axpy3(const float *x, float *y, float a, uint32_t n, hipStream_t st) {
    hipLaunchKernelGGL(k_axpy3, dim3(cdiv(3ull * n, 256)), dim3(256), 0, st, x, y, a, 3u * n);
}

}  // namespace bh
