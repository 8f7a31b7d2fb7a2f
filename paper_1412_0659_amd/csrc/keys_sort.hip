// Bounding box, Morton keys, LSD radix sort of (key, index) and the gather of
// the particle state into key order (Sec. III.B.1: keys computed from the
// bounding box; Table II "Sorting SFC").
//
// Keys: 21 bits per axis, x the high bit of each 3-bit digit,
//   q = min(trunc(fl32(fl32(x - lo) * scale)), 2^21 - 1),
//   scale = fl32(2^21 / side) with the division in FP64,
// built with contraction off so the FP32 quantisation is exactly the one
// written above.
#include "bh_internal.h"
#include "wave.h"

namespace bh {

constexpr int kBoxThreads = 256;
constexpr int kBoxBlocks = 1024;

struct Extent {
    float lo[3], hi[3];
};

__device__ __forceinline__ Extent no_extent() {
    return Extent{{INFINITY, INFINITY, INFINITY}, {-INFINITY, -INFINITY, -INFINITY}};
}

// Particle i of s joins e; bit mask of what is wrong with it.
__device__ __forceinline__ uint32_t join_particle(const Source &s, uint32_t i, Extent &e,
                                                  float p[3]) {
    const size_t o = (size_t)i * s.ps;
    p[0] = s.x[o]; p[1] = s.y[o]; p[2] = s.z[o];
    uint32_t bad = isfinite(p[0]) && isfinite(p[1]) && isfinite(p[2]) ? 0u : kStNonFinite;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        e.lo[k] = fminf(e.lo[k], p[k]);
        e.hi[k] = fmaxf(e.hi[k], p[k]);
    }
    if (s.check) {
        const float m = s.m[i];
        if (!(m > 0.f) || !isfinite(m)) bad |= kStMass;
        if (s.vx) {
            const size_t v = (size_t)i * s.vs;
            if (!(isfinite(s.vx[v]) && isfinite(s.vy[v]) && isfinite(s.vz[v]))) bad |= kStNonFinite;
        }
    }
    return bad;
}

__device__ __forceinline__ void wave_extent(Extent &e) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        e.lo[k] = wave_min(e.lo[k]);
        e.hi[k] = wave_max(e.hi[k]);
    }
}

__global__ __launch_bounds__(kBoxThreads) void k_bbox_partial(Source s, uint32_t n, float *part,
                                                              uint32_t *status) {
    __shared__ Extent lds[kBoxThreads / 64];
    Extent e = no_extent();
    uint32_t bad = 0;
    for (uint32_t i = blockIdx.x * kBoxThreads + threadIdx.x; i < n;
         i += gridDim.x * kBoxThreads) {
        float p[3];
        bad |= join_particle(s, i, e, p);
    }
    if (bad) atomicOr(status, bad);
    wave_extent(e);
    if (lane_id() == 0) lds[threadIdx.x >> 6] = e;
    __syncthreads();
    if (threadIdx.x < 6) {
        const uint32_t k = threadIdx.x % 3u;
        const bool lo = threadIdx.x < 3u;
        float v = lo ? lds[0].lo[k] : lds[0].hi[k];
        for (int w = 1; w < kBoxThreads / 64; ++w)
            v = lo ? fminf(v, lds[w].lo[k]) : fmaxf(v, lds[w].hi[k]);
        part[blockIdx.x * 6 + threadIdx.x] = v;
    }
}

// The key box (lo xyz, side, scale) of particles of extent e.  fixed == 0: the
// cube of side = largest extent at the minimum corner.  fixed == 1: the
// caller's box (flo, fside), and kStOutside is latched (by the thread that is
// asked to) when on some axis a particle lies below flo or has
// fl32(x - flo) > fside (the difference the keys quantise).
struct FixedBox {
    int fixed;
    float lo[3], side;
};

__device__ __forceinline__ void key_box(const Extent &e, const FixedBox &f, bool latch,
                                        uint32_t *status, float box[5]) {
    if (f.fixed) {
        bool out = false;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            out = out || e.lo[k] < f.lo[k] || e.hi[k] - f.lo[k] > f.side;
            box[k] = f.lo[k];
        }
        if (latch && out) atomicOr(status, kStOutside);
        box[3] = f.side;
    } else {
        float side = 0.f;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float d = e.hi[k] - e.lo[k];
            if (d > side) side = d;
            box[k] = e.lo[k];
        }
        if (side == 0.f) side = 1.f;
        box[3] = side;
    }
    box[4] = (float)(2097152.0 / (double)box[3]);
}

// The extent of the nb partials, by one wave.
__device__ __forceinline__ Extent join_partials(const float *__restrict__ part, uint32_t nb,
                                                uint32_t lane) {
    Extent e = no_extent();
    for (uint32_t b = lane; b < nb; b += 64) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            e.lo[k] = fminf(e.lo[k], part[6 * b + k]);
            e.hi[k] = fmaxf(e.hi[k], part[6 * b + 3 + k]);
        }
    }
    wave_extent(e);
    return e;
}

__global__ __launch_bounds__(64) void k_bbox_final(const float *__restrict__ part, uint32_t nb,
                                                   float *box, FixedBox f, uint32_t *status) {
    const Extent e = join_partials(part, nb, threadIdx.x);
    if (threadIdx.x == 0) {
        float b[5];
        key_box(e, f, true, status, b);
        for (int k = 0; k < 5; ++k) box[k] = b[k];
    }
}

static FixedBox fixed_box(const bh_ctx *c) {
    return FixedBox{c->fixed_box ? 1 : 0, {c->box_lo[0], c->box_lo[1], c->box_lo[2]}, c->box_side};
}

static uint32_t launch_bbox_partial(bh_ctx *c, const Source &s, uint32_t n, hipStream_t st) {
    uint32_t nb = cdiv(n, kBoxThreads * 8);
    if (nb > kBoxBlocks) nb = kBoxBlocks;
    hipLaunchKernelGGL(k_bbox_partial, dim3(nb), dim3(kBoxThreads), 0, st, s, n, c->box_part,
                       c->status);
    return nb;
}

// 21 bits -> every third bit of a 63-bit word
__device__ __forceinline__ uint64_t spread3(uint32_t v) {
    uint64_t x = v & 0x1fffffu;
    x = (x | (x << 32)) & 0x001f00000000ffffull;
    x = (x | (x << 16)) & 0x001f0000ff0000ffull;
    x = (x | (x << 8)) & 0x100f00f00f00f00full;
    x = (x | (x << 4)) & 0x10c30c30c30c30c3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

__device__ __forceinline__ uint32_t quantise(float v, float lo, float scale) {
    float t = v - lo;
    float u = t * scale;
    if (!(u > 0.f)) return 0u;  // below a caller-given box: the first cell
    uint32_t q = (uint32_t)u;
    return q > 0x1fffffu ? 0x1fffffu : q;
}

// 63-bit key of a position: the quantised coordinates interleaved (Morton), or
// their Peano-Hilbert transposed index interleaved the same way
struct KeyBox {
    float lo0, lo1, lo2, scale;
};

template <bool kPH>
__device__ __forceinline__ uint64_t key_of(float x, float y, float z, const KeyBox &b) {
    uint32_t X[3] = {quantise(x, b.lo0, b.scale), quantise(y, b.lo1, b.scale),
                     quantise(z, b.lo2, b.scale)};
    if (kPH) ph_encode(X, kKeyBits);
    return (spread3(X[0]) << 2) | (spread3(X[1]) << 1) | spread3(X[2]);
}

template <bool kPH>
__global__ __launch_bounds__(256) void k_keys(Source s, uint32_t n, const float *__restrict__ box,
                                              uint64_t *__restrict__ key,
                                              uint32_t *__restrict__ idx) {
    uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const size_t o = (size_t)i * s.ps;
    key[i] = key_of<kPH>(s.x[o], s.y[o], s.z[o], KeyBox{box[0], box[1], box[2], box[4]});
    idx[i] = i;
}

static void launch_keys(bh_ctx *c, const Source &s, uint32_t n, hipStream_t st) {
    if (c->p.curve == 1)
        hipLaunchKernelGGL(k_keys<true>, dim3(cdiv(n, 256)), dim3(256), 0, st, s, n,
                           (const float *)c->box, c->sort.key[0], c->sort.idx[0]);
    else
        hipLaunchKernelGGL(k_keys<false>, dim3(cdiv(n, 256)), dim3(256), 0, st, s, n,
                           (const float *)c->box, c->sort.key[0], c->sort.idx[0]);
}

// ---- gather the state into sorted order ------------------------------------

// Particle s of a becomes sorted particle i of b.  Read from the caller's
// arrays a particle in random order costs two or three cache lines instead of
// the eight of a copy as separate arrays.
__device__ __forceinline__ void move_particle(const Source &a, uint32_t s, const State &b,
                                              uint32_t i, float4 *__restrict__ xyzm) {
    const size_t o = (size_t)s * a.ps;
    const float px = a.x[o], py = a.y[o], pz = a.z[o], pm = a.m[s];
    float vx = 0.f, vy = 0.f, vz = 0.f;
    if (a.vx) {
        const size_t v = (size_t)s * a.vs;
        vx = a.vx[v]; vy = a.vy[v]; vz = a.vz[v];
    }
    xyzm[i] = make_float4(px, py, pz, pm);
    b.cid[i] = a.cid ? a.cid[s] : s;
    if (!b.x) return;  // (tree_force_static keeps no state)
    b.x[i] = px;
    b.y[i] = py;
    b.z[i] = pz;
    b.m[i] = pm;
    b.vx[i] = vx;
    b.vy[i] = vy;
    b.vz[i] = vz;
    if (b.x64) {
        b.x64[i] = a.x64 ? a.x64[s] : (double)px;
        b.y64[i] = a.y64 ? a.y64[s] : (double)py;
        b.z64[i] = a.z64 ? a.z64[s] : (double)pz;
    }
}

__global__ __launch_bounds__(256) void k_gather(const uint32_t *__restrict__ idx, uint32_t n,
                                                Source a, State b, float4 *__restrict__ xyzm) {
    uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) move_particle(a, idx[i], b, i, xyzm);
}

static void launch_gather(bh_ctx *c, const Source &s, uint32_t n, hipStream_t st) {
    hipLaunchKernelGGL(k_gather, dim3(cdiv(n, 256)), dim3(256), 0, st,
                       (const uint32_t *)c->sort.idx[0], n, s, c->st[c->cur ^ 1], c->xyzm);
    c->cur ^= 1;
}

// ---- block sort and merges ------------------------------------------------
//
// Sets of up to kMergeMax particles.  k_sort_block computes the keys of a tile
// of 1024 kRounds particles and sorts them in LDS, all eight digits in one
// launch (stable, least significant first: the order of equal keys is input
// order).  Up to kRankMax particles k_sort_rank then finds every particle's
// place among all tiles at once and moves it there; above, k_sort_merge merges
// pairs of sorted runs, ties from the earlier run first.  A block of a merge
// takes kMergeTile consecutive outputs, finds where they begin and end in both
// runs by a 64-way search on the diagonal (one wave per end), and merges them
// in LDS.
//
// Bound: latency on small sets (one launch up to 1024 particles, two up to
// 12288, then one per doubling, where the radix passes over memory below take five launches
// per digit), 24 B per particle and merge on larger ones.  Measured, bounding
// box, keys, sort and gather of a set in random order, in us, these against
// the radix passes: n = 1000: 18 / 135; 4096: 31 / 148; 16384: 54 / 192; 65536:
// 73 / 213; 500000: 136 / 257; 1M: 192 / 297; 2M: 312 / 373; 3M: 460 / 529; 4M:
// 625 / 615; 8M: 1235 / 1105.
constexpr uint32_t kMergeMax = 3u << 20;

constexpr int kSortThreads = 1024;
constexpr int kSortWaves = kSortThreads / 64;

// nb == 0: every block finds the bounding box of all particles itself (and
// block 0 checks them); else it folds the nb partials.  Block 0 writes box.
// xyzm: the set is one tile, whose particles move to their places in dst here
// (a launch of its own costs 4.5 us of 98 at n = 1000).
template <bool kPH, int kRounds>
__global__ __launch_bounds__(kSortThreads) void k_sort_block(
    Source s, uint32_t n, const float *__restrict__ part, uint32_t nb, FixedBox fb, float *box,
    uint32_t *status, uint64_t *__restrict__ key_out, uint32_t *__restrict__ idx_out, State dst,
    float4 *__restrict__ xyzm, bool clear) {
    constexpr uint32_t kTile = kSortThreads * kRounds;
    __shared__ uint64_t skey[kTile];
    __shared__ uint16_t sidx[kTile];
    __shared__ uint32_t cnt[kSortWaves][256];
    __shared__ uint32_t wsum[4];
    __shared__ Extent ext[kSortWaves];
    const uint32_t w = threadIdx.x >> 6, lane = lane_id();
    const uint32_t t0 = blockIdx.x * kTile;
    const uint32_t p0 = w * 64u * kRounds + lane;  // this wave's positions: p0 + 64 r
    const uint64_t lt = mask_lt(lane);
    float px[kRounds], py[kRounds], pz[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const uint32_t i = t0 + p0 + 64u * r;
        px[r] = py[r] = pz[r] = 0.f;
        if (i < n) {
            const size_t o = (size_t)i * s.ps;
            px[r] = s.x[o]; py[r] = s.y[o]; pz[r] = s.z[o];
        }
    }
    Extent e = no_extent();
    uint32_t bad = 0;
    if (nb == 0) {
        Source all = s;
        all.check = s.check && blockIdx.x == 0;
        for (uint32_t i = threadIdx.x; i < n; i += kSortThreads) {
            float p[3];
            bad |= join_particle(all, i, e, p);
        }
    }
    if (nb == 0) {
        if (clear) {  // the status words hold an earlier call's; only block 0 writes them here
            if (blockIdx.x == 0 && threadIdx.x < 4u) status[threadIdx.x] = 0u;
            __syncthreads();
        }
        if (bad && blockIdx.x == 0) atomicOr(status, bad);
        wave_extent(e);
        if (lane == 0) ext[w] = e;
        __syncthreads();
        e = ext[lane % kSortWaves];
        wave_extent(e);
    } else {
        if (w == 0) {
            e = join_partials(part, nb, lane);
            if (lane == 0) ext[0] = e;
        }
        __syncthreads();
        e = ext[0];
    }
    float b[5];
    key_box(e, fb, blockIdx.x == 0 && threadIdx.x == 0, status, b);
    if (blockIdx.x == 0 && threadIdx.x == 0)
        for (int k = 0; k < 5; ++k) box[k] = b[k];
    const KeyBox kb{b[0], b[1], b[2], b[4]};
    uint64_t kk[kRounds];
    uint32_t vv[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        // past the end: a key above all others, so it stays behind them
        kk[r] = t0 + p0 + 64u * r < n ? key_of<kPH>(px[r], py[r], pz[r], kb) : ~0ull;
        vv[r] = p0 + 64u * r;
    }
    for (uint32_t shift = 0; shift < 64u; shift += 8u) {
        for (uint32_t k = threadIdx.x; k < kSortWaves * 256u; k += kSortThreads) (&cnt[0][0])[k] = 0u;
        __syncthreads();
        uint32_t rk[kRounds];
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const uint32_t d = (uint32_t)(kk[r] >> shift) & 255u;
            uint64_t peers = ~0ull;  // lanes of this round holding the same digit
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const bool bit = (d >> b) & 1u;
                const uint64_t m = ballot(bit);
                peers &= bit ? m : ~m;
            }
            const uint32_t before = (uint32_t)__popcll(peers & lt);
            const uint32_t run = cnt[w][d];
            wave_sync();
            if (before == 0) cnt[w][d] = run + (uint32_t)__popcll(peers);
            wave_sync();
            rk[r] = run + before;
        }
        __syncthreads();
        uint32_t tot = 0, inc = 0;
        if (threadIdx.x < 256) {  // waves 0..3: one digit per thread
#pragma unroll
            for (int k = 0; k < kSortWaves; ++k) tot += cnt[k][threadIdx.x];
            inc = wave_incl_scan(tot, lane);
            if (lane == 63) wsum[w] = inc;
        }
        __syncthreads();
        if (threadIdx.x < 256) {
            uint32_t run = inc - tot;
            for (uint32_t k = 0; k < w; ++k) run += wsum[k];
#pragma unroll
            for (int k = 0; k < kSortWaves; ++k) {
                const uint32_t c = cnt[k][threadIdx.x];
                cnt[k][threadIdx.x] = run;
                run += c;
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const uint32_t lp = cnt[w][(uint32_t)(kk[r] >> shift) & 255u] + rk[r];
            skey[lp] = kk[r];
            sidx[lp] = (uint16_t)vv[r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            kk[r] = skey[p0 + 64u * r];
            vv[r] = sidx[p0 + 64u * r];
        }
    }
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const uint32_t i = t0 + p0 + 64u * r;
        if (i < n) {
            key_out[i] = kk[r];
            idx_out[i] = t0 + vv[r];
            if (xyzm) move_particle(s, t0 + vv[r], dst, i, xyzm);
        }
    }
}

constexpr int kMergeThreads = 256;
constexpr int kMergeItems = 8;
constexpr int kMergeTile = kMergeThreads * kMergeItems;

// Of the first d outputs of the merge of A (na keys) and B (nb keys), ties
// from A first: how many come from A.  One wave, 64 probes a round.
__device__ __forceinline__ uint32_t merge_split(const uint64_t *__restrict__ A, uint32_t na,
                                                const uint64_t *__restrict__ B, uint32_t nb,
                                                uint32_t d, uint32_t lane) {
    uint32_t lo = d > nb ? d - nb : 0u, hi = d < na ? d : na;  // the answer is in [lo, hi]
    while (lo < hi) {
        const uint32_t len = hi - lo, step = (len + 63u) >> 6;
        const uint32_t i = lo + lane * step;  // probe: does output d take A[i]?
        const bool take = i < hi && A[i] <= B[d - 1u - i];
        const uint32_t k = (uint32_t)__popcll(ballot(take));  // (true for the first k probes)
        if (k == 0u) return lo;
        lo = lo + (k - 1u) * step + 1u;
        hi = k < 64u && lo - 1u + step < hi ? lo - 1u + step : hi;
    }
    return lo;
}

// Merge runs of `run` keys in pairs.
__global__ __launch_bounds__(kMergeThreads) void k_sort_merge(
    const uint64_t *__restrict__ key, const uint32_t *__restrict__ idx, uint32_t n, uint32_t run,
    uint64_t *__restrict__ key_out, uint32_t *__restrict__ idx_out) {
    __shared__ uint64_t sk[kMergeTile];
    __shared__ uint32_t si[kMergeTile];
    __shared__ uint32_t split[2];
    const uint32_t o0 = blockIdx.x * kMergeTile;
    const uint32_t a0 = o0 / (2u * run) * (2u * run);  // (run is a multiple of the tile)
    const uint32_t na = min(run, n - a0), nb = min(run, n - a0 - na);
    const uint32_t d0 = o0 - a0, d1 = min(d0 + (uint32_t)kMergeTile, na + nb);
    const uint64_t *A = key + a0, *B = A + na;
    const uint32_t lane = lane_id(), w = threadIdx.x >> 6;
    if (w < 2) {
        const uint32_t s = merge_split(A, na, B, nb, w ? d1 : d0, lane);
        if (lane == 0) split[w] = s;
    }
    __syncthreads();
    const uint32_t i0 = split[0], ca = split[1] - i0, j0 = d0 - i0, m = d1 - d0, cb = m - ca;
    for (uint32_t t = threadIdx.x; t < m; t += kMergeThreads) {
        const uint32_t s = a0 + (t < ca ? i0 + t : na + j0 + (t - ca));
        sk[t] = key[s];
        si[t] = idx[s];
    }
    __syncthreads();
    // this thread's outputs [d, d + kMergeItems) of the m: A part at sk[0, ca), B part behind it
    const uint32_t d = min(threadIdx.x * (uint32_t)kMergeItems, m);
    uint32_t lo = d > cb ? d - cb : 0u, hi = d < ca ? d : ca;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (sk[mid] <= sk[ca + d - 1u - mid]) lo = mid + 1u;
        else hi = mid;
    }
    uint32_t i = lo, j = ca + d - lo;
    uint64_t ok[kMergeItems];
    uint32_t oi[kMergeItems];
#pragma unroll
    for (int t = 0; t < kMergeItems; ++t) {
        const bool va = i < ca, vb = j < m;
        const uint64_t x = va ? sk[i] : ~0ull, y = vb ? sk[j] : ~0ull;
        const bool ta = va && (!vb || x <= y);
        const uint32_t s = ta ? i : (vb ? j : 0u);
        ok[t] = ta ? x : y;
        oi[t] = si[s];
        if (ta) ++i;
        else ++j;
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kMergeItems; ++t) {
        const uint32_t o = threadIdx.x * kMergeItems + t;
        if (o < m) {
            sk[o] = ok[t];
            si[o] = oi[t];
        }
    }
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < m; t += kMergeThreads) {
        key_out[o0 + t] = sk[t];
        idx_out[o0 + t] = si[t];
    }
}

template <int kRounds>
static void launch_sort_block(bh_ctx *c, const Source &s, uint32_t n, uint32_t nb, int dst,
                              hipStream_t st) {
    const dim3 grid(cdiv(n, (uint64_t)kSortThreads * kRounds));
    const State &to = c->st[c->cur ^ 1];
    float4 *xyzm = grid.x == 1 ? c->xyzm : nullptr;
    if (c->p.curve == 1)
        hipLaunchKernelGGL((k_sort_block<true, kRounds>), grid, dim3(kSortThreads), 0, st, s, n,
                           (const float *)c->box_part, nb, fixed_box(c), c->box, c->status,
                           c->sort.key[dst], c->sort.idx[dst], to, xyzm, c->clear_status);
    else
        hipLaunchKernelGGL((k_sort_block<false, kRounds>), grid, dim3(kSortThreads), 0, st, s, n,
                           (const float *)c->box_part, nb, fixed_box(c), c->box, c->status,
                           c->sort.key[dst], c->sort.idx[dst], to, xyzm, c->clear_status);
}

// Sets of up to kRankMax particles: the place of every particle among all runs
// of 1024 in one launch, its place in its own run plus the keys before it in
// each other run (ties from the earlier run first), found by binary searches
// that do not wait for each other; the particle is moved there at once.  The
// sort phase by four / eight / sixteen searches at once, in us: 4099 31.7 / 30.8 /
// 31.7; 8192 42.6 / 40.2 / 41.2.  The line: 12000 particles 53.4 against 57.8 by
// merges, 16384 57.2 against 54.2.
constexpr uint32_t kRankRun = 1024;
constexpr uint32_t kRankAtOnce = 8;  // searches that do not wait for each other
constexpr uint32_t kRankMax = 12 * kRankRun;

__global__ __launch_bounds__(256) void k_sort_rank(const uint64_t *__restrict__ key,
                                                   const uint32_t *__restrict__ idx, uint32_t n,
                                                   Source a, State b, float4 *__restrict__ xyzm,
                                                   uint64_t *__restrict__ key_out) {
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    const uint32_t own = blockIdx.x * 256 / kRankRun, runs = (n + kRankRun - 1u) / kRankRun;
    if (i >= n) return;
    const uint64_t k = key[i];
    uint32_t rank = i - own * kRankRun;
    for (uint32_t q0 = 0; q0 < runs; q0 += kRankAtOnce) {
        uint32_t pos[kRankAtOnce] = {};
#pragma unroll
        for (uint32_t step = kRankRun; step > 0u; step >>= 1) {
#pragma unroll
            for (uint32_t q = 0; q < kRankAtOnce; ++q) {
                const uint32_t r = q0 + q, base = r * kRankRun;
                if (r >= runs || r == own) continue;
                const uint32_t len = min(kRankRun, n - base), e = pos[q] + step;
                const uint64_t v = key[base + min(e, len) - 1u];
                if (e <= len && (r < own ? v <= k : v < k)) pos[q] = e;
            }
        }
#pragma unroll
        for (uint32_t q = 0; q < kRankAtOnce; ++q) rank += pos[q];
    }
    key_out[rank] = k;
    move_particle(a, idx[i], b, rank, xyzm);
}

// Sorted keys into key[0], the particles into st[cur ^ 1].
static void launch_merge_sort(bh_ctx *c, const Source &s, uint32_t n, hipStream_t st) {
    if (n <= kRankMax) {
        const int src = n > kRankRun ? 1 : 0;
        launch_sort_block<1>(c, s, n, 0u, src, st);
        if (src)
            hipLaunchKernelGGL(k_sort_rank, dim3(cdiv(n, 256)), dim3(256), 0, st,
                               (const uint64_t *)c->sort.key[1], (const uint32_t *)c->sort.idx[1],
                               n, s, c->st[c->cur ^ 1], c->xyzm, c->sort.key[0]);
        c->cur ^= 1;
        return;
    }
    // 65536 particles take 73 us with tiles of 2048, 77 with 4096, 95 with 8192
    // (a tile's sort grows with its size, a merge costs 7 us); 1M: 200 / 192 /
    // 203; 3M: 489 / 460 / 479
    const bool small = n <= (1u << 19);
    const uint32_t tile = kSortThreads * (small ? 2u : 4u);
    int passes = 0;
    while (((uint64_t)tile << passes) < n) ++passes;
    int src = passes & 1;
    const uint32_t nb = launch_bbox_partial(c, s, n, st);
    if (small) launch_sort_block<2>(c, s, n, nb, src, st);
    else launch_sort_block<4>(c, s, n, nb, src, st);
    for (int p = 0; p < passes; ++p, src ^= 1)
        hipLaunchKernelGGL(k_sort_merge, dim3(cdiv(n, kMergeTile)), dim3(kMergeThreads), 0, st,
                           (const uint64_t *)c->sort.key[src], (const uint32_t *)c->sort.idx[src],
                           n, tile << p, c->sort.key[src ^ 1], c->sort.idx[src ^ 1]);
    launch_gather(c, s, n, st);
}

// ---- LSD radix sort, 8 bits per pass -------------------------------------
//
// Sets of more than kMergeMax particles.
// A tile is 8192 keys handled by 1024 threads (16 waves x 8 rounds x 64
// lanes); wave w owns the contiguous keys [512 w, 512 w + 512) of the tile,
// in rounds of 64 consecutive keys, so (wave, round, lane) order is input
// order and the ranking below is stable.  Pass structure: per-tile digit
// counts -> one exclusive scan over (digit, tile) -> stable scatter.  A tile
// of 8192 keys gives digit runs of 32 keys on average, so the scatter writes
// mostly whole cache lines (the tile and its reorder buffer, 112 KB of LDS,
// fit one workgroup of gfx950).

constexpr int kSortRounds = 8;
constexpr int kSortTile = kSortThreads * kSortRounds;

int64_t sort_counts_len(int64_t nmax) { return 256 * ((nmax + kSortTile - 1) / kSortTile) + 1; }

__global__ __launch_bounds__(kSortThreads) void k_sort_count(const uint64_t *__restrict__ key,
                                                             uint32_t n, uint32_t shift,
                                                             uint32_t ntiles,
                                                             uint32_t *__restrict__ counts) {
    __shared__ uint32_t hist[256];
    if (threadIdx.x < 256) hist[threadIdx.x] = 0;
    __syncthreads();
    uint32_t w = threadIdx.x >> 6, lane = lane_id();
    uint64_t base = (uint64_t)blockIdx.x * kSortTile + w * 512 + lane;
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        uint64_t i = base + r * 64;
        if (i < n) atomicAdd(&hist[(uint32_t)(key[i] >> shift) & 255u], 1u);
    }
    __syncthreads();
    if (threadIdx.x < 256) counts[(uint64_t)threadIdx.x * ntiles + blockIdx.x] = hist[threadIdx.x];
}

__global__ __launch_bounds__(kSortThreads) void k_sort_scatter(
    const uint64_t *__restrict__ key_in, const uint32_t *__restrict__ idx_in, uint32_t n,
    uint32_t shift, uint32_t ntiles, const uint32_t *__restrict__ offsets,
    uint64_t *__restrict__ key_out, uint32_t *__restrict__ idx_out) {
    __shared__ uint32_t cnt[kSortWaves][256];
    uint32_t w = threadIdx.x >> 6, lane = lane_id();
    for (int k = 0; k < kSortWaves * 256; k += kSortThreads)
        (&cnt[0][0])[k + threadIdx.x] = 0;
    __syncthreads();
    uint64_t base = (uint64_t)blockIdx.x * kSortTile + w * 512 + lane;
    uint64_t kk[kSortRounds];
    uint32_t vv[kSortRounds], dd[kSortRounds], rk[kSortRounds];
    uint64_t lt = mask_lt(lane);
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        uint64_t i = base + r * 64;
        bool valid = i < n;
        uint64_t k = valid ? key_in[i] : 0ull;
        uint32_t v = valid ? idx_in[i] : 0u;
        uint32_t d = (uint32_t)(k >> shift) & 255u;
        // lanes of this round holding the same digit
        uint64_t peers = ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            bool bit = (d >> b) & 1u;
            uint64_t m = ballot(bit);
            peers &= bit ? m : ~m;
        }
        uint32_t before = __popcll(peers & lt);
        uint32_t run = valid ? cnt[w][d] : 0u;
        __builtin_amdgcn_wave_barrier();
        if (valid && before == 0) cnt[w][d] = run + (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
        kk[r] = k;
        vv[r] = v;
        dd[r] = valid ? d : 256u;
        rk[r] = run + before;
    }
    __syncthreads();
    // the tile reordered by digit in LDS: digit d starts at lo[d] (an
    // exclusive scan of the tile's digit counts), wave w's keys of digit d
    // after those of the waves before it; then written out in LDS order,
    // so that consecutive threads store consecutive keys of one digit run
    // (whole cache lines) instead of one key per run
    __shared__ uint64_t skey[kSortTile];
    __shared__ uint32_t sidx[kSortTile];
    __shared__ uint32_t wsum[4];
    __shared__ int32_t delta[256];
    uint32_t tot = 0, lo = 0;
    if (threadIdx.x < 256) {  // waves 0..3: one digit per thread
        const uint32_t d = threadIdx.x;
#pragma unroll
        for (int k = 0; k < kSortWaves; ++k) tot += cnt[k][d];
        const uint32_t inc = wave_incl_scan(tot, lane);
        if (lane == 63) wsum[w] = inc;
        lo = inc - tot;
    }
    __syncthreads();
    if (threadIdx.x < 256) {
        const uint32_t d = threadIdx.x;
        for (uint32_t k = 0; k < w; ++k) lo += wsum[k];
        const uint32_t g = offsets[(uint64_t)d * ntiles + blockIdx.x];
        delta[d] = (int32_t)(g - lo);
        uint32_t run = lo;
#pragma unroll
        for (int k = 0; k < kSortWaves; ++k) {
            const uint32_t c = cnt[k][d];
            cnt[k][d] = run;
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        if (dd[r] < 256u) {
            const uint32_t lp = cnt[w][dd[r]] + rk[r];
            skey[lp] = kk[r];
            sidx[lp] = vv[r];
        }
    }
    __syncthreads();
    const uint64_t t0 = (uint64_t)blockIdx.x * kSortTile;
    const uint32_t valid = n - t0 < (uint64_t)kSortTile ? (uint32_t)(n - t0) : (uint32_t)kSortTile;
    for (uint32_t t = threadIdx.x; t < valid; t += kSortThreads) {
        const uint64_t k = skey[t];
        const uint32_t pos = (uint32_t)(delta[(uint32_t)(k >> shift) & 255u] + (int32_t)t);
        key_out[pos] = k;
        idx_out[pos] = sidx[t];
    }
}

void launch_sort(bh_ctx *c, const Source &s, uint32_t n, hipStream_t st) {
    // (up to kRankMax particles the sort's first launch clears the words itself:
    // 2.5 us less of 71 at 1000 particles)
    if (c->clear_status && n > kRankMax) launch_fill_u32(c->status, 0u, 4, st);
    if (n <= kMergeMax) return launch_merge_sort(c, s, n, st);
    const uint32_t nb = launch_bbox_partial(c, s, n, st);
    hipLaunchKernelGGL(k_bbox_final, dim3(1), dim3(64), 0, st, (const float *)c->box_part, nb,
                       c->box, fixed_box(c), c->status);
    launch_keys(c, s, n, st);
    uint32_t ntiles = cdiv(n, kSortTile);
    uint32_t len = 256u * ntiles;
    int src = 0;
    for (uint32_t pass = 0; pass < 8; ++pass) {
        uint32_t shift = 8 * pass;
        hipLaunchKernelGGL(k_sort_count, dim3(ntiles), dim3(kSortThreads), 0, st,
                           (const uint64_t *)c->sort.key[src], n, shift, ntiles, c->sort.counts);
        launch_exclusive_scan(c->sort.counts, c->sort.counts, len, c->sort.scan_part, st);
        hipLaunchKernelGGL(k_sort_scatter, dim3(ntiles), dim3(kSortThreads), 0, st,
                           (const uint64_t *)c->sort.key[src], (const uint32_t *)c->sort.idx[src],
                           n, shift, ntiles, (const uint32_t *)c->sort.counts,
                           c->sort.key[src ^ 1], c->sort.idx[src ^ 1]);
        src ^= 1;
    }
    // 8 passes: the result is back in buffer 0
    launch_gather(c, s, n, st);
}

}  // namespace bh
