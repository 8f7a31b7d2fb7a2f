// Octree construction from the sorted keys (Sec. I.A: octants are split until
// a cell holds at most nleaf particles; Table II "Tree-construction"), and
// the target groups of the walk.
//
// Cells are numbered breadth first: the cells of level l, in key order, then
// those of level l + 1.  No level waits for the one above it: which cells a
// particle lies in follows from the keys next to its own.  With common(a, b)
// the number of leading 3-bit digits two keys share,
//   * the cell of level l holding sorted particle i has more than m particles
//     iff l <= D_m(i) = max over j in [i - m, i] of common(key[j], key[j + m])
//     (m + 1 consecutive keys around i share the level's prefix);
//   * so i lies in cells of the levels 0 .. hi(i) = min(D_nleaf(i) + 1, 21),
//     all but the last of them split;
//   * the cells whose first particle is i are those of the levels
//     lo(i) = common(key[i - 1], key[i]) + 1 .. hi(i) (lo(0) = 0), and the
//     cells whose last particle is i those of the levels lo(i + 1) .. hi(i);
//   * the number of a cell is its level's start plus the number of cells of
//     that level that start before it, its parent is the last cell of the
//     level above that starts at or before it, its children begin with the
//     cell of the next level that starts with it and end with the one that
//     ends with it.
// Three launches: per tile of particles the levels of each particle and the
// cells that start in the tile per level (k_tree_levels), the running sums of
// those counts over the tiles (k_tree_scan; up to kScanTiles tiles each block of
// the next sums them itself, 4 us less), and the cells (k_tree_write), ranked
// inside the tile by a bit mask per level.  The build never waits on
// the host and does not depend on the depth of the tree.
//
// Bound: memory, 16 B of keys and 4 B of levels per particle and 36 B per
// cell; on small sets the latency of the three launches.  Measured at 13M
// (disk + halo): 0.20 ms, where splitting level by level with binary searches
// (three launches per level) took 0.76 ms; at 16384: 18 against 260 us.
//
// A cell is a group iff (count <= ncrit or it is a leaf) and (it is the root
// or its parent holds more than ncrit), so the group of particle i is the
// cell of level g(i) = min(D_ncrit(i) + 1, hi(i)); groups are numbered in key
// order as one more level.  A group cell larger than ncrit (a leaf, for
// nleaf > ncrit or coincident keys) is cut into chunks of ncrit.
#include <type_traits>

#include "bh_internal.h"
#include "wave.h"

namespace bh {

constexpr int kTreeWords = kTreeTile / 64;
constexpr int kHalo = 64;               // nleaf, ncrit <= 64
constexpr int kGroupCh = kLevels;       // the groups' channel of the tile counts

// leading 3-bit digits (of 21) that two 63-bit keys share
__device__ __forceinline__ int common_digits(uint64_t a, uint64_t b) {
    const uint64_t x = a ^ b;
    return x == 0ull ? kKeyBits : (__clzll((long long)x) - 1) / 3;
}

__device__ __forceinline__ uint32_t key_lower_bound(const uint64_t *__restrict__ k, uint32_t lo,
                                                    uint32_t hi, uint64_t v) {
    while (lo < hi) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        if (k[mid] < v) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// Levels of every particle and, per tile, the number of cells of each level
// (and of groups) that start in it.  Window maxima by doubling: entry j holds
// max over [j, j + 2^k) of common(key[j], key[j + m]) + 1, for m = nleaf and
// m = ncrit in the two halves of a word.
template <int kThreads>
__global__ __launch_bounds__(kThreads) void k_tree_levels(const uint64_t *__restrict__ key,
                                                              uint32_t n, uint32_t nleaf,
                                                              uint32_t ncrit, uint32_t ntiles,
                                                              uint16_t *__restrict__ lev,
                                                              uint32_t *__restrict__ tcnt) {
    constexpr int kItems = kTreeTile / kThreads;
    constexpr int kSpan = kTreeTile + kHalo;  // entries j = t0 - kHalo .. t0 + kTreeTile - 1
    __shared__ uint64_t k[kTreeTile + 2 * kHalo];
    __shared__ u16x2 win[2][kSpan];
    __shared__ uint32_t cnt[kLevels + 1];
    const int64_t t0 = (int64_t)blockIdx.x * kTreeTile;
    for (int q = threadIdx.x; q < kTreeTile + 2 * kHalo; q += kThreads) {
        const int64_t j = t0 - kHalo + q;
        k[q] = j >= 0 && j < (int64_t)n ? key[j] : 0ull;
    }
    if (threadIdx.x <= kLevels) cnt[threadIdx.x] = 0u;
    __syncthreads();
    for (int q = threadIdx.x; q < kSpan; q += kThreads) {
        const int64_t j = t0 - kHalo + q;
        u16x2 v = {0, 0};
        if (j >= 0) {
            if (j + nleaf < (int64_t)n) v.x = (unsigned short)(common_digits(k[q], k[q + nleaf]) + 1);
            if (j + ncrit < (int64_t)n) v.y = (unsigned short)(common_digits(k[q], k[q + ncrit]) + 1);
        }
        win[0][q] = v;
    }
    __syncthreads();
    const int kl = 31 - __clz((int)nleaf + 1), kc = 31 - __clz((int)ncrit + 1);
    const int steps = max(kl, kc);
    uint32_t dl[kItems], dc[kItems];  // D + 1 of this thread's particles
    for (int s = 0; s <= steps; ++s) {
        const u16x2 *w = win[s & 1];
        if (s == kl || s == kc) {
#pragma unroll
            for (int r = 0; r < kItems; ++r) {
                const int q = kHalo + r * kThreads + (int)threadIdx.x;
                if (s == kl)
                    dl[r] = max((uint32_t)w[q - (int)nleaf].x, (uint32_t)w[q - (1 << kl) + 1].x);
                if (s == kc)
                    dc[r] = max((uint32_t)w[q - (int)ncrit].y, (uint32_t)w[q - (1 << kc) + 1].y);
            }
        }
        if (s == steps) break;
        u16x2 *o = win[(s + 1) & 1];
        for (int q = threadIdx.x; q < kSpan; q += kThreads) {
            const u16x2 a = w[q], b = q + (1 << s) < kSpan ? w[q + (1 << s)] : a;
            o[q] = __builtin_elementwise_max(a, b);
        }
        __syncthreads();
    }
    const uint32_t lane = lane_id();
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const int q = kHalo + r * kThreads + (int)threadIdx.x;
        const int64_t i = t0 + q - kHalo;
        const bool valid = i < (int64_t)n;
        uint32_t lo = 31u, hi = 0u;
        bool gs = false;
        if (valid) {
            lo = i == 0 ? 0u : (uint32_t)common_digits(k[q - 1], k[q]) + 1u;
            hi = min(dl[r], (uint32_t)(kLevels - 1));
            const uint32_t g = min(dc[r], hi);
            gs = lo <= g;
            if (dc[r] > g) {  // the group's cell holds more than ncrit: chunks of ncrit
                const uint32_t sh = 3u * (kKeyBits - g);
                const uint64_t p = g == 0u ? 0ull : (k[q] >> sh) << sh;
                const uint32_t b = gs ? (uint32_t)i : key_lower_bound(key, 0u, (uint32_t)i, p);
                gs = ((uint32_t)i - b) % ncrit == 0u;
            }
            lev[i] = (uint16_t)(lo | (hi << 5) | (g << 10) | (gs ? 1u << 15 : 0u));
        }
        const uint64_t gm = ballot(gs);
        if (lane == 0 && gm) atomicAdd(&cnt[kGroupCh], (uint32_t)__popcll(gm));
        const bool starts = valid && lo <= hi;
        if (ballot(starts) == 0ull) continue;
        const uint32_t l1 = wave_max(starts ? hi : 0u),
                       l0 = 31u - wave_max(starts ? 31u - lo : 0u);
        for (uint32_t l = l0; l <= l1; ++l) {
            const uint64_t m = ballot(starts && lo <= l && l <= hi);
            if (lane == 0 && m) atomicAdd(&cnt[l], (uint32_t)__popcll(m));
        }
    }
    __syncthreads();
    if (threadIdx.x <= kLevels) tcnt[(size_t)threadIdx.x * ntiles + blockIdx.x] = cnt[threadIdx.x];
}

// One block per level (and one for the groups): exclusive running sums of its
// counts over the tiles, in place; the total into tot[channel].
__global__ __launch_bounds__(1024) void k_tree_scan(uint32_t *__restrict__ tcnt, uint32_t ntiles,
                                                    uint32_t *__restrict__ tot) {
    __shared__ uint32_t ws[16];
    uint32_t *row = tcnt + (size_t)blockIdx.x * ntiles;
    const uint32_t lane = lane_id(), w = threadIdx.x >> 6;
    constexpr uint32_t kPer = 8;
    uint32_t carry = 0;
    for (uint32_t base = 0; base < ntiles; base += 1024u * kPer) {
        uint32_t v[kPer], s = 0;
#pragma unroll
        for (uint32_t q = 0; q < kPer; ++q) {
            const uint32_t i = base + threadIdx.x * kPer + q;
            v[q] = i < ntiles ? row[i] : 0u;
            s += v[q];
        }
        const uint32_t inc = wave_incl_scan(s, lane);
        if (lane == 63) ws[w] = inc;
        __syncthreads();
        uint32_t off = carry + inc - s, all = 0;
#pragma unroll
        for (uint32_t q = 0; q < 16; ++q) {
            if (q < w) off += ws[q];
            all += ws[q];
        }
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < kPer; ++q) {
            const uint32_t i = base + threadIdx.x * kPer + q;
            if (i < ntiles) row[i] = off;
            off += v[q];
        }
        carry += all;
    }
    if (threadIdx.x == 0) tot[blockIdx.x] = carry;
}

// The cells and groups that start or end in the tile.  A cell's end (one past
// its last particle) is left in count and the end of its children (0 for a
// leaf) in nchild: its first and last particle may lie in different tiles.
// The moment pass turns both into counts.
template <int kThreads>
__global__ __launch_bounds__(kThreads) void k_tree_write(
    Cells c, const uint64_t *__restrict__ key, const uint16_t *__restrict__ lev, uint32_t n,
    uint32_t ntiles, const uint32_t *__restrict__ tcnt, uint32_t *__restrict__ tot,
    uint32_t cap, uint32_t *__restrict__ gbeg, uint32_t gcap, uint32_t *__restrict__ gpar,
    uint32_t *ngroups, uint32_t *status) {
    constexpr int kItems = kTreeTile / kThreads;
    // cells of each level (and groups) that start before the tile, and in all tiles
    __shared__ uint32_t tb[kLevels + 1], tt[kLevels + 1];
    __shared__ uint64_t mask[kLevels + 1][kTreeWords];
    __shared__ uint32_t pre[kLevels + 1][kTreeWords];  // starts of the level before the word
    const uint32_t lane = lane_id(), w = threadIdx.x >> 6;
    const uint32_t t0 = blockIdx.x * kTreeTile;
    for (uint32_t q = threadIdx.x; q < (kLevels + 1) * kTreeWords; q += kThreads)
        (&mask[0][0])[q] = 0ull;
    if (ntiles <= kScanTiles) {  // (no k_tree_scan) a lane per tile
        for (uint32_t l = w; l <= kLevels; l += kThreads / 64) {
            const uint32_t v = lane < ntiles ? tcnt[(size_t)l * ntiles + lane] : 0u;
            const uint32_t inc = wave_incl_scan(v, lane);
            if (lane == blockIdx.x) {
                tb[l] = inc - v;
                tot[kLevels + 1u + l * ntiles + lane] = inc - v;
            }
            if (lane == 63u) {
                tt[l] = inc;
                if (blockIdx.x == 0) tot[l] = inc;
            }
        }
    } else if (threadIdx.x <= kLevels) {
        tb[threadIdx.x] = tcnt[(size_t)threadIdx.x * ntiles + blockIdx.x];
        tt[threadIdx.x] = tot[threadIdx.x];
    }
    __syncthreads();
    // level starts (every wave for itself; lane l holds level l's)
    const uint32_t lt = lane < kLevels ? tt[lane] : 0u;
    const uint32_t lend = wave_incl_scan(lt, lane), lstart = lend - lt;
    if (blockIdx.x == 0 && threadIdx.x <= kLevels) {
        c.ls[threadIdx.x] = min(lstart, cap);  // (lane kLevels: the cell count)
        if (threadIdx.x == kLevels) {
            if (lstart > cap) atomicOr(status, kStOverflow);
            *ngroups = tt[kGroupCh];
            if (tt[kGroupCh] < gcap) gbeg[tt[kGroupCh]] = n;
        }
    }
    uint32_t lv[kItems], ln[kItems];
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const uint32_t i = t0 + r * kThreads + threadIdx.x;
        lv[r] = i < n ? lev[i] : 31u;           // no cell
        ln[r] = i + 1u < n ? lv_lo(lev[i + 1u]) : 0u;  // every cell ends with the last particle
        const uint32_t lo = lv_lo(lv[r]), hi = lv_hi(lv[r]);
        const uint32_t word = r * (kThreads / 64) + w;
        const uint64_t gm = ballot(i < n && lv_group(lv[r]));
        if (lane == 0) mask[kGroupCh][word] = gm;
        const bool starts = lo <= hi;
        if (ballot(starts) == 0ull) continue;
        const uint32_t l1 = wave_max(starts ? hi : 0u),
                       l0 = 31u - wave_max(starts ? 31u - lo : 0u);
        for (uint32_t l = l0; l <= l1; ++l) {
            const uint64_t m = ballot(starts && lo <= l && l <= hi);
            if (lane == 0) mask[l][word] = m;
        }
    }
    __syncthreads();
    static_assert(kTreeWords == 16, "a level's words in a row of 16 lanes");
    for (uint32_t q0 = 0; q0 < (kLevels + 1) * kTreeWords; q0 += kThreads) {
        const uint32_t q = q0 + threadIdx.x, l = q / kTreeWords, word = q % kTreeWords;
        const bool have = l <= kLevels;
        const uint32_t cnt = have ? (uint32_t)__popcll(mask[l][word]) : 0u;
        const uint32_t s = row_incl_scan(cnt) - cnt;
        if (have) pre[l][word] = tb[l] + s;
    }
    __syncthreads();
    // numbers of the cells of level l: those that start before particle
    // (word, lane), and the start of the level
    auto before = [&](uint32_t l, uint32_t word) {
        return pre[l][word] + (uint32_t)__popcll(mask[l][word] & mask_lt(lane));
    };
    auto upto = [&](uint32_t l, uint32_t word) {
        return pre[l][word] + (uint32_t)__popcll(mask[l][word] & mask_le(lane));
    };
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const uint32_t i = t0 + r * kThreads + threadIdx.x;
        const uint32_t word = r * (kThreads / 64) + w;
        const uint32_t lo = lv_lo(lv[r]), hi = lv_hi(lv[r]);
        const bool valid = i < n;
        const uint64_t ky = valid ? key[i] : 0ull;
        const bool grp = valid && lv_group(lv[r]);
        const uint32_t gn = before(kGroupCh, word);
        if (grp) gbeg[gn] = i;
        if (gpar && ballot(grp) != 0ull) {  // the parent of the group's cell
            const uint32_t gl = lv_glev(lv[r]), up = gl ? gl - 1u : 0u;
            const uint32_t s = shfl(lstart, (int)up);
            if (grp) gpar[gn] = gl ? s + upto(up, word) - 1u : kNone;
        }
        const bool starts = valid && lo <= hi, ends = valid && ln[r] <= hi;
        if (ballot(starts || ends) == 0ull) continue;
        const uint32_t first = min(starts ? lo : 31u, ends ? ln[r] : 31u);
        const uint32_t l1 = wave_max(starts || ends ? hi : 0u), l0 = 31u - wave_max(31u - first);
        for (uint32_t l = l0; l <= l1; ++l) {
            const uint32_t s0 = read_lane(lstart, l);
            const uint32_t s1 = read_lane(lend, l);  // the start of level l + 1
            const uint32_t sp = read_lane(lstart, l ? l - 1u : 0u);
            if (starts && lo <= l && l <= hi) {
                const uint32_t ch = s0 + before(l, word);
                if (ch < cap) {
                    c.prefix[ch] = l == 0u ? 0ull : ky >> (3u * (kKeyBits - l));
                    c.level[ch] = l;
                    c.begin[ch] = i;
                    c.child0[ch] = l < hi ? s1 + before(l + 1u, word) : kNone;
                    c.parent[ch] = l == 0u ? kNone : sp + upto(l - 1u, word) - 1u;
                }
            }
            if (ends && ln[r] <= l && l <= hi) {
                const uint32_t e = s0 + upto(l, word) - 1u;
                if (e < cap) {
                    c.count[e] = i + 1u;
                    c.nchild[e] = l < hi ? s1 + upto(l + 1u, word) : 0u;
                }
            }
        }
    }
}

// Paired target sets (bh_params.pair_groups = cap, off by default): groups
// 2k and 2k + 1 that are siblings (group cells with one parent, gpar) and hold
// at most cap particles together become one target set, walked once against
// the box of their union.  flag[j] = 1 where group j stays the first of a set.
__global__ __launch_bounds__(256) void k_pair_flags(const uint32_t *__restrict__ gbeg,
                                                    const uint32_t *__restrict__ ngroups,
                                                    const uint32_t *__restrict__ gpar, uint32_t n,
                                                    uint32_t cap, uint32_t *__restrict__ flag) {
    const uint32_t j = blockIdx.x * 256 + threadIdx.x;
    if (j >= n) return;
    const uint32_t ng = *ngroups;
    bool keep = j < ng;
    if (keep && (j & 1u)) {
        const uint32_t end = j + 1u < ng ? gbeg[j + 1u] : n;
        keep = !(end - gbeg[j - 1u] <= cap && gpar[j - 1u] == gpar[j] && gpar[j] != kNone);
    }
    flag[j] = keep ? 1u : 0u;
}

__global__ __launch_bounds__(256) void k_pair_fill(const uint32_t *__restrict__ gbeg0,
                                                   const uint32_t *__restrict__ flag,
                                                   const uint32_t *__restrict__ scan, uint32_t n,
                                                   uint32_t *__restrict__ gbeg,
                                                   uint32_t *ngroups) {
    const uint32_t j = blockIdx.x * 256 + threadIdx.x;
    if (j >= n) return;
    if (flag[j]) gbeg[scan[j]] = gbeg0[j];
    if (j == n - 1u) {
        const uint32_t ng = scan[j] + flag[j];
        *ngroups = ng;
        gbeg[ng] = n;
    }
}

// Cells (count and nchild completed by the moment pass) and groups.
void launch_build(bh_ctx *ctx, uint32_t n, hipStream_t st) {
    Cells &c = ctx->cells;
    Groups &g = ctx->groups;
    const uint64_t *key = ctx->sort.key[0];
    const uint32_t nt = cdiv(n, kTreeTile);
    // paired target sets: the groups first go to the sort's second index
    // buffer, each group's parent cell to npp
    uint32_t *gbeg0 = ctx->pair_groups ? ctx->sort.idx[1] : g.begin;
    uint32_t *gpar = ctx->pair_groups ? g.npp : nullptr;
    auto launch = [&](auto threads) {
        constexpr int kThreads = decltype(threads)::value;
        hipLaunchKernelGGL(k_tree_levels<kThreads>, dim3(nt), dim3(kThreads), 0, st, key, n,
                           (uint32_t)ctx->p.nleaf, (uint32_t)ctx->p.ncrit, nt, c.lev, c.tcnt);
        if (nt > kScanTiles)
            hipLaunchKernelGGL(k_tree_scan, dim3(kLevels + 1), dim3(1024), 0, st, c.tcnt, nt, c.ttot);
        hipLaunchKernelGGL(k_tree_write<kThreads>, dim3(nt), dim3(kThreads), 0, st, c, key,
                           (const uint16_t *)c.lev, n, nt, (const uint32_t *)c.tcnt,
                           c.ttot, (uint32_t)ctx->cap_cells, gbeg0,
                           ctx->pair_groups ? n : n + 1u, gpar, g.count_dev, ctx->status);
    };
    // Threads of a tile.  Up to a tile a CU and beyond, a thread per particle
    // keeps the chain of levels short; with many tiles the waves of other blocks
    // fill the gaps and 16 waves waiting for each other are slower.  The three
    // launches by 256 / 512 / 1024 threads, in us: 1000 27 / 20 / 17; 16384 29 / 22
    // / 18; 65536 28 / 21 / 18; 1M 37 / 32 / 37; 13M 201 / 221 / 283.
    if (n <= 524288u) launch(std::integral_constant<int, 1024>());
    else if (n <= 4194304u) launch(std::integral_constant<int, 512>());
    else launch(std::integral_constant<int, 256>());
    if (!ctx->pair_groups) return;
    hipLaunchKernelGGL(k_pair_flags, dim3(cdiv(n, 256)), dim3(256), 0, st,
                       (const uint32_t *)gbeg0, (const uint32_t *)g.count_dev,
                       (const uint32_t *)gpar, n, ctx->pair_groups, g.flag);
    launch_exclusive_scan(g.flag, g.scan, n, ctx->sort.scan_part, st);
    hipLaunchKernelGGL(k_pair_fill, dim3(cdiv(n, 256)), dim3(256), 0, st,
                       (const uint32_t *)gbeg0, (const uint32_t *)g.flag,
                       (const uint32_t *)g.scan, n, g.begin, g.count_dev);
}

}  // namespace bh
