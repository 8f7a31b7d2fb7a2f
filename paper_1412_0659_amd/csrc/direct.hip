// FP64 direct summation at chosen target particles over every particle of
// the current state: the theta -> 0 limit of the tree force (Sec. I.A), with
// Plummer softening, and the reference the error of the tree forces is
// stated against.  Positions are the FP32 values the tree is built from,
// widened exactly; every product and sum is FP64.  The self pair is skipped
// (no force, no potential); a zero-separation pair without softening has no
// finite term and is skipped too.
//
// Work split: a block of 256 lanes takes 512 targets, two per lane, and one
// span of the sources, staged through LDS as FP64 256 at a time (converted
// once per block, read once for both targets).  Up to 256 targets each lane
// takes one, and below 129 two or four parts of the block share the sources
// of a chunk, so that all its waves have work.  The partial sums of one
// target are added with FP64 atomics, so their order (and the last bits of
// the result) may vary between runs.
//
// Bound: FP64 VALU, 18 operations and one v_rsq_f64 per pair.  1 / r is the
// hardware's estimate and one third-order step, y (1 + e (1/2 + 3/8 e)) with
// e = 1 - r^2 y^2, which leaves only rounding; a square root and a division
// cost more than the rest of the pair.  8192 targets of 1M sources: 5.38 ms,
// 1.52e12 pairs/s, against 13.4 ms with the square root, the division and the
// conversions in the loop; the error against a sum in another order is no
// larger (9.6e-16, before 1.1e-15).  64 targets of 100000: 36 against 798 us.
#include <algorithm>
#include <cmath>

#include "bh_internal.h"

namespace bh {

__global__ __launch_bounds__(256) void k_inverse(const uint32_t *__restrict__ cid, uint32_t n,
                                                 uint32_t *__restrict__ inv) {
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) inv[cid[i]] = i;
}

struct Src64 {
    double x, y, z, m;
};

struct Target {
    double x, y, z;
    double ax, ay, az, ph;
    uint32_t self;  // sorted slot, kNone: no target
};

// One pair.  kSelf: the source may be the target itself (slot j).
template <bool kEps0, bool kSelf>
__device__ __forceinline__ void direct_pair(Target &t, const Src64 &s, uint32_t j, double eps2) {
    const double dx = s.x - t.x, dy = s.y - t.y, dz = s.z - t.z;
    const double r2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, eps2)));
    double y = __builtin_amdgcn_rsq(r2);
    const double e = fma(-(r2 * y), y, 1.0);
    y = fma(y * e, fma(e, 0.375, 0.5), y);
    if (kEps0) y = r2 == 0.0 ? 0.0 : y;
    if (kSelf) y = j == t.self ? 0.0 : y;
    const double mr = s.m * y;
    const double mr3 = mr * (y * y);
    t.ax = fma(mr3, dx, t.ax);
    t.ay = fma(mr3, dy, t.ay);
    t.az = fma(mr3, dz, t.az);
    t.ph = t.ph - mr;
}

// kT targets per lane; `parts` (1, 2 or 4; 1 if kT == 2) parts of the block
// take every parts-th source of a chunk.
template <bool kEps0, int kT>
__global__ __launch_bounds__(256) void k_direct(const float4 *__restrict__ xyzm,
                                                const uint32_t *__restrict__ inv,
                                                const int64_t *__restrict__ tgt, uint32_t nt,
                                                uint32_t n, uint32_t span, uint32_t parts,
                                                double eps2, double *acc, double *pot,
                                                uint32_t *status) {
    __shared__ Src64 src[256];
    Target t[kT];
    const uint32_t lanes = 256u / parts, tl = threadIdx.x & (lanes - 1u),
                   part = threadIdx.x / lanes;
#pragma unroll
    for (int q = 0; q < kT; ++q) {
        const uint32_t k = (blockIdx.x * kT + q) * lanes + tl;
        t[q] = Target{0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, kNone};
        if (k >= nt) continue;
        const int64_t i = tgt[k];
        if (i < 0 || i >= (int64_t)n) {
            if (blockIdx.y == 0 && part == 0) atomicOr(status, kStIndex);
            continue;  // still takes part in the block's barriers
        }
        t[q].self = inv[i];
        const float4 p = xyzm[t[q].self];
        t[q].x = p.x;
        t[q].y = p.y;
        t[q].z = p.z;
    }
    const uint32_t j0 = blockIdx.y * span;
    const uint32_t j1 = j0 + span < n ? j0 + span : n;
    for (uint32_t base = j0; base < j1; base += 256) {
        const uint32_t j = base + threadIdx.x;
        __syncthreads();
        const float4 p = xyzm[j < j1 ? j : base];
        src[threadIdx.x] = Src64{p.x, p.y, p.z, p.w};
        __syncthreads();
        const uint32_t m = j1 - base < 256u ? j1 - base : 256u;
        // only the few chunks that hold a target of the wave look for it
        bool own = false;
#pragma unroll
        for (int k = 0; k < kT; ++k) own = own || t[k].self - base < m;
        if (__any(own)) {
            for (uint32_t q = part; q < m; q += parts)
#pragma unroll
                for (int k = 0; k < kT; ++k)
                    direct_pair<kEps0, true>(t[k], src[q], base + q, eps2);
        } else {
#pragma unroll 2
            for (uint32_t q = part; q < m; q += parts)
#pragma unroll
                for (int k = 0; k < kT; ++k) direct_pair<kEps0, false>(t[k], src[q], 0u, eps2);
        }
    }
    if (parts > 1u) {  // (one target per lane) the parts' sums to the first
        double *sum = reinterpret_cast<double *>(src);  // [256][4]
        __syncthreads();
        sum[4 * threadIdx.x] = t[0].ax; sum[4 * threadIdx.x + 1] = t[0].ay;
        sum[4 * threadIdx.x + 2] = t[0].az; sum[4 * threadIdx.x + 3] = t[0].ph;
        __syncthreads();
        if (part != 0u) return;
        for (uint32_t q = 1; q < parts; ++q) {
            const double *o = sum + 4 * (q * lanes + tl);
            t[0].ax += o[0]; t[0].ay += o[1]; t[0].az += o[2]; t[0].ph += o[3];
        }
    }
#pragma unroll
    for (int q = 0; q < kT; ++q) {
        if (t[q].self == kNone) continue;
        const size_t k = (blockIdx.x * kT + q) * lanes + tl;
        atomicAdd(acc + 3 * k, t[q].ax);
        atomicAdd(acc + 3 * k + 1, t[q].ay);
        atomicAdd(acc + 3 * k + 2, t[q].az);
        atomicAdd(pot + k, t[q].ph);
    }
}

__global__ __launch_bounds__(256) void k_zero_f64(double *p, uint64_t n) {
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * 256)
        p[i] = 0.0;
}

void launch_direct(bh_ctx *c, const int64_t *tgt, uint32_t nt, float eps, double *acc,
                   double *pot, hipStream_t st) {
    const uint32_t n = (uint32_t)c->n;
    hipLaunchKernelGGL(k_inverse, dim3(cdiv(n, 256)), dim3(256), 0, st,
                       (const uint32_t *)c->st[c->cur].cid, n, c->inv);
    hipLaunchKernelGGL(k_zero_f64, dim3(cdiv(3ull * nt, 256)), dim3(256), 0, st, acc,
                       3ull * nt);
    hipLaunchKernelGGL(k_zero_f64, dim3(cdiv(nt, 256)), dim3(256), 0, st, pot, (uint64_t)nt);
    const uint32_t parts = nt <= 64u ? 4u : (nt <= 128u ? 2u : 1u);
    const uint32_t tb = nt <= 256u ? 1u : cdiv(nt, 512);
    // Spans: blocks to fill the chip several times over, but every span adds to
    // the same sums (70 ns each, one after another) and a lane takes about as
    // long per source, so of the order of the square root of a part's sources
    // (64 targets of 1M sources: 1026 us with 3906 spans and four adds each, 104
    // us so; of 100000: 114 us with 391, 36 us).
    const uint32_t most = (uint32_t)std::sqrt(2.0 * n / parts) + 1u;
    uint32_t ns = std::min({cdiv(8192, tb), most, cdiv(n, 256)});
    const uint32_t span = cdiv(cdiv(n, ns), 256) * 256;
    ns = cdiv(n, span);
    const double e2 = (double)eps * (double)eps;
    auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(tb, ns), dim3(256), 0, st, (const float4 *)c->xyzm,
                           (const uint32_t *)c->inv, tgt, nt, n, span, parts, e2, acc, pot,
                           c->status);
    };
    if (nt <= 256u) eps == 0.f ? run(k_direct<true, 1>) : run(k_direct<false, 1>);
    else eps == 0.f ? run(k_direct<true, 2>) : run(k_direct<false, 2>);
}

}  // namespace bh
