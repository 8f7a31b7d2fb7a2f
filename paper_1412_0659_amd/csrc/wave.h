// Cross-lane helpers for 64-lane CDNA wavefronts.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bh {

__device__ __forceinline__ uint32_t lane_id() {
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// lanes strictly below / at-or-below this lane
__device__ __forceinline__ uint64_t mask_lt(uint32_t lane) {
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}
__device__ __forceinline__ uint64_t mask_le(uint32_t lane) {
    return ~0ull >> (63 - lane);
}

__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// popcount of the set bits of m below this lane (v_mbcnt)
__device__ __forceinline__ uint32_t count_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// value of v in lane src (modulo 64)
__device__ __forceinline__ uint32_t shfl(uint32_t v, uint32_t src) {
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(src << 2), (int)v);
}

// inclusive prefix sum over the 64 lanes (all lanes active): a Hillis-Steele
// scan inside each row of 16 lanes with DPP row shifts (lanes whose source is
// outside the row add 0), then the row totals carried by the row broadcasts.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v, uint32_t lane) {
    (void)lane;
    int s = (int)v;
    s += __builtin_amdgcn_update_dpp(0, s, 0x111, 0xf, 0xf, false);  // row_shr:1
    s += __builtin_amdgcn_update_dpp(0, s, 0x112, 0xf, 0xf, false);  // row_shr:2
    s += __builtin_amdgcn_update_dpp(0, s, 0x114, 0xf, 0xf, false);  // row_shr:4
    s += __builtin_amdgcn_update_dpp(0, s, 0x118, 0xf, 0xf, false);  // row_shr:8
    s += __builtin_amdgcn_update_dpp(0, s, 0x142, 0xa, 0xf, false);  // row_bcast:15 -> rows 1, 3
    s += __builtin_amdgcn_update_dpp(0, s, 0x143, 0xc, 0xf, false);  // row_bcast:31 -> rows 2, 3
    return (uint32_t)s;
}

// inclusive prefix sum inside each row of 16 lanes
__device__ __forceinline__ uint32_t row_incl_scan(uint32_t v) {
    int s = (int)v;
    s += __builtin_amdgcn_update_dpp(0, s, 0x111, 0xf, 0xf, false);
    s += __builtin_amdgcn_update_dpp(0, s, 0x112, 0xf, 0xf, false);
    s += __builtin_amdgcn_update_dpp(0, s, 0x114, 0xf, 0xf, false);
    s += __builtin_amdgcn_update_dpp(0, s, 0x118, 0xf, 0xf, false);
    return (uint32_t)s;
}

// value of v in lane src (src uniform across the wave)
__device__ __forceinline__ uint32_t read_lane(uint32_t v, uint32_t src) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)src);
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

// minimum / maximum over the 64 lanes (all lanes active), uniform: the steps
// of the scan above, a lane without a source keeping its own value
template <int kCtrl, int kRowMask>
__device__ __forceinline__ float dpp_or_own(float v) {
    const int i = __float_as_int(v);
    return __int_as_float(__builtin_amdgcn_update_dpp(i, i, kCtrl, kRowMask, 0xf, false));
}
__device__ __forceinline__ float last_lane(float v) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float wave_min(float v) {
    v = fminf(v, dpp_or_own<0x111, 0xf>(v));
    v = fminf(v, dpp_or_own<0x112, 0xf>(v));
    v = fminf(v, dpp_or_own<0x114, 0xf>(v));
    v = fminf(v, dpp_or_own<0x118, 0xf>(v));
    v = fminf(v, dpp_or_own<0x142, 0xa>(v));
    return last_lane(fminf(v, dpp_or_own<0x143, 0xc>(v)));
}
__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, dpp_or_own<0x111, 0xf>(v));
    v = fmaxf(v, dpp_or_own<0x112, 0xf>(v));
    v = fmaxf(v, dpp_or_own<0x114, 0xf>(v));
    v = fmaxf(v, dpp_or_own<0x118, 0xf>(v));
    v = fmaxf(v, dpp_or_own<0x142, 0xa>(v));
    return last_lane(fmaxf(v, dpp_or_own<0x143, 0xc>(v)));
}

template <int kCtrl, int kRowMask>
__device__ __forceinline__ uint32_t dpp_or_own(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, kCtrl, kRowMask, 0xf, false);
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
    v = max(v, dpp_or_own<0x111, 0xf>(v));
    v = max(v, dpp_or_own<0x112, 0xf>(v));
    v = max(v, dpp_or_own<0x114, 0xf>(v));
    v = max(v, dpp_or_own<0x118, 0xf>(v));
    v = max(v, dpp_or_own<0x142, 0xa>(v));
    return read_lane(max(v, dpp_or_own<0x143, 0xc>(v)), 63u);
}

// Order the LDS accesses of one wave: the DS unit runs a wave's accesses in
// program order, so only the compiler has to keep them in it (no barrier, no
// wait; a workgroup may hold several waves that walk different groups).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// a / b for a <= 128, 1 <= b <= 128: (a + 1/2) / b is at least 1/256 from the
// next whole number, and the approximate quotient off by 4e-5 at most
__device__ __forceinline__ uint32_t small_div(uint32_t a, uint32_t b) {
    return (uint32_t)(((float)a + 0.5f) * __builtin_amdgcn_rcpf((float)b));
}

// uniform value from lane 0 held in a scalar register
__device__ __forceinline__ uint32_t uniform(uint32_t v) {
    return __builtin_amdgcn_readfirstlane(v);
}

}  // namespace bh
