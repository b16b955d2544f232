// Small device helpers shared by the libjas kernels (wave64, gfx950).
#pragma once
#include <type_traits>

#include <hip/hip_runtime.h>

#include <cstdint>

namespace jas {

constexpr int kWave = 64;

__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & (kWave - 1); }

__device__ __forceinline__ uint64_t lanemask_lt() {
    const uint32_t l = lane_id();
    return l == 0 ? 0ull : (~0ull >> (64 - l));
}

// The lanes of the wave whose value agrees with this lane's in its low NB bits
// (all 64 lanes must call it).  Per bit one ballot and, for each half of the
// mask, one three-input operation: m & ~(vote ^ own bit), the own bit spread
// over the word.
template <int NB>
__device__ __forceinline__ uint64_t wave_match(uint32_t v) {
    uint32_t lo = ~0u, hi = ~0u;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        int32_t own = __builtin_amdgcn_sbfe((int32_t)v, b, 1);
        asm("" : "+v"(own));  // compared as it is (else the bit is shifted out a second time)
        const uint64_t vote = __ballot(own < 0);
        lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)vote, (uint32_t)own, 0x90);
        hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(vote >> 32), (uint32_t)own, 0x90);
    }
    return ((uint64_t)hi << 32) | lo;
}

// Set lanes of m below this lane.
__device__ __forceinline__ uint32_t lanes_before(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

// Inclusive scan across the 64 lanes of a wave.
__device__ __forceinline__ uint64_t wave_incl_scan(uint64_t v) {
    const uint32_t l = lane_id();
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint64_t t = __shfl_up(v, d, kWave);
        if (l >= (uint32_t)d) v += t;
    }
    return v;
}

__device__ __forceinline__ uint32_t wave_incl_scan_u32(uint32_t v) {
    const uint32_t l = lane_id();
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t t = __shfl_up(v, d, kWave);
        if (l >= (uint32_t)d) v += t;
    }
    return v;
}

// Exclusive scan of one value per thread across a block of NT threads.
// sh needs NT/64 entries.  Every thread of the block must call it.
template <int NT>
__device__ __forceinline__ uint64_t block_excl_scan(uint64_t v, uint64_t *sh, uint64_t *total) {
    const uint32_t l = lane_id(), w = threadIdx.x / kWave;
    const uint64_t inc = wave_incl_scan(v);
    if (l == kWave - 1) sh[w] = inc;
    __syncthreads();
    uint64_t before = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < NT / kWave; ++k) {
        const uint64_t x = sh[k];
        before += (k < (int)w) ? x : 0;
        tot += x;
    }
    __syncthreads();
    *total = tot;
    return before + inc - v;
}

// The same for 32-bit values, without the total.
template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan_u32(uint32_t v, uint32_t *sh) {
    const uint32_t l = lane_id(), w = threadIdx.x / kWave;
    const uint32_t inc = wave_incl_scan_u32(v);
    if (l == kWave - 1) sh[w] = inc;
    __syncthreads();
    uint32_t before = 0;
#pragma unroll
    for (int k = 0; k < NT / kWave; ++k) before += (k < (int)w) ? sh[k] : 0;
    __syncthreads();
    return before + inc - v;
}

// Largest v of this lane and the ones before it.
__device__ __forceinline__ uint32_t wave_incl_max(uint32_t v) {
    const auto from = [](uint32_t x, auto ctrl, auto rows) {
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, decltype(rows)::value, 0xf, false);
    };
    using std::integral_constant;
    v = max(v, from(v, integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{}));  // row_shr:1
    v = max(v, from(v, integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{}));  // row_shr:2
    v = max(v, from(v, integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{}));  // row_shr:4
    v = max(v, from(v, integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{}));  // row_shr:8
    v = max(v, from(v, integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{}));  // row_bcast:15
    return max(v, from(v, integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{}));  // row_bcast:31
}

// The value of the lane before (0 in lane 0).
__device__ __forceinline__ uint32_t wave_shift_up(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xf, 0xf, false);  // wave_shr:1
}

// Largest s in [lo, hi] with off[s] <= t (CSR sample of entry t).
__device__ __forceinline__ int32_t find_sample(const uint64_t *off, int32_t lo, int32_t hi, uint64_t t) {
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (off[mid] <= t) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// First position in [lo, hi) of the ascending array v whose value is >= target
// (hi if none).  The search starts at the place `frac` (a fraction of 2^64) of the
// range and widens from there: where the values are spread evenly it reads the
// one or two cache lines around its target, and however they are spread it
// takes a logarithmic number of steps.
__device__ __forceinline__ uint64_t lower_bound_from(const uint64_t *__restrict__ v, uint64_t lo, uint64_t hi,
                                                     uint64_t target, uint64_t frac) {
    if (lo >= hi) return lo;
    const uint64_t m = lo + __umul64hi(frac, hi - lo);  // < hi
    uint64_t step = 4;
    if (v[m] < target) {
        lo = m + 1;
        while (lo < hi) {
            const uint64_t t = min(lo + step, hi) - 1;
            if (v[t] >= target) {
                hi = t;
                break;
            }
            lo = t + 1;
            step *= 2;
        }
    } else {
        hi = m;
        while (lo < hi) {
            const uint64_t t = hi - lo > step ? hi - step : lo;
            if (v[t] < target) {
                lo = t + 1;
                break;
            }
            hi = t;
            step *= 2;
        }
    }
    while (lo < hi) {
        const uint64_t t = (lo + hi) >> 1;
        if (v[t] < target) lo = t + 1;
        else hi = t;
    }
    return lo;
}

// Position of (i, j), i <= j, in an n x n output: row-major full or packed upper.
__device__ __forceinline__ uint64_t out_index(uint32_t i, uint32_t j, uint32_t n, bool upper) {
    return upper ? (uint64_t)i * n - (uint64_t)i * (i - 1) / 2 + (j - i) : (uint64_t)i * n + j;
}

}  // namespace jas
