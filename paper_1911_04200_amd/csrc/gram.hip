// Gram product B = A^T A on the encoding, and the similarity (Sec. III-A/B).
//
// Packed rows (Eq. (7)):  B_ij += sum_w popcount(W[w][i] & W[w][j]), summed
//   over every word row of every batch (Eq. (4)).  The upper triangle of
//   128 x 128 column tiles is computed; word rows are split into K ranges so
//   the grid fills the chip, and each block adds its tile into B with integer
//   atomics (exact and order independent).
// Row lists: a row shared by d = 2..dmin-1 sets adds 1 to B_ij for each of its
//   d(d-1)/2 pairs i < j (its outer product a_k a_k^T, unpacked).
// Diagonal: B_ii = |X_i| (column sums, Eq. (4)).
// Finalize: C_ij = |X_i| + |X_j| - B_ij, J_ij = B_ij / C_ij, J = 1 if C_ij = 0
//   (Sec. II-A, Eq. (2)); IEEE binary64 division, round to nearest.
#include <algorithm>
#include <vector>

#include <cmath>
#include <map>
#include <mutex>
#include <tuple>

#include "device_util.hpp"
#include "jas_internal.hpp"

namespace jas {
namespace {

constexpr int kNT = 256;
constexpr int kT = 128;   // column tile
constexpr int kKC = 16;   // word rows per LDS stage

__global__ void k_fill_i32(int32_t *p, uint64_t len, int32_t v) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < len; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// The chip's 8 XCDs each have their own L2, and workgroups go to them
// round-robin by linear id (x fastest), so consecutive ids land on different
// XCDs.  Renumbered so that XCD x runs the ids x*per, x*per + 1, ... in turn,
// all tile pairs of one K range run on one XCD and read that range's column
// slabs through its L2 once instead of once per XCD.  A bijection of the
// grid (ids past the last multiple of 8 keep their own number).  Used by the
// 128 x 128 kernels (paperlike fp4: 30.2 -> 4.9 GB fetched, same time); the
// 256 x 256 kernels measured 2-4 % slower with it and keep launch order.
constexpr uint64_t kXcds = 8;
__device__ __forceinline__ void xcd_pair_split(uint32_t &pair, uint64_t &split) {
    const uint64_t nx = gridDim.x, total = nx * gridDim.y;
    const uint64_t L = (uint64_t)blockIdx.y * nx + blockIdx.x;
    const uint64_t per = total / kXcds;
    const uint64_t V = L < per * kXcds ? (L % kXcds) * per + L / kXcds : L;
    pair = (uint32_t)(V % nx);
    split = V / nx;
}

// Thread (ty, tx) of a 16 x 16 grid owns rows 32c + 2ty + e and columns
// 32c + 2tx + e (c = 0..3, e = 0..1) of the 128 x 128 tile: every LDS read is
// a 16-byte load, consecutive lanes read consecutive 16-byte pieces.
__global__ __launch_bounds__(kNT) void k_gram_popc(const uint64_t *__restrict__ W, uint64_t ldw, uint64_t H,
                                                    uint64_t kper, uint32_t nt, uint32_t n,
                                                    int32_t *__restrict__ B, int upper) {
    __shared__ ulonglong2 As[kKC][kT / 2];
    __shared__ ulonglong2 Bs[kKC][kT / 2];
    // the (renumbered) block enumerates the tile pairs I <= J row by row, then the K ranges
    uint32_t p, I = 0, rowlen = nt;
    uint64_t split;
    xcd_pair_split(p, split);
    while (p >= rowlen) {
        p -= rowlen;
        ++I;
        --rowlen;
    }
    const uint32_t Jt = I + p;
    const uint32_t I0 = I * kT, J0 = Jt * kT;
    const uint64_t k0 = split * kper;
    const uint64_t k1 = min(H, k0 + kper);
    if (k0 >= k1) return;
    const uint32_t tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
    const bool diag = I == Jt;

    uint32_t acc[8][8];
#pragma unroll
    for (int x = 0; x < 8; ++x)
#pragma unroll
        for (int y = 0; y < 8; ++y) acc[x][y] = 0;

    // global -> register staging: 4 x 16 B per matrix per thread
    ulonglong2 ra[4], rb[4];
    auto gload = [&](uint64_t kb) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const uint32_t idx = tid + kNT * m;      // 0..1023
            const uint32_t kk = idx >> 6, cp = idx & 63;
            const uint64_t k = kb + kk;
            if (k < k1) {
                ra[m] = *reinterpret_cast<const ulonglong2 *>(W + k * ldw + I0 + 2 * cp);
                rb[m] = diag ? ra[m] : *reinterpret_cast<const ulonglong2 *>(W + k * ldw + J0 + 2 * cp);
            } else {
                ra[m] = make_ulonglong2(0, 0);
                rb[m] = make_ulonglong2(0, 0);
            }
        }
    };
    auto sstore = [&]() {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const uint32_t idx = tid + kNT * m;
            As[idx >> 6][idx & 63] = ra[m];
            Bs[idx >> 6][idx & 63] = rb[m];
        }
    };

    gload(k0);
    for (uint64_t kb = k0; kb < k1; kb += kKC) {
        __syncthreads();
        sstore();
        __syncthreads();
        if (kb + kKC < k1) gload(kb + kKC);
#pragma unroll 4
        for (int kk = 0; kk < kKC; ++kk) {
            uint64_t a[8], b[8];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const ulonglong2 va = As[kk][16 * c + ty];
                const ulonglong2 vb = Bs[kk][16 * c + tx];
                a[2 * c] = va.x;
                a[2 * c + 1] = va.y;
                b[2 * c] = vb.x;
                b[2 * c + 1] = vb.y;
            }
#pragma unroll
            for (int x = 0; x < 8; ++x)
#pragma unroll
                for (int y = 0; y < 8; ++y) {
                    const uint64_t v = a[x] & b[y];
                    acc[x][y] += __popc((uint32_t)v) + __popc((uint32_t)(v >> 32));
                }
        }
    }
    // epilogue: add the strict upper part of the tile into B
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        const uint32_t i = I0 + 32 * (x >> 1) + 2 * ty + (x & 1);
#pragma unroll
        for (int y = 0; y < 8; ++y) {
            const uint32_t j = J0 + 32 * (y >> 1) + 2 * tx + (y & 1);
            if (acc[x][y] && i < j && j < n) atomicAdd(B + out_index(i, j, n, upper), (int32_t)acc[x][y]);
        }
    }
}

// ---------------------------------------------------------------------------
// int8 MFMA form of the same product.  Each bit of a packed word becomes a
// 0/1 byte in registers (never in memory; through a 256-entry LDS table of
// byte patterns) and V_MFMA_I32_32X32X32_I8 sums the byte products in int32:
// sum_k a_ki a_kj over the 32 bits of a half word, exact (every partial sum
// is a count <= 2^31).  The K order inside the instruction does not matter:
// lane group g (lanes 32g..32g+31) feeds bits 16g..16g+15 of the half word
// for both operands, so every bit pairs with itself.
// Block = 2 waves over a 128 x 128 tile; wave c owns columns 64c..64c+63,
// i.e. 4 x 2 MFMA tiles of 32 x 32 (128 int32 accumulators per lane).
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kMfmaNT = 128;

// 8 bits -> 8 bytes (byte k = bit k), 256 entries: an operand of 16 bits is
// two table reads instead of a dozen VALU operations.
__device__ __forceinline__ void fill_byte_lut(unsigned long long *lut) {
    for (uint32_t i = threadIdx.x; i < 256; i += blockDim.x) {
        const unsigned long long lo = ((i & 0xFu) * 0x00204081u) & 0x01010101u;
        const unsigned long long hi = (((i >> 4) & 0xFu) * 0x00204081u) & 0x01010101u;
        lut[i] = lo | (hi << 32);
    }
}

__device__ __forceinline__ v4i bits16_lut(const unsigned long long *lut, uint32_t x) {
    const unsigned long long lo = lut[__builtin_amdgcn_ubfe(x, 0, 8)];
    const unsigned long long hi = lut[__builtin_amdgcn_ubfe(x, 8, 8)];
    v4i r;
    r[0] = (int)(uint32_t)lo;
    r[1] = (int)(uint32_t)(lo >> 32);
    r[2] = (int)(uint32_t)hi;
    r[3] = (int)(uint32_t)(hi >> 32);
    return r;
}

// STEP word rows per loop iteration; the next STEP rows are loaded while the
// current ones are multiplied.  WPE = waves per SIMD the register budget is
// sized for (2: 256 VGPRs).
template <int WPE, int STEP>
__global__ __launch_bounds__(kMfmaNT) __attribute__((amdgpu_waves_per_eu(WPE, WPE))) void k_gram_mfma(
    const uint64_t *__restrict__ W, uint64_t ldw, uint64_t H, uint64_t kper, uint32_t nt, uint32_t n,
    int32_t *__restrict__ B, int upper) {
    __shared__ unsigned long long lut[256];
    // the (renumbered) block enumerates the tile pairs I <= J row by row, then the K ranges
    uint32_t p, I = 0, rowlen = nt;
    uint64_t split;
    xcd_pair_split(p, split);
    while (p >= rowlen) {
        p -= rowlen;
        ++I;
        --rowlen;
    }
    const uint32_t Jt = I + p;
    const uint64_t k0 = split * kper;
    const uint64_t k1 = min(H, k0 + kper);
    if (k0 >= k1) return;
    fill_byte_lut(lut);
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63, wc = threadIdx.x >> 6;
    const uint32_t lm = lane & 31, lg = lane >> 5;
    const uint32_t I0 = I * kT, J0 = Jt * kT + 64 * wc;
    v16i acc[4][2];
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[x][y][r] = 0;

    const uint64_t *pa = W + I0 + lm;
    const uint64_t *pb = W + J0 + lm;
    // STEP word rows per iteration; the next STEP rows are loaded while these are multiplied
    uint64_t a[STEP][4], b[STEP][2];
#pragma unroll
    for (int u = 0; u < STEP; ++u) {
        const uint64_t ku = min(k0 + u, k1 - 1);
#pragma unroll
        for (int x = 0; x < 4; ++x) a[u][x] = pa[ku * ldw + 32 * x];
#pragma unroll
        for (int y = 0; y < 2; ++y) b[u][y] = pb[ku * ldw + 32 * y];
    }
    for (uint64_t k = k0; k < k1; k += STEP) {
        uint64_t na[STEP][4], nb[STEP][2];
#pragma unroll
        for (int u = 0; u < STEP; ++u) {
            const uint64_t kn = min(k + STEP + u, k1 - 1);
#pragma unroll
            for (int x = 0; x < 4; ++x) na[u][x] = pa[kn * ldw + 32 * x];
#pragma unroll
            for (int y = 0; y < 2; ++y) nb[u][y] = pb[kn * ldw + 32 * y];
        }
#pragma unroll
        for (int u = 0; u < STEP; ++u) {
            if (k + u >= k1) break;  // wave-uniform: the tail of the range
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t sh = 32 * h + 16 * lg;
                v4i va[4], vb[2];
#pragma unroll
                for (int x = 0; x < 4; ++x) va[x] = bits16_lut(lut, (uint32_t)(a[u][x] >> sh));
#pragma unroll
                for (int y = 0; y < 2; ++y) vb[y] = bits16_lut(lut, (uint32_t)(b[u][y] >> sh));
#pragma unroll
                for (int x = 0; x < 4; ++x)
#pragma unroll
                    for (int y = 0; y < 2; ++y)
                        acc[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(va[x], vb[y], acc[x][y], 0, 0, 0);
            }
        }
#pragma unroll
        for (int u = 0; u < STEP; ++u) {
#pragma unroll
            for (int x = 0; x < 4; ++x) a[u][x] = na[u][x];
#pragma unroll
            for (int y = 0; y < 2; ++y) b[u][y] = nb[u][y];
        }
    }
    // accumulator r of lane (lg, lm) holds row 8*(r/4) + 4*lg + r%4, column lm of each 32 x 32 tile
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const uint32_t i = I0 + 32 * x + 8 * (r >> 2) + 4 * lg + (r & 3);
                const uint32_t j = J0 + 32 * y + lm;
                const int32_t v = acc[x][y][r];
                if (v && i < j && j < n) atomicAdd(B + out_index(i, j, n, upper), v);
            }
}

// 256 x 256 tiles: four waves (2 x 2), each a 128 x 128 block of 16 MFMA
// tiles with its accumulators in the AGPRs (one wave per SIMD).  Against the
// 128 x 128 kernel this halves the words loaded per multiply (each column
// slab feeds twice the tiles) and expands 8 operands per 16 MFMAs instead of
// 6 per 8.  Columns at or past ldw (n rounded to 128) are clamped to a valid
// column; their products land outside j < n and are dropped.
constexpr int kWideT = 256;
constexpr int kWideNT = 256;

template <int STEP>
__global__ __launch_bounds__(kWideNT) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_gram_mfma_wide(
    const uint64_t *__restrict__ W, uint64_t ldw, uint64_t H, uint64_t kper, uint32_t nt, uint32_t n,
    int32_t *__restrict__ B, int upper) {
    __shared__ unsigned long long lut[256];
    const uint64_t split = blockIdx.y;
    uint32_t p = blockIdx.x, I = 0, rowlen = nt;
    while (p >= rowlen) {
        p -= rowlen;
        ++I;
        --rowlen;
    }
    const uint32_t Jt = I + p;
    const uint64_t k0 = split * kper;
    const uint64_t k1 = min(H, k0 + kper);
    if (k0 >= k1) return;
    fill_byte_lut(lut);
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint32_t lm = lane & 31, lg = lane >> 5;
    const uint32_t I0 = I * kWideT + 128 * (wv >> 1), J0 = Jt * kWideT + 128 * (wv & 1);
    if (I0 >= J0 + 128) return;  // the wave's block lies below the diagonal (no syncs follow)
    v16i acc[4][4];
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[x][y][r] = 0;
    uint64_t ca[4], cb[4];  // this lane's columns, clamped below ldw
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        ca[x] = min<uint64_t>(I0 + lm + 32 * x, ldw - 1);
        cb[x] = min<uint64_t>(J0 + lm + 32 * x, ldw - 1);
    }
    uint64_t a[STEP][4], b[STEP][4];
#pragma unroll
    for (int u = 0; u < STEP; ++u) {
        const uint64_t ku = min(k0 + u, k1 - 1);
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            a[u][x] = W[ku * ldw + ca[x]];
            b[u][x] = W[ku * ldw + cb[x]];
        }
    }
    for (uint64_t k = k0; k < k1; k += STEP) {
        uint64_t na[STEP][4], nb[STEP][4];
#pragma unroll
        for (int u = 0; u < STEP; ++u) {
            const uint64_t kn = min(k + STEP + u, k1 - 1);
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                na[u][x] = W[kn * ldw + ca[x]];
                nb[u][x] = W[kn * ldw + cb[x]];
            }
        }
#pragma unroll
        for (int u = 0; u < STEP; ++u) {
            if (k + u >= k1) break;  // wave-uniform: the tail of the range
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t sh = 32 * h + 16 * lg;
                v4i va[4], vb[4];
#pragma unroll
                for (int x = 0; x < 4; ++x) va[x] = bits16_lut(lut, (uint32_t)(a[u][x] >> sh));
#pragma unroll
                for (int y = 0; y < 4; ++y) vb[y] = bits16_lut(lut, (uint32_t)(b[u][y] >> sh));
#pragma unroll
                for (int x = 0; x < 4; ++x)
#pragma unroll
                    for (int y = 0; y < 4; ++y)
                        acc[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(va[x], vb[y], acc[x][y], 0, 0, 0);
            }
        }
#pragma unroll
        for (int u = 0; u < STEP; ++u)
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                a[u][x] = na[u][x];
                b[u][x] = nb[u][x];
            }
    }
    // accumulator r of lane (lg, lm) holds row 8*(r/4) + 4*lg + r%4, column lm of each 32 x 32 tile
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 4; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const uint32_t i = I0 + 32 * x + 8 * (r >> 2) + 4 * lg + (r & 3);
                const uint32_t j = J0 + 32 * y + lm;
                const int32_t v = acc[x][y][r];
                if (v && i < j && j < n) atomicAdd(B + out_index(i, j, n, upper), v);
            }
}

// The same 128 x 128 tiles on the fp4 form of the scaled MFMA
// (V_MFMA_F32_32X32X64_F8F6F4, both operands e2m1): one 64-bit word is one
// K = 64 step, 32 bits per lane group (lanes 32g..32g+31 read half g of the
// word).  The lanes' k order is the same for both operands, so the dot
// product is the popcount of the AND.  Products are 0 or 1 and the float32 sums stay below 2^24
// (at most kFp4MaxK word rows per block), so every count is exact.
constexpr uint64_t kFp4MaxK = (1u << 24) / 64 - 1;
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

// A lane expands its 32 bits by masks alone, in registers: nibble i of operand
// dword r holds bit 4i + r, so each dword is one AND (after a shift where the
// bit has to move).  A bit that stays where it is in its nibble stands for
// 0.5, 1.0 or 2.0 (e2m1 0b0001, 0b0010, 0b0100), so the A form takes 0.5, 1,
// 2, 2 for r = 0..3 and the B form the inverses 2, 1, 0.5, 0.5: every product
// of two set bits is exactly 1.  5 and 7 VALU operations per 32 bits; looking
// 8 bits at a time up in an LDS table took 4 reads and as many address
// operations and left the matrix units waiting.
__device__ __forceinline__ v8i expand_a(uint32_t x) {
    v8i r = {0, 0, 0, 0, 0, 0, 0, 0};
    r[0] = (int)(x & 0x11111111u);
    r[1] = (int)(x & 0x22222222u);
    r[2] = (int)(x & 0x44444444u);
    r[3] = (int)((x >> 1) & 0x44444444u);
    return r;
}
__device__ __forceinline__ v8i expand_b(uint32_t x) {
    v8i r = {0, 0, 0, 0, 0, 0, 0, 0};
    r[0] = (int)((x << 2) & 0x44444444u);
    r[1] = (int)(x & 0x22222222u);
    r[2] = (int)((x >> 2) & 0x11111111u);
    r[3] = (int)((x >> 3) & 0x11111111u);
    return r;
}

typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// A wave's TA x TB MFMA tiles (TA, TB even) over word rows [k0, k1) of W.
// Lane group g takes row g of each pair of rows: a lane loads 16 bytes, the
// words of two adjacent columns, which serve two tiles and two MFMA steps
// (the low, then the high halves), so a pair of rows takes (TA + TB) / 2
// loads.  Tile x's row m is column 64 (x / 2) + 2 m + x % 2 of the wave's
// block (fp4_add undoes it).  A pair is read through a buffer descriptor of
// its own: the address is wave-uniform, a lane adds a 32-bit offset (oa, ob:
// its columns' bytes, plus one row for group 1), and the descriptor ends with
// row k1, so rows past it read as zeros and add nothing.  D pairs are in
// flight; a step's operands are expanded while the step before it is in the
// matrix unit.
template <int TA, int TB, int D>
__device__ __forceinline__ void fp4_block(const uint64_t *__restrict__ W, uint64_t ldw, uint64_t k0, uint64_t k1,
                                          const uint32_t (&oa)[TA / 2], const uint32_t (&ob)[TB / 2],
                                          v16f (&acc)[TA][TB]) {
#pragma unroll
    for (int x = 0; x < TA; ++x)
#pragma unroll
        for (int y = 0; y < TB; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;
    const uint32_t rows = (uint32_t)(k1 - k0), bytes = (uint32_t)(ldw * 8);
    const uint64_t *p = W + k0 * ldw;
    v4u ra[D][TA / 2], rb[D][TB / 2];
    const auto load = [&](uint32_t q, v4u (&a)[TA / 2], v4u (&b)[TB / 2]) {
        const uint32_t left = 2 * q < rows ? rows - 2 * q : 0;  // rows from this pair on
        const auto pair = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint64_t *>(p + (uint64_t)(2 * q) * ldw), 0,
                                                            min(left, 2u) * bytes, 0x00020000);
#pragma unroll
        for (int x = 0; x < TA / 2; ++x) a[x] = __builtin_amdgcn_raw_buffer_load_b128(pair, oa[x], 0, 0);
#pragma unroll
        for (int y = 0; y < TB / 2; ++y) b[y] = __builtin_amdgcn_raw_buffer_load_b128(pair, ob[y], 0, 0);
    };
    v8i va[TA], vb[TB];  // operands of the step about to be multiplied
    const auto step = [&](const v4u (&a)[TA / 2], const v4u (&b)[TB / 2], int h) {
        v8i wa[TA], wb[TB];  // operands of the step after it: half h of a pair's words
#pragma unroll
        for (int x = 0; x < TA; ++x) wa[x] = expand_a(a[x / 2][2 * (x & 1) + h]);
#pragma unroll
        for (int y = 0; y < TB; ++y) wb[y] = expand_b(b[y / 2][2 * (y & 1) + h]);
#pragma unroll
        for (int x = 0; x < TA; ++x)
#pragma unroll
            for (int y = 0; y < TB; ++y)
                acc[x][y] =
                    __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(va[x], vb[y], acc[x][y], 4, 4, 0, 0, 0, 0);
        // issue order: an MFMA, then its share of the masks
#pragma unroll
        for (int m = 0; m < TA * TB; ++m) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x002, (5 * TA + 7 * TB + TA * TB - 1) / (TA * TB), 0);
        }
#pragma unroll
        for (int x = 0; x < TA; ++x) va[x] = wa[x];
#pragma unroll
        for (int y = 0; y < TB; ++y) vb[y] = wb[y];
    };
#pragma unroll
    for (int s = 0; s < D; ++s) load(s, ra[s], rb[s]);
#pragma unroll
    for (int x = 0; x < TA; ++x) va[x] = expand_a(ra[0][x / 2][2 * (x & 1)]);
#pragma unroll
    for (int y = 0; y < TB; ++y) vb[y] = expand_b(rb[0][y / 2][2 * (y & 1)]);
    for (uint32_t q = 0; 2 * q < rows; q += D) {
#pragma unroll
        for (int s = 0; s < D; ++s) {
            step(ra[s], rb[s], 1);  // multiplies the low halves of pair q + s
            load(q + s + D, ra[s], rb[s]);
            step(ra[(s + 1) % D], rb[(s + 1) % D], 0);  // its high halves
        }
    }
}

// Adds a wave's tiles at (I0, J0) into the strict upper part of B:
// accumulator r of lane (lg, lm) holds row 8*(r/4) + 4*lg + r%4, column lm of
// each 32 x 32 tile, and a pair of tiles holds every other column each.  With
// kTrade the lanes trade values so that an addition of 32 lanes covers 32 columns
// in a row instead of every other one of 64: 0.19 ms for 0.30 where 3160 tile pairs
// of 16 word rows are hardly more than additions, 0.23 for 0.34 with 94 rows.
// Blocks of kTradeRows word rows or more go without (65 K rows: 57.6 ms, 57.9 with).
constexpr uint64_t kTradeRows = 1024;
template <bool kTrade, int TA, int TB>
__device__ __forceinline__ void fp4_add(const v16f (&acc)[TA][TB], uint32_t I0, uint32_t J0, uint32_t lm, uint32_t lg,
                                        uint32_t n, int32_t *__restrict__ B, int upper) {
    const int from = (int)(32 * lg + lm / 2);  // the lane with columns lm & ~1 and lm | 1 of the pair's first half
#pragma unroll
    for (int x = 0; x < TA; ++x)
#pragma unroll
        for (int y = 0; y < TB; y += 2) {
            bool some = true;
            if constexpr (kTrade) {  // a plan's word rows may be empty
                uint32_t bits = 0;
#pragma unroll
                for (int r = 0; r < 16; ++r) bits |= __float_as_uint(acc[x][y][r]) | __float_as_uint(acc[x][y + 1][r]);
                some = __ballot(bits != 0) != 0;
            }
#pragma unroll
            for (int r0 = 0; r0 < 16; r0 += 4) {
                const uint32_t i0 = I0 + 64 * (x >> 1) + 4 * r0 + (x & 1);  // the first of these rows
                float c[4][2];
                if constexpr (kTrade) {  // columns 0..31, then 32..63 of the pair; eight trades in flight
                    if (!some || i0 >= n || J0 + 32 * y >= n) continue;
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const float even = __shfl(acc[x][y][r0 + r], from + 16 * h, kWave);
                            const float odd = __shfl(acc[x][y + 1][r0 + r], from + 16 * h, kWave);
                            c[r][h] = lm & 1 ? odd : even;
                        }
                }
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const uint32_t i = i0 + 8 * lg + 2 * r;
                        const uint32_t j = kTrade ? J0 + 32 * (y + h) + lm : J0 + 32 * y + 2 * lm + h;
                        const int32_t v = (int32_t)(kTrade ? c[r][h] : acc[x][y + h][r0 + r]);  // an exact integer below 2^24
                        if (v && i < j && j < n) atomicAdd(B + out_index(i, j, n, upper), v);
                    }
            }
        }
}

// 128 x 128 tiles, two waves of 128 x 64 each, two waves per SIMD (232 VGPRs),
// so one wave's loads and masks run beside the other's MFMAs.  On a diagonal
// tile the first wave's lower half lies below the diagonal and is not
// computed.  Bound by the matrix unit: 7.1 to 7.9 PF/s of 10.1 (n = 1024,
// 1.25 M word rows: 20.9 -> 11.4 ms against the LDS-table form; n = 4096, 65 K:
// 16.9 -> 10.0; n = 10000, 65 K: 96 -> 57.6).  256 x 256 tiles of four 128 x 128
// waves, one per SIMD, reach 6.5: nothing runs beside a wave that waits.
constexpr int kFp4Pairs = 4;  // row pairs in flight (3, 4 and 6 measured alike)
template <bool kTrade>
__global__ __launch_bounds__(kMfmaNT) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gram_fp4(
    const uint64_t *__restrict__ W, uint64_t ldw, uint64_t H, uint64_t kper, uint32_t nt, uint32_t n,
    int32_t *__restrict__ B, int upper) {
    uint32_t p, I = 0, rowlen = nt;
    uint64_t split;
    xcd_pair_split(p, split);
    while (p >= rowlen) {
        p -= rowlen;
        ++I;
        --rowlen;
    }
    const uint32_t Jt = I + p;
    const uint64_t k0 = split * kper;
    const uint64_t k1 = min(H, k0 + kper);
    if (k0 >= k1) return;
    const uint32_t lane = threadIdx.x & 63, wc = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t lm = lane & 31, lg = lane >> 5;
    const uint32_t I0 = I * kT, J0 = Jt * kT + 64 * wc;
    const uint32_t row = lg * (uint32_t)ldw * 8;
    const uint32_t oa[2] = {row + 8 * (I0 + 2 * lm), row + 8 * (I0 + 64 + 2 * lm)}, ob[1] = {row + 8 * (J0 + 2 * lm)};
    if (J0 == I0) {
        const uint32_t oh[1] = {oa[0]};
        v16f acc[2][2];
        fp4_block<2, 2, kFp4Pairs>(W, ldw, k0, k1, oh, ob, acc);
        fp4_add<kTrade, 2, 2>(acc, I0, J0, lm, lg, n, B, upper);
        return;
    }
    v16f acc[4][2];
    fp4_block<4, 2, kFp4Pairs>(W, ldw, k0, k1, oa, ob, acc);
    fp4_add<kTrade, 4, 2>(acc, I0, J0, lm, lg, n, B, upper);
}

// Row lists: one thread per row, every pair of its (ascending) samples.
__global__ void k_list_pairs(const uint64_t *__restrict__ lp, const uint32_t *__restrict__ ls, uint64_t nl,
                             uint32_t n, int32_t *__restrict__ B, int upper) {
    for (uint64_t r = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; r < nl; r += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t a0 = lp[r], a1 = lp[r + 1];
        for (uint64_t a = a0; a < a1; ++a) {
            const uint32_t i = ls[a];
            for (uint64_t b = a + 1; b < a1; ++b) atomicAdd(B + out_index(i, ls[b], n, upper), 1);
        }
    }
}

// Row-list pairs sorted by their smaller sample a: block g takes pairs
// [g*chunk, ...).  For each run of one a in it of at least n/8 words (and
// kPairRun), an LDS row cnt[b] counts the rows holding both a and b, and each
// touched counter is added to row a of B once (one atomic per touched pair and
// chunk instead of one per row and pair).  A shorter run touches few counters
// twice, and finding its end, waiting and looking through the counters take longer
// than its own atomics on B (0.5 us a run: 778 K words of 8192 samples 0.19 ms, and
// 0.028 directly), so the words up to the next long run go to B all at once.
// Neighbours that are equal are added together: atomics on one word of B take 11 ns
// each, one after another (two samples of 10000 that share 3 M rows of their own:
// 34 ms with every word by itself, 0.04 ms so; 1 M words on 500 pairs 0.12 and
// 0.013 ms).
// Chunks of at least kPairChunk words (and n/8, so that a run that fills its
// chunk is counted in LDS), at most kPairBlocks of them: longer chunks split a
// sample's run fewer times, so fewer atomics, but a block takes its long runs one
// after another.  1.7 G words of 10000 samples: 1.9 ms.
constexpr uint64_t kPairChunk = 1024;
constexpr uint64_t kPairBlocks = 4096;
constexpr uint64_t kPairRun = 512;
static_assert(kPairRun <= kPairChunk, "a chunk of one run is counted in LDS");

constexpr int kPairCountNT = 512;  // threads per pair-count block (one LDS row of counters each)
__global__ __launch_bounds__(kPairCountNT) void k_pair_count(const uint32_t *__restrict__ pairs, uint64_t P, uint64_t chunk,
                                                     uint32_t n, int32_t *__restrict__ B, int upper,
                                                     const uint64_t *__restrict__ dsz) {
    extern __shared__ uint32_t lds[];
    uint32_t *cnt = lds;  // n counters
    __shared__ uint64_t seg_end;
    __shared__ uint32_t next_run;
    if (dsz) P = min(P, dsz[PZ_P]);  // a plan's db: P is the capacity, the count is on the device
    const uint64_t lo = (uint64_t)blockIdx.x * chunk, hi = min(P, lo + chunk);
    if (lo >= hi) return;
    // words [p0, p1) straight to B, the first of equal neighbours in a wave for all of them
    const auto add = [&](uint64_t p0, uint64_t p1) {
        for (uint64_t p = p0 + threadIdx.x; p - threadIdx.x < p1; p += blockDim.x) {  // uniform
            const bool have = p < p1;
            const uint32_t w = have ? pairs[p] : ~0u;  // (no word: a < b)
            const uint32_t before = wave_shift_up(w);
            const bool first = lane_id() == 0 || before != w;
            const uint64_t after = __ballot(first) & ~(lanemask_lt() | (uint64_t(1) << lane_id()));
            const uint32_t c = (after ? (uint32_t)__builtin_ctzll(after) : (uint32_t)kWave) - lane_id();
            if (first && have) atomicAdd(B + out_index(w >> 16, w & 0xFFFFu, n, upper), (int32_t)c);
        }
    };
    const uint64_t far = max((uint64_t)(n + 7) / 8, kPairRun);  // <= chunk
    bool cleared = false;
    for (uint64_t s0 = lo; s0 < hi;) {
        const uint32_t a = pairs[s0] >> 16;
        if (hi - s0 < far || (pairs[s0 + far - 1] >> 16) != a) {  // block-uniform
            // a short run: on to the first of the places far words apart from which a
            // sample goes on for as long (twice as long a run holds such a place)
            if (threadIdx.x == 0) next_run = (uint32_t)(hi - lo);
            __syncthreads();
            for (uint64_t p = s0 + (threadIdx.x + 1) * far; p + far <= hi; p += blockDim.x * far)
                if ((pairs[p] >> 16) == (pairs[p + far - 1] >> 16)) atomicMin(&next_run, (uint32_t)(p - lo));
            __syncthreads();
            const uint64_t s1 = lo + next_run;
            add(s0, s1);
            s0 = s1;
            __syncthreads();  // next_run is read
            continue;
        }
        if (!cleared) {
            for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) cnt[i] = 0;  // (the barrier below)
            cleared = true;
        }
        // end of the run of a inside the chunk (the chunk is sorted by a): the
        // first wave narrows [l, h] by 64 probes per step; positions before l
        // hold samples <= a, positions from h on samples > a
        if (threadIdx.x < kWave) {
            const uint32_t lane = threadIdx.x;
            uint64_t l = s0 + 1, h = hi;
            while (h - l > kWave) {
                const uint64_t step = (h - l) / kWave;  // >= 1; probe 64 is l + 64*step <= h
                const uint64_t m = l + (lane + 1) * step;
                const uint64_t gt = __ballot(m >= h || (pairs[m] >> 16) > a);
                if (gt == 0) {
                    l = l + kWave * step + 1;
                } else {
                    const uint32_t k = (uint32_t)__builtin_ctzll(gt);  // probe k+1 is the first above
                    h = min(h, l + (k + 1) * step);
                    if (k > 0) l = l + k * step + 1;
                }
            }
            const uint64_t m = l + lane;
            const uint64_t gt = __ballot(m < h && (pairs[m] >> 16) > a);
            if (lane == 0) seg_end = gt ? l + __builtin_ctzll(gt) : h;
        }
        __syncthreads();
        const uint64_t s1 = seg_end;
        // Words are read 16 bytes at a time (four per thread in flight); the
        // buffer is 16-byte aligned, the unaligned ends by word.
        const auto count = [&](uint32_t w) {
            __hip_atomic_fetch_add(&cnt[w & 0xFFFFu], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        };
        const uint64_t va = min(s1, (s0 + 3) & ~uint64_t(3));  // first aligned word (or s1)
        const uint64_t vb = max(va, s1 & ~uint64_t(3));        // end of the aligned body
        for (uint64_t p = s0 + threadIdx.x; p < va; p += blockDim.x) count(pairs[p]);
        for (uint64_t p = vb + threadIdx.x; p < s1; p += blockDim.x) count(pairs[p]);
        const uint4 *pv = reinterpret_cast<const uint4 *>(pairs);
        const uint64_t q1 = vb / 4;
        for (uint64_t q0 = va / 4; q0 < q1; q0 += 4 * (uint64_t)blockDim.x) {
            uint4 x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint64_t q = q0 + (uint64_t)u * blockDim.x + threadIdx.x;
                if (q < q1) x[u] = pv[q];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (q0 + (uint64_t)u * blockDim.x + threadIdx.x < q1) {
                    count(x[u].x);
                    count(x[u].y);
                    count(x[u].z);
                    count(x[u].w);
                }
            }
        }
        __syncthreads();
        for (uint32_t b = a + 1 + threadIdx.x; b < n; b += blockDim.x) {
            const uint32_t c = cnt[b];
            if (c) {
                atomicAdd(B + out_index(a, b, n, upper), (int32_t)c);
                cnt[b] = 0;
            }
        }
        s0 = s1;
        __syncthreads();
    }
}

// Diagonal, mirror (full layout), unions and J.
// dst[i] += src[i], i < n (the sample sizes of one row batch into the running sums).
__global__ void k_add_i64(int64_t *__restrict__ dst, const int64_t *__restrict__ src, uint32_t n) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] += src[i];
}

// flag[0] = 1 when some card[i] >= limit.
__global__ void k_card_check(const int64_t *__restrict__ card, uint32_t n, int64_t limit, uint32_t *flag) {
    bool over = false;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        over |= card[i] >= limit;
    if (__ballot(over) && lane_id() == 0) atomicOr(flag, 1u);
}

__global__ void k_zero_flag(uint32_t *flag) { *flag = 0; }

// Full layout: a block per 64 x 64 tile of the upper triangle (in rows of
// tiles: tile row x, then its n/64 - x tiles), which writes that tile and its
// mirror image.  Memory bound: 4 bytes read and 8 to 36 written per pair; the
// tile goes through LDS so that the mirror's writes run along rows too, and B
// is read once.  n = 8192 with J: 0.54 ms a row at a time
// (the mirror half read B down columns), 0.27 ms by tiles, 0.23 with stores
// that do not stay in the caches (0.30 with 16 rows of tiles at a time, column by
// column).
constexpr uint32_t kFinT = 64;
constexpr int kFinNT = 256;
__global__ __launch_bounds__(kFinNT) void k_finalize(int32_t *__restrict__ B, const int64_t *__restrict__ card,
                                                     uint32_t n, uint32_t nt, int64_t *__restrict__ den,
                                                     double *__restrict__ J) {
    constexpr uint32_t kRows = kFinNT / kWave, kSteps = kFinT / kRows;
    __shared__ int32_t tile[kFinT][kFinT + 1];
    __shared__ int64_t ci[kFinT], cj[kFinT];
    // the tile: rows 0 .. x-1 hold x * nt - x (x - 1) / 2 of them
    const double h = nt + 0.5;
    uint32_t x = (uint32_t)max(0.0, h - sqrt(h * h - 2.0 * (double)blockIdx.x));
    const auto before = [&](uint32_t r) { return (uint64_t)r * nt - (uint64_t)r * (r - (r ? 1u : 0u)) / 2; };
    while (x > 0 && before(x) > blockIdx.x) --x;
    while (before(x + 1) <= blockIdx.x) ++x;
    const uint32_t y = x + (uint32_t)(blockIdx.x - before(x));
    const uint32_t i0 = x * kFinT, j0 = y * kFinT, lane = lane_id(), w = threadIdx.x / kWave;
    if (threadIdx.x < kFinT) ci[threadIdx.x] = i0 + threadIdx.x < n ? card[i0 + threadIdx.x] : 0;
    else if (threadIdx.x < 2 * kFinT) cj[lane] = j0 + lane < n ? card[j0 + lane] : 0;
    int32_t v[kSteps];
#pragma unroll
    for (uint32_t k = 0; k < kSteps; ++k) {
        const uint32_t i = i0 + k * kRows + w, j = j0 + lane;
        v[k] = i < j && j < n ? B[(uint64_t)i * n + j] : 0;
    }
#pragma unroll
    for (uint32_t k = 0; k < kSteps; ++k) tile[k * kRows + w][lane] = v[k];
    __syncthreads();
    const auto put = [&](uint32_t i, uint32_t j, int64_t b, int64_t ca, int64_t cb) {
        const uint64_t pos = (uint64_t)i * n + j;
        const int64_t c = ca + cb - b;
        if (den) __builtin_nontemporal_store(c, den + pos);
        if (J) __builtin_nontemporal_store(c == 0 ? 1.0 : (double)b / (double)c, J + pos);
    };
#pragma unroll 4
    for (uint32_t k = 0; k < kSteps; ++k) {
        const uint32_t r = k * kRows + w, i = i0 + r, j = j0 + lane;
        if (i > j || j >= n) continue;
        const int64_t b = i == j ? ci[r] : tile[r][lane];
        if (i == j) B[(uint64_t)i * n + i] = (int32_t)b;
        put(i, j, b, ci[r], cj[lane]);
    }
#pragma unroll 4
    for (uint32_t k = 0; k < kSteps; ++k) {  // row j of the mirror image, column i
        const uint32_t r = k * kRows + w, j = j0 + r, i = i0 + lane;
        if (i >= j || j >= n) continue;
        const int32_t b = tile[lane][r];
        B[(uint64_t)j * n + i] = b;
        put(j, i, b, cj[r], ci[lane]);
    }
}

// Packed upper layout: rows i and n-1-i share a row of blocks over their
// n - i and i + 1 entries (n + 1 in all), so no thread of the grid is idle.
// kFinPer entries per thread, their loads in flight together: n = 10000 with J
// 0.246 ms one at a time, 0.231 so (600 MB).
constexpr uint32_t kFinPer = 4;
__global__ __launch_bounds__(kFinNT) void k_finalize_upper(int32_t *__restrict__ B, const int64_t *__restrict__ card,
                                                           uint32_t n, uint32_t jblocks, int64_t *__restrict__ den,
                                                           double *__restrict__ J) {
    const uint32_t i0 = blockIdx.x / jblocks, i1 = n - 1 - i0;
    const uint32_t t0 = (blockIdx.x % jblocks) * kFinNT * kFinPer + threadIdx.x;
    const uint32_t len0 = n - i0;  // entries of row i0
    const uint32_t len = i0 == i1 ? len0 : n + 1;
    const uint64_t row0 = out_index(i0, i0, n, true), row1 = out_index(i1, i1, n, true);
    const int64_t c0 = card[i0], c1 = card[i1];
    int32_t v[kFinPer];
    int64_t cj[kFinPer];
#pragma unroll
    for (uint32_t k = 0; k < kFinPer; ++k) {
        const uint32_t t = t0 + k * kFinNT;
        const bool first = t < len0;
        v[k] = t < len ? B[first ? row0 + t : row1 + (t - len0)] : 0;
        cj[k] = t < len ? card[first ? i0 + t : i1 + (t - len0)] : 0;
    }
#pragma unroll
    for (uint32_t k = 0; k < kFinPer; ++k) {
        const uint32_t t = t0 + k * kFinNT;
        if (t >= len) break;
        const bool first = t < len0;
        const uint32_t off = first ? t : t - len0;  // column minus row
        const uint64_t pos = (first ? row0 : row1) + off;
        const int64_t ci = first ? c0 : c1, b = off ? v[k] : ci;
        if (off == 0) B[pos] = (int32_t)b;
        const int64_t c = ci + cj[k] - b;
        if (den) __builtin_nontemporal_store(c, den + pos);
        if (J) __builtin_nontemporal_store(c == 0 ? 1.0 : (double)b / (double)c, J + pos);
    }
}

// Tile variants of the MFMA Gram: word rows per step of the int8 K loops, and
// how many blocks the K split aims for (int8: at least that many; fp4: at most,
// or 0: the split fp4_split chooses).  The autotuner (JAS_TUNE) times each on
// the caller's db and keeps the fastest for dbs of the same shape: the fixed
// numbers of blocks are there for shapes on which the fitted rule is off (n = 60
// with 65 K word rows: 0.056 ms, 0.051 with 512 blocks; most shapes by less than
// the noise), for a program that multiplies many of one shape.
enum GramKind { kInt8 = 0, kInt8Wide = 1, kFp4 = 2 };
struct GramVariant {
    int step;
    uint64_t want_blocks;
    int kind;  // kInt8: k_gram_mfma; kInt8Wide: 256 x 256 tiles (k_gram_mfma_wide); kFp4: k_gram_fp4
};
// (int8 variants aimed at 1024 blocks, or with 2 rows per step at 2048, measured
// slower everywhere and are not listed)
constexpr GramVariant kVariants[] = {{4, 2048, kInt8},     {4, 4096, kInt8}, {2, 4096, kInt8},  {4, 4096, kInt8Wide},
                                     {4, 8192, kInt8Wide}, {2, 0, kFp4},     {2, 512, kFp4},    {2, 1024, kFp4},
                                     {2, 2048, kFp4},      {2, 3072, kFp4},  {2, 4096, kFp4},   {2, 6144, kFp4},
                                     {2, 8192, kFp4},      {2, 12288, kFp4}, {2, 16384, kFp4},  {2, 24576, kFp4},
                                     {2, 32768, kFp4}};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);
constexpr int kDefaultVariant = 5;  // untuned
static_assert(kVariants[kDefaultVariant].kind == kFp4 && kVariants[kDefaultVariant].want_blocks == 0, "default");

std::mutex g_tune_mu;
std::map<std::tuple<int, uint32_t, uint32_t>, int> g_tuned;  // (device, n, ceil(log2 H)) -> variant

void k_split(uint64_t H, uint64_t np, uint64_t want, uint64_t &kper, uint64_t &splits) {
    splits = std::max<uint64_t>(1, div_up(want, np));
    kper = div_up(H, splits);
    kper = std::max<uint64_t>(kper, 64);
    kper = div_up(kper, kKC) * kKC;
    splits = div_up(H, kper);
    if (splits > 65535) {
        splits = 65535;
        kper = div_up(div_up(H, splits), kKC) * kKC;
        splits = div_up(H, kper);
    }
}

// The K split of the fp4 kernel over np tile pairs and H word rows: word rows
// per block (a multiple of kKC) and blocks per tile pair.  kFp4Slots blocks run
// at once, so the grid takes ceil(blocks / kFp4Slots) rounds, each of the time a
// block takes for its rows, and the blocks drift apart by up to one block's time.
// Fewer rounds are fewer additions to B, but a last round that is nearly empty
// costs a whole one (n = 1024: 36 x 114 = 4104 blocks take 13.6 ms, 36 x 113
// 12.8), and long blocks drift out of step and share less of their XCD's L2 (1
// round 13.4 ms, 8 rounds 12.4, 24 rounds 11.4; less so where more tile pairs than
// slots share a range of rows).  A block's additions take kBlockUs of the chip's
// time whatever its length, more where all blocks add to one tile.  Over long
// grids they hide behind the multiplications (the two times add up like the sides
// of a right angle, nearly enough), but with few rows they are nearly all there
// is: blocks of 16 rows that fill the slots took 0.171 ms (n = 128, 16 K word
// rows), 0.040 as 128 blocks now, and 0.076 (n = 1024, 313), now 0.027.
// The split with the least modelled time is taken, of those that fill 1/64 to 7/8
// of the slots or a whole number of rounds.  The constants are fitted to 82
// products of n = 10 to 10000 and 13 to 65 K word rows at up to 18 splits each;
// over 198 of n = 3 to 10000 the split taken is at most 1.4 times the best, 1.04 on
// average.
constexpr uint64_t kFp4Slots = 256 * 4;  // blocks resident: two waves of 232 VGPRs each, eight waves per CU
constexpr uint64_t kFp4Rounds = 64;      // most rounds considered
constexpr uint64_t kFp4Part[] = {16, 21, 32, 42, 64, 85, 128, 170, 256, 341, 384, 512, 640, 768, 896};  // of a round
constexpr double kRowUs = 0.20, kRowFullUs = 0.08;      // a word row of a block; more with every slot in use
constexpr double kBlockUs = 0.07, kBlockTileUs = 0.02;  // a block's additions; more, per tile pair, with few of them

void fp4_split(uint64_t H, uint64_t np, uint64_t want, uint64_t &kper, uint64_t &splits) {
    const auto rows = [&](uint64_t sp) { return std::min(div_up(div_up(H, sp), kKC) * kKC, kFp4MaxK / kKC * kKC); };
    uint64_t best = 1;
    if (want) {
        best = std::max<uint64_t>(1, want / np);
    } else {
        double best_t = INFINITY;
        const auto consider = [&](uint64_t grid) {
            const uint64_t sp = std::max<uint64_t>(1, std::min(grid / np, div_up(H, kKC)));
            const uint64_t k = rows(sp), blocks = div_up(H, k) * np;
            const double drift = (double)std::min(k, H * np / kFp4Slots / 8) * std::min(1.0, (double)kFp4Slots / np);
            const double row = kRowUs + kRowFullUs * std::min(1.0, (double)blocks / kFp4Slots);
            const double multiply = ((double)(div_up(blocks, kFp4Slots) * k) + drift) * row;
            const double add = (double)blocks * (kBlockUs + kBlockTileUs / (double)np);
            const double time = std::hypot(multiply, add);
            if (time < best_t) {
                best_t = time;
                best = sp;
            }
        };
        for (const uint64_t grid : kFp4Part) consider(grid);
        for (uint64_t r = 1; r <= kFp4Rounds; ++r) consider(r * kFp4Slots);
    }
    kper = rows(best);
    splits = div_up(H, kper);
}

void launch_mfma(const jas_db *db, int v, hipStream_t s, int32_t *B, bool upper) {
    const uint32_t n = (uint32_t)db->n;
    const uint64_t ldw = div_up(n, 128) * 128;
    uint64_t kper, splits;
    if (kVariants[v].kind == kInt8Wide) {
        const uint32_t nt = (uint32_t)div_up(n, kWideT);
        const uint64_t np = (uint64_t)nt * (nt + 1) / 2;
        k_split(db->H, np, kVariants[v].want_blocks, kper, splits);
        dim3 grid((uint32_t)np, (uint32_t)splits);
        k_gram_mfma_wide<4><<<grid, kWideNT, 0, s>>>(db->W.p, ldw, db->H, kper, nt, n, B, upper);  // 4 rows per step
        return;
    }
    const uint32_t nt = (uint32_t)div_up(n, kT);
    const uint64_t np = (uint64_t)nt * (nt + 1) / 2;
    // a pair of rows has to be within the 32-bit offsets of a buffer descriptor
    if (kVariants[v].kind == kFp4 && ldw <= 0xFFFFFFFFull / 16) {
        fp4_split(db->H, np, kVariants[v].want_blocks, kper, splits);
        if (splits <= 65535) {
            dim3 grid((uint32_t)np, (uint32_t)splits);
            if (kper < kTradeRows) k_gram_fp4<true><<<grid, kMfmaNT, 0, s>>>(db->W.p, ldw, db->H, kper, nt, n, B, upper);
            else k_gram_fp4<false><<<grid, kMfmaNT, 0, s>>>(db->W.p, ldw, db->H, kper, nt, n, B, upper);
            return;
        }
    }
    // (fp4: a grid too large, the int8 kernel)
    k_split(db->H, np, std::max<uint64_t>(kVariants[v].want_blocks, 2048), kper, splits);
    dim3 grid((uint32_t)np, (uint32_t)splits);
    if (kVariants[v].step == 4)
        k_gram_mfma<2, 4><<<grid, kMfmaNT, 0, s>>>(db->W.p, ldw, db->H, kper, nt, n, B, upper);
    else
        k_gram_mfma<2, 2><<<grid, kMfmaNT, 0, s>>>(db->W.p, ldw, db->H, kper, nt, n, B, upper);
}

}  // namespace

int32_t gram_variants() { return kNumVariants; }

void finalize(uint32_t n, bool upper, hipStream_t s, int32_t *B, const int64_t *card, int64_t *den, double *J) {
    if (n == 0) return;
    if (upper) {
        // pairs of rows (i, n-1-i), the middle row alone when n is odd
        const uint32_t jb = (uint32_t)div_up((uint64_t)n + 1, kFinNT * kFinPer);
        const uint64_t fb = div_up((uint64_t)n, 2) * jb;
        if (div_up((uint64_t)n, 2) * div_up((uint64_t)n + 1, 256) > 0xFFFFFFFFull)
            fail(JAS_EUNSUPPORTED, "n too large for finalize grid");
        JAS_TIMED("finalize", s);
        k_finalize_upper<<<(uint32_t)fb, kFinNT, 0, s>>>(B, card, n, jb, den, J);
    } else {
        const uint32_t nt = (uint32_t)div_up(n, kFinT);
        const uint64_t fb = (uint64_t)nt * (nt + 1) / 2;
        if ((uint64_t)n * div_up(n, 256) > 0xFFFFFFFFull) fail(JAS_EUNSUPPORTED, "n too large for finalize grid");
        JAS_TIMED("finalize", s);
        k_finalize<<<(uint32_t)fb, kFinNT, 0, s>>>(B, card, n, nt, den, J);
    }
    check_launch("finalize");
}

void check_card_limit(const int64_t *card, uint32_t n, hipStream_t s) {
    if (n == 0) return;
    DevBuf<uint32_t> flag;
    flag.alloc(1, s, nullptr, true, "overflow flag");
    {
        JAS_TIMED("card_check", s);
        k_zero_flag<<<1, 1, 0, s>>>(flag.p);
        k_card_check<<<(uint32_t)std::min<uint64_t>(div_up(n, 256), 1024), 256, 0, s>>>(card, n,
                                                                                        (int64_t)card_limit(), flag.p);
    }
    check_launch("card check");
    uint32_t h = 0;
    JAS_HIP(hipMemcpyAsync(&h, flag.p, sizeof(h), hipMemcpyDeviceToHost, s));
    JAS_HIP(hipStreamSynchronize(s));
    if (h)
        fail(JAS_EOVERFLOW, "a summed |X_i| reaches " + std::to_string(card_limit()) +
                                " distinct IDs: int32 intersections would overflow");
}

void gram(const jas_db *db, uint32_t flags, hipStream_t s, int32_t *B, int64_t *card, int64_t *den, double *J) {
    const uint32_t n = (uint32_t)db->n;
    const bool upper = flags & JAS_UPPER;
    const bool accumulate = flags & JAS_ACCUMULATE;
    const uint64_t len = upper ? (uint64_t)n * (n + 1) / 2 : (uint64_t)n * n;
    if (n == 0) return;
    if (!accumulate) {
        JAS_TIMED("fill_i32", s);
        k_fill_i32<<<(uint32_t)std::min<uint64_t>(div_up(len, 256), 65536), 256, 0, s>>>(B, len, 0);
    }
    check_launch("zero B");
    if (db->H > 0 && n >= 2) {
        if (flags & JAS_FORCE_POPCOUNT) {
            const uint32_t nt = (uint32_t)div_up(n, kT);
            const uint64_t np = (uint64_t)nt * (nt + 1) / 2;
            uint64_t kper, splits;
            k_split(db->H, np, 2048, kper, splits);
            const uint64_t ldw = div_up(n, 128) * 128;
            dim3 grid((uint32_t)np, (uint32_t)splits);
            JAS_TIMED("gram_popc", s);
            k_gram_popc<<<grid, kNT, 0, s>>>(db->W.p, ldw, db->H, kper, nt, n, B, upper);
        } else {
            const auto key = std::make_tuple(db->device, n, ceil_log2_u64(db->H));
            int v = kDefaultVariant;
            const uint32_t forced = (flags >> 16) & 0xFFu;  // JAS_GRAM_VARIANT(v): v + 1
            if (forced) {
                v = (int)forced - 1;
            } else if (flags & JAS_TUNE) {
                // time every variant on this db (each adds into B, which is cleared again after)
                JAS_HOST_TIMED("gram_tune");
                hipEvent_t e0, e1;
                JAS_HIP(hipEventCreate(&e0));
                JAS_HIP(hipEventCreate(&e1));
                float best = INFINITY;
                for (int c = 0; c < kNumVariants; ++c) {
                    JAS_HIP(hipEventRecord(e0, s));
                    launch_mfma(db, c, s, B, upper);
                    check_launch("gram (tuning)");
                    JAS_HIP(hipEventRecord(e1, s));
                    JAS_HIP(hipEventSynchronize(e1));
                    float ms = 0.f;
                    JAS_HIP(hipEventElapsedTime(&ms, e0, e1));
                    if (ms < best) {
                        best = ms;
                        v = c;
                    }
                }
                (void)hipEventDestroy(e0);
                (void)hipEventDestroy(e1);
                {
                    std::lock_guard<std::mutex> lk(g_tune_mu);
                    g_tuned[key] = v;
                }
                k_fill_i32<<<(uint32_t)std::min<uint64_t>(div_up(len, 256), 65536), 256, 0, s>>>(B, len, 0);
                check_launch("zero B");
            } else {
                std::lock_guard<std::mutex> lk(g_tune_mu);
                const auto it = g_tuned.find(key);
                if (it != g_tuned.end()) v = it->second;
            }
            JAS_TIMED(kVariants[v].kind == kFp4 ? "gram_fp4" : "gram_mfma", s);
            launch_mfma(db, v, s, B, upper);
        }
        check_launch("gram");
    }
    if (db->n_list > 0 && db->n_lpairs > 0) {
        const uint64_t chunk = std::max<uint64_t>({kPairChunk, div_up(n, 8), div_up(db->n_lpairs, kPairBlocks)});
        const uint64_t blocks = div_up(db->n_lpairs, chunk);
        if (blocks > 0xFFFFFFFFull) fail(JAS_EUNSUPPORTED, "row lists too long");
        const size_t lds = (size_t)n * sizeof(uint32_t);
        {
            JAS_TIMED("pair_count", s);
            k_pair_count<<<(uint32_t)blocks, kPairCountNT, lds, s>>>(db->pairs.p, db->n_lpairs, chunk, n, B, upper, db->dsz);
        }
        check_launch("row-list pairs");
    } else if (db->n_list > 0) {
        const uint64_t blocks = std::min<uint64_t>(div_up(db->n_list, 256), 65536);
        {
            JAS_TIMED("list_pairs", s);
            k_list_pairs<<<(uint32_t)blocks, 256, 0, s>>>(db->list_ptr.p, db->list_smp.p, db->n_list, n, B, upper);
        }
        check_launch("row list pairs");
    }
    if (accumulate) {
        {
            JAS_TIMED("add_card", s);
            k_add_i64<<<(uint32_t)div_up(n, 256), 256, 0, s>>>(card, db->card.p, n);
        }
        check_launch("add card");
        return;
    }
    finalize(n, upper, s, B, db->card.p, den, J);
    if (card) JAS_HIP(hipMemcpyAsync(card, db->card.p, sizeof(int64_t) * n, hipMemcpyDeviceToDevice, s));
}

}  // namespace jas
