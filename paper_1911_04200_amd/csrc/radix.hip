// Stable LSD radix sorts of keys on a bit range.
//
// Used to group equal IDs (the zero-row filter f of Eq. (5) and the
// compaction of Eq. (6) need every nonzero row's entries together).
// radix_sort_u64 (the path for inputs the single-pass scatter below cannot
// take): each pass is reduce-then-scan with no inter-block waiting:
//   1. k_radix_hist:    per-chunk digit histograms (digit-major counts[d][chunk]);
//   2. exclusive scan:  global start of every (digit, chunk) bucket;
//   3. k_radix_scatter: per 4096-key tile, a wave64 ballot multisplit ranks
//      keys by digit (stable: waves own consecutive quarters of the tile,
//      rounds go in order), the tile is reordered in LDS, and each digit run
//      is written out contiguously (coalesced).
#include <algorithm>
#include <type_traits>

#include "device_util.hpp"
#include "jas_internal.hpp"
#include "onesweep_index.hpp"

namespace jas {
namespace {

constexpr int kNT = 256;                     // 4 waves
constexpr int kWaves = kNT / kWave;
constexpr int kRounds = 16;                  // keys per lane per tile
constexpr uint32_t kTile = kNT * kRounds;    // 4096 keys
constexpr uint32_t kTilesPerChunk = 16;
constexpr uint64_t kChunk = (uint64_t)kTile * kTilesPerChunk;  // 65536 keys per block
constexpr int kRadix = 256;

__global__ __launch_bounds__(kNT) void k_radix_hist(const uint64_t *__restrict__ keys, uint64_t N, uint32_t shift,
                                                     uint32_t mask, uint32_t *__restrict__ counts,
                                                     uint32_t nchunks) {
    __shared__ uint32_t h[kWaves][kRadix];
    const uint32_t tid = threadIdx.x, w = tid / kWave;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) h[k][tid] = 0;
    __syncthreads();
    const uint64_t c0 = (uint64_t)blockIdx.x * kChunk;
    const uint64_t c1 = min(N, c0 + kChunk);
    for (uint64_t t0 = c0; t0 < c1; t0 += kTile) {
        uint64_t k[kRounds];
#pragma unroll
        for (int j = 0; j < kRounds; ++j) {
            const uint64_t t = t0 + (uint64_t)j * kNT + tid;
            k[j] = t < c1 ? keys[t] : 0;
        }
#pragma unroll
        for (int j = 0; j < kRounds; ++j) {
            const uint64_t t = t0 + (uint64_t)j * kNT + tid;
            if (t < c1) atomicAdd(&h[w][(uint32_t)(k[j] >> shift) & mask], 1u);
        }
    }
    __syncthreads();
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) c += h[k][tid];
    counts[(uint64_t)tid * nchunks + blockIdx.x] = c;
}

__global__ __launch_bounds__(kNT) void k_radix_scatter(const uint64_t *__restrict__ in, uint64_t *__restrict__ out,
                                                        uint64_t N, uint32_t shift, uint32_t nbits,
                                                        const uint64_t *__restrict__ offs, uint32_t nchunks) {
    __shared__ uint64_t stage[kTile];
    __shared__ uint32_t wcnt[kWaves][kRadix];
    __shared__ uint32_t tdp[kRadix];
    __shared__ uint64_t base[kRadix];
    __shared__ uint64_t sh[kWaves];
    const uint32_t tid = threadIdx.x, lane = lane_id(), w = tid / kWave;
    const uint32_t mask = (1u << nbits) - 1u;
    const uint64_t c0 = (uint64_t)blockIdx.x * kChunk;
    const uint64_t c1 = min(N, c0 + kChunk);
    const uint64_t lt = lanemask_lt();
    base[tid] = offs[(uint64_t)tid * nchunks + blockIdx.x];

    for (uint64_t t0 = c0; t0 < c1; t0 += kTile) {
#pragma unroll
        for (int k = 0; k < kWaves; ++k) wcnt[k][tid] = 0;
        __syncthreads();
        // wave w owns positions [t0 + w*1024, t0 + (w+1)*1024), 64 per round
        const uint64_t wb = t0 + (uint64_t)w * (kTile / kWaves);
        uint64_t key[kRounds];
        uint32_t rank[kRounds];
#pragma unroll
        for (int j = 0; j < kRounds; ++j) {
            const uint64_t t = wb + (uint64_t)j * kWave + lane;
            key[j] = t < c1 ? in[t] : 0;
        }
#pragma unroll
        for (int j = 0; j < kRounds; ++j) {
            const uint64_t t = wb + (uint64_t)j * kWave + lane;
            const bool valid = t < c1;
            const uint32_t d = (uint32_t)(key[j] >> shift) & mask;
            uint64_t peers = __ballot(valid);
            for (uint32_t b = 0; b < nbits; ++b) {
                const bool bit = (d >> b) & 1u;
                const uint64_t vote = __ballot(valid && bit);
                peers &= bit ? vote : ~vote;
            }
            const uint32_t before = __popcll(peers & lt);
            const uint32_t cnt = __popcll(peers);
            uint32_t b0 = 0;
            if (valid) b0 = wcnt[w][d];
            if (valid && before == 0) wcnt[w][d] = b0 + cnt;
            rank[j] = b0 + before;
        }
        __syncthreads();
        // per digit: tile count, exclusive prefix over digits, prefix over waves
        uint32_t c[kWaves];
        uint32_t tc = 0;
#pragma unroll
        for (int k = 0; k < kWaves; ++k) {
            c[k] = wcnt[k][tid];
            tc += c[k];
        }
        uint64_t tot;
        const uint32_t ex = (uint32_t)block_excl_scan<kNT>(tc, sh, &tot);
        tdp[tid] = ex;
        uint32_t run = 0;
#pragma unroll
        for (int k = 0; k < kWaves; ++k) {
            wcnt[k][tid] = run;
            run += c[k];
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kRounds; ++j) {
            const uint64_t t = wb + (uint64_t)j * kWave + lane;
            if (t < c1) {
                const uint32_t d = (uint32_t)(key[j] >> shift) & mask;
                stage[tdp[d] + wcnt[w][d] + rank[j]] = key[j];
            }
        }
        __syncthreads();
        const uint32_t cnt_tile = (uint32_t)min((uint64_t)kTile, c1 - t0);
        for (uint32_t i = tid; i < cnt_tile; i += kNT) {
            const uint64_t k = stage[i];
            const uint32_t d = (uint32_t)(k >> shift) & mask;
            out[base[d] + (i - tdp[d])] = k;
        }
        __syncthreads();
        base[tid] += tc;
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Single-pass scatter with decoupled look-back (chained scan: Merrill &
// Garland, "Single-pass parallel prefix scan with decoupled look-back",
// 2016; as in Adinets & Merrill's Onesweep, 2022).  Persistent blocks take
// tiles by ticket from an atomic counter in launch order, so every
// tile a block waits for already belongs to a running block.  Per tile and
// digit a 32-bit status word holds a flag (aggregate / inclusive prefix) and
// a 30-bit count; the caller guarantees every digit total is < 2^30.  The
// same kernel sorts 64-bit keys (the encoder and the query path) and 32-bit
// row-list pair words.
// A load the compiler may issue through the scalar cache: the data stays
// unchanged while the kernel runs (written by an earlier launch) and the
// address is the same across the wave.
template <class T>
__device__ __forceinline__ T const_load(const T *p) {
    return *(const __attribute__((address_space(4))) T *)(p);
}

using onesweep::kFlagA;
using onesweep::kFlagP;
using onesweep::kValMask;
using onesweep::kLookWindow;  // three passes over 1.78 G keys: 18.9 ms with 3; 20.2 with 4, 19.5 with 2, 20.6 with 8
constexpr uint32_t kMaxSpin = 1u << 20;  // bounded wait (~0.1 s of polls), then give up and flag

__device__ __forceinline__ void status_store(uint32_t *p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t status_load(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One tile = kOsNT threads x R keys; a thread also owns a digit.
constexpr int kOsNT = 512;
constexpr int kOsWaves = kOsNT / kWave;
constexpr uint32_t kOsStageBytes = 65536;  // LDS the tile is reordered in (two blocks per CU fit)
typedef uint16_t __attribute__((may_alias)) u16_alias;

template <class K, class Rsrc>
__device__ __forceinline__ K buffer_key(Rsrc r, uint32_t off) {
    if constexpr (sizeof(K) == 8) {
        typedef uint32_t v2u __attribute__((ext_vector_type(2)));
        const v2u v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
        return (uint64_t)v[1] << 32 | v[0];
    } else {
        return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
    }
}

// With kFromIds the pass reads CSR IDs and forms each key id << src.sbits |
// sample itself.  Its digit is ID bits only (shift >= src.sbits), so the IDs
// are ranked as loaded (each rank starts as soon as its load arrives) and the
// sample joins a key before it is placed in LDS: src.tinfo holds the samples of
// the tile's first and last entries (k_tile_samples), and an entry's sample is
// the first one plus the sample starts inside the tile at or before it (scalar
// loads, each start passed once by the wave whose entries it lies in: with every
// thread passing all of a tile's 78 starts, 638 K
// IDs in sets of 78 took 0.165 ms instead of 0.02).
//
// A pass moves 16 bytes per 64-bit key; each tile's chain of latencies (loads,
// ranks, look-back, stores) bounds it more than memory does, so a tile is as
// large as the registers hold (R = 32 keys per thread) and is reordered in LDS
// a half at a time (64-bit keys), except where that leaves too few tiles.
// Ranks come from unrolled ballots for a fixed number of digit bits, with the
// counter operations in flight together.  Spilled registers cost more than
// their bytes: a reload waits for the status stores before it.
//
// 1.78 G keys, three passes (8, 8 and 6 bits): 25.3 ms with a ballot loop whose
// rounds waited for each other's counters and 16 keys per thread, 23.3 with
// unrolled ballots, 20.7 with 32 (24) keys per thread: 4.1 TB/s of the 6.2 a
// copy through such tiles reaches.  1.85 G pair words, two passes: 12.2, 11.0,
// 8.8 (8.3 with 64).  A tile's time (paperlike, 16384 keys): loads and ranks 37 %, look-back
// 23 %, writes 16 %, counts and scan 12 %, placing 8 %.
template <class K, int R, int NB, bool kFromIds = false>
__global__ __launch_bounds__(kOsNT) __attribute__((amdgpu_waves_per_eu(4))) void k_radix_onesweep(
    const K *__restrict__ in, K *__restrict__ out, uint64_t N, uint32_t shift, uint32_t nbits,
    const uint64_t *__restrict__ gstart, uint32_t *__restrict__ status, uint32_t *__restrict__ next_status,
    uint32_t *__restrict__ ticket, uint32_t ntiles, uint32_t *__restrict__ err, const uint64_t *__restrict__ dN,
    KeySource src) {
    constexpr uint32_t kDigits = NB > 8 ? onesweep::kWideRadix : onesweep::kRadix;
    constexpr uint32_t kTileKeys = kOsNT * R;
    constexpr uint32_t kParts = (kTileKeys * sizeof(K) + kOsStageBytes - 1) / kOsStageBytes;
    constexpr uint32_t kStage = kTileKeys / kParts;  // the tile is reordered in LDS in kParts parts
    static_assert(kTileKeys % kStage == 0 && kDigits <= kOsNT && R % 8 == 0 && kTileKeys <= 65536, "tile");
    static_assert(!kFromIds || sizeof(K) == 8, "keys formed from IDs are 64-bit");
    __shared__ K stage[kStage];
    // per wave and digit d: a 16-bit count (then the first position of the wave's
    // keys of digit d in the tile) in half d & 1 of word d >> 1
    __shared__ uint32_t wcnt[kOsWaves][kDigits / 2];
    __shared__ uint64_t offs[kDigits];  // output position of a key minus its position in the tile
    __shared__ uint32_t sh[kOsWaves];
    __shared__ uint32_t tile_sh;
    if (dN) {  // key count from device memory (planned encode): at most the buffers' N
        N = min(N, *dN);
        ntiles = (uint32_t)onesweep::num_tiles(N, kTileKeys);
    }
    const uint32_t mask = (1u << nbits) - 1u;
    const uint32_t dshift = kFromIds ? shift - src.sbits : shift;  // digit position in a loaded value
    const uint64_t gs = threadIdx.x < kDigits ? gstart[threadIdx.x] : 0;
    // persistent: take tiles in ticket order until none is left
    for (;;) {
        // opaque, so that nothing derived from it is held in registers from tile to tile
        uint32_t tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const uint32_t lane = tid % kWave, w = __builtin_amdgcn_readfirstlane(tid / kWave);
        const u16_alias *wpos = reinterpret_cast<const u16_alias *>(wcnt[w]);
        const bool digit = tid < kDigits;  // this thread owns digit tid
        if (tid == 0) tile_sh = atomicAdd(ticket, 1u);
        for (uint32_t i = tid; i < kOsWaves * kDigits / 2; i += kOsNT) (&wcnt[0][0])[i] = 0;
        __syncthreads();
        const uint32_t tile = __builtin_amdgcn_readfirstlane(tile_sh);  // uniform: every thread reads the same ticket
        if (tile >= ntiles) break;  // uniform: every thread read the same ticket
        const uint64_t t0 = onesweep::tile_first(tile, kTileKeys);
        const uint64_t c1 = onesweep::tile_end(tile, kTileKeys, N);
        const uint32_t cnt_tile = (uint32_t)(c1 - t0);
        K key[R];
        uint32_t pos[R / 2];  // 16 bits per key: rank within the wave and digit, then position in the tile
        // The tile's keys, read through a buffer descriptor that ends with them
        // (entries past the end read as 0).  Rank within the wave: the lanes of
        // a round with the same digit take consecutive slots after the digit's
        // count so far, and the lowest of them adds the group to the count.  One
        // wave's LDS operations run in order, so the rounds' reads and additions
        // are issued back to back without waiting for one another, each as its
        // keys arrive.  Entries past the end are given the largest digit; they
        // come last in it, so they land past the tile's keys and only that
        // digit's count has to be corrected.
        const auto tile_in = __builtin_amdgcn_make_buffer_rsrc(const_cast<K *>(in + t0), 0,
                                                               cnt_tile * (uint32_t)sizeof(K), 0x00020000);
        const uint32_t wl = w * (kTileKeys / kOsWaves) + lane;  // this lane's first entry in the tile
#pragma unroll
        for (int j = 0; j < R; ++j) key[j] = buffer_key<K>(tile_in, (wl + j * kWave) * (uint32_t)sizeof(K));
#pragma unroll
        for (int g = 0; g < R; g += 8) {
            uint32_t rank[8], before[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint32_t past = wl + (g + j) * kWave < cnt_tile ? 0u : ~0u;
                key[g + j] |= sizeof(K) == 8 ? (K)((uint64_t)past << 32 | past) : (K)past;
                const uint32_t d = (uint32_t)(key[g + j] >> dshift) & mask;
                const uint64_t peers = wave_match<NB>(d);
                before[j] = lanes_before(peers);
                rank[j] = __hip_atomic_load(&wcnt[w][d >> 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >>
                          (16 * (d & 1));
                if (before[j] == 0)
                    __hip_atomic_fetch_add(&wcnt[w][d >> 1], (uint32_t)__popcll(peers) << (16 * (d & 1)),
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                // a round's temporaries end with it (interleaved rounds would not fit the registers)
                if (R > 16) __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int j = 0; j < 8; j += 2) {
                pos[(g + j) / 2] = ((rank[j] & 0xFFFFu) + before[j]) | ((rank[j + 1] + before[j + 1]) << 16);
                asm volatile("" : "+v"(pos[(g + j) / 2]));  // packed here, not where it is used
            }
        }
        __syncthreads();
        uint32_t tc = 0;
        if (digit) {
#pragma unroll
            for (int k = 0; k < kOsWaves; ++k) tc += reinterpret_cast<const u16_alias *>(wcnt[k])[tid];
            if (tid == mask) tc -= kTileKeys - cnt_tile;  // the entries past the last tile's end
            // publish the tile's count of digit tid at once, and clear its word for the next pass
            status_store(status + onesweep::status_index(tile, tid, kDigits), (tile == 0 ? kFlagP : kFlagA) | tc);
            if (next_status) next_status[onesweep::status_index(tile, tid, kDigits)] = 0;
        }
        const uint32_t ex = block_excl_scan_u32<kOsNT>(tc, sh);  // digit tid's first position in the tile
        if (digit) {  // the counts become where wave k's keys of digit tid start in the tile
            uint32_t run = ex;
#pragma unroll
            for (int k = 0; k < kOsWaves; ++k) {
                u16_alias *p = reinterpret_cast<u16_alias *>(wcnt[k]) + tid;
                const uint32_t v = *p;
                *p = (uint16_t)run;
                run += v;
            }
        }
        __syncthreads();
        if constexpr (R > 16) {
            // the digits are taken from the keys again: kept from the ranking, they would not fit the registers
#pragma unroll
            for (int j = 0; j < R; ++j) asm volatile("" : "+v"(key[j]));
        }
#pragma unroll
        for (int j = 0; j < R; j += 2) {
            pos[j / 2] += (uint32_t)wpos[(uint32_t)(key[j] >> dshift) & mask] |
                          (uint32_t)wpos[(uint32_t)(key[j + 1] >> dshift) & mask] << 16;
            if (R > 16) asm volatile("" : "+v"(pos[j / 2]));
        }
        if constexpr (kFromIds) {
            // the sample starts inside the tile lie in (t0, c1), so tile-relative
            // positions compare in 32 bits; a wave's entries are consecutive, 64
            // each round, so it looks for its first sample once and then passes
            // each start in its part of the tile once
            const uint64_t tsmp = const_load(reinterpret_cast<const uint64_t *>(src.tinfo) + tile);
            const uint32_t s0 = (uint32_t)tsmp, s1 = (uint32_t)(tsmp >> 32);  // samples of the first and last entries
            const auto start = [&](uint32_t k) { return (uint32_t)(const_load(src.off + k) - t0); };
            uint32_t at = (uint32_t)__builtin_amdgcn_readfirstlane((int)(wl - lane));  // the wave's first entry
            uint32_t cur = s0;  // the last sample that starts at or before it
            for (uint32_t hi = s1; cur < hi;) {
                const uint32_t mid = cur + (hi - cur + 1) / 2;
                if (start(mid) <= at) cur = mid;
                else hi = mid - 1;
            }
            uint32_t next = cur < s1 ? start(cur + 1) : ~0u;
#pragma unroll
            for (int j = 0; j < R; ++j, at += kWave) {
                uint32_t smp = cur;
                while (next < at + kWave) {
                    smp += wl + j * kWave >= next;
                    ++cur;
                    next = cur < s1 ? start(cur + 1) : ~0u;
                }
                key[j] = (key[j] << src.sbits) | smp;
            }
        }
        // reorder the tile (its first part) in LDS by digit
        const auto place = [&](uint32_t part) {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                if (kParts > 1 && j % 2 == 0) asm volatile("" : "+v"(pos[j / 2]));
                const uint32_t p = (pos[j / 2] >> (16 * (j & 1))) & 0xFFFFu;
                if (kParts == 1) stage[p] = key[j];
                else if (p - part * kStage < kStage) stage[p - part * kStage] = key[j];
            }
        };
        place(0);
        // then look back for the digit's global offset: kLookWindow
        // predecessor tiles per step, loaded together (one memory round trip)
        // and taken nearest first
        if (digit) {
            uint32_t excl = 0;
            if (tile > 0) {
                bool found = false;
                for (int64_t j0 = (int64_t)tile - 1; j0 >= 0 && !found; j0 -= kLookWindow) {
                    uint32_t v[kLookWindow];
#pragma unroll
                    for (int k = 0; k < kLookWindow; ++k)
                        v[k] = j0 - k >= 0 ? status_load(status + onesweep::status_index(j0 - k, tid, kDigits)) : kFlagP;
#pragma unroll
                    for (int k = 0; k < kLookWindow; ++k) {
                        if (found) break;
                        uint32_t spins = 0;
                        while ((v[k] & ~kValMask) == 0) {
                            // give up after kMaxSpin polls, or at once when any tile has given up
                            if (++spins > kMaxSpin || (status_load(err) & 2u)) {
                                atomicOr(err, 2u);
                                v[k] = kFlagP;
                                break;
                            }
                            __builtin_amdgcn_s_sleep(1);
                            v[k] = status_load(status + onesweep::status_index(j0 - k, tid, kDigits));
                        }
                        excl += v[k] & kValMask;
                        found = (v[k] & ~kValMask) == kFlagP;
                    }
                }
                status_store(status + onesweep::status_index(tile, tid, kDigits), kFlagP | ((excl + tc) & kValMask));
            }
            offs[tid] = onesweep::out_offset(gs + excl, ex);
        }
        __syncthreads();
        for (uint32_t part = 0; part < kParts; ++part) {
            const uint32_t p0 = part * kStage;
            if (part > 0) {
                if (p0 >= cnt_tile) break;  // uniform
                place(part);
                __syncthreads();
            }
            const uint32_t len = min(kStage, cnt_tile - p0);
            // a few keys per thread at a time, their LDS reads in flight together
            constexpr uint32_t kAhead = kParts > 1 ? 4 : 8;
            for (uint32_t i = tid; i < len; i += kAhead * kOsNT) {
                K k[kAhead];
                uint64_t o[kAhead];
#pragma unroll
                for (uint32_t u = 0; u < kAhead; ++u) k[u] = stage[(i + u * kOsNT) % kStage];
#pragma unroll
                for (uint32_t u = 0; u < kAhead; ++u)
                    o[u] = offs[(uint32_t)(k[u] >> shift) & mask] + (p0 + i + u * kOsNT);
#pragma unroll
                for (uint32_t u = 0; u < kAhead; ++u)
                    if (i + u * kOsNT < len) out[o[u]] = k[u];
            }
            __syncthreads();  // stage, offs and tile_sh are rewritten
        }
    }
}

// Block q: gstart[q][d] = exclusive scan over pass q's digits of the summed
// replicas; maxima[q] = largest digit total.  ghist and gstart have rows of
// `radix` digits per pass (256, or 512 for 9-bit passes).
__global__ __launch_bounds__(kOsNT) void k_digit_starts(const unsigned long long *__restrict__ ghist, uint32_t radix,
                                                         uint64_t *__restrict__ gstart, uint64_t *__restrict__ maxima,
                                                         uint32_t *__restrict__ err) {
    __shared__ uint64_t sh[kOsWaves];
    const uint32_t tid = threadIdx.x, q = blockIdx.x;
    uint64_t t = 0;
    if (tid < radix) {
#pragma unroll
        for (uint32_t r = 0; r < kGhistReplicas; ++r)
            t += ghist[(uint64_t)r * kMaxPasses * kRadix + q * radix + tid];
    }
    uint64_t all;
    const uint64_t ex = block_excl_scan<kOsNT>(t, sh, &all);
    if (tid < radix) gstart[q * radix + tid] = ex;
    uint64_t m = t;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) m = max(m, (uint64_t)__shfl_xor((unsigned long long)m, d, kWave));
    if (lane_id() == 0) sh[tid / kWave] = m;
    __syncthreads();
    if (tid == 0) {
        for (int k = 1; k < kOsWaves; ++k) m = max(m, sh[k]);
        maxima[q] = m;
        if (err && m >= kValMask) atomicOr(err, 4u);  // planned sort: cannot run single-pass
    }
}

__global__ void k_fill32(uint32_t *p, uint64_t len) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < len; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

// Per tile of tile_keys entries: tinfo[2 t] and tinfo[2 t + 1] = the samples
// holding the tile's first and last entries.
__global__ void k_tile_samples(const uint64_t *__restrict__ off, int32_t n, uint64_t N, uint32_t tile_keys,
                               uint32_t *__restrict__ tinfo, const uint64_t *__restrict__ dN) {
    if (dN) N = min(N, *dN);
    const uint64_t ntiles = onesweep::num_tiles(N, tile_keys);
    for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < ntiles;
         t += (uint64_t)gridDim.x * blockDim.x) {
        const int32_t s0 = find_sample(off, 0, n - 1, onesweep::tile_first(t, tile_keys));
        tinfo[2 * t] = (uint32_t)s0;
        tinfo[2 * t + 1] = (uint32_t)find_sample(off, s0, n - 1, onesweep::tile_end(t, tile_keys, N) - 1);
    }
}

}  // namespace

SortPlan sort_plan(uint64_t N, uint32_t U, uint32_t sbits, uint32_t max_width) {
    SortPlan p;
    if (N <= kLocalCapKeys) return p;  // one LDS range holds everything
    p.top_bits = std::min<uint32_t>(U, ceil_log2_u64(div_up(N, kBucketKeys)));
    const uint32_t fewer = std::min<uint32_t>(U, ceil_log2_u64(div_up(N, 2 * kBucketKeys)));
    if (fewer > 0 && (U - fewer) + kSpanBits + sbits <= 32) p.top_bits = fewer;
    // the fewest passes of at most 9 (max_width) bits, of equal width: a pass over 18 bits'
    // halves takes 1.4 times one over 6 (1.78 G keys: 9.0, 6.3 ms), so two beat three
    p.npass = (p.top_bits + max_width - 1) / max_width;
    p.width = p.npass ? (p.top_bits + p.npass - 1) / p.npass : 8;
    return p;
}

uint64_t radix_work_bytes(uint64_t N) {
    const uint64_t nchunks = div_up(N, kChunk);
    const uint64_t len = (uint64_t)kRadix * nchunks;
    return len * 4 + (len + 1) * 8 + scan_tmp_elems(len) * 8;
}

uint64_t radix_prepare(RadixWork &w, uint64_t N, hipStream_t s, Budget *b, Arena *ar) {
    const uint64_t nchunks = div_up(std::max<uint64_t>(N, 1), kChunk);
    if (nchunks > 0xFFFFFFFFull) fail(JAS_EUNSUPPORTED, "radix sort: too many keys");
    const uint64_t len = (uint64_t)kRadix * nchunks;
    if (w.counts.n < len) temp_buf(w.counts, len, s, b, ar, "radix counts");
    if (w.offs.n < len + 1) temp_buf(w.offs, len + 1, s, b, ar, "radix offsets");
    const size_t tl = scan_tmp_elems(len);
    if (w.tmp.n < tl) temp_buf(w.tmp, tl, s, b, ar, "radix scan scratch");
    return nchunks;
}

void radix_sort_u64(DevBuf<uint64_t> &keys, DevBuf<uint64_t> &alt, uint64_t N, uint32_t lo_bit, uint32_t hi_bit,
                    RadixWork &w, hipStream_t s, Budget *b, Arena *ar) {
    if (N <= 1 || hi_bit <= lo_bit) return;
    const uint64_t nchunks = radix_prepare(w, N, s, b, ar);
    const uint64_t len = (uint64_t)kRadix * nchunks;
    for (uint32_t bit = lo_bit; bit < hi_bit; bit += 8) {
        const uint32_t nbits = min(8u, hi_bit - bit);
        const uint32_t mask = (1u << nbits) - 1u;
        {
            JAS_TIMED("radix_hist", s);
            k_radix_hist<<<(uint32_t)nchunks, kNT, 0, s>>>(keys.p, N, bit, mask, w.counts.p, (uint32_t)nchunks);
        }
        check_launch("radix histogram");
        scan_excl_u32(w.counts.p, w.offs.p, len, w.tmp.p, s);
        {
            JAS_TIMED("radix_scatter", s);
            k_radix_scatter<<<(uint32_t)nchunks, kNT, 0, s>>>(keys.p, alt.p, N, bit, nbits, w.offs.p,
                                                             (uint32_t)nchunks);
        }
        check_launch("radix scatter");
        swap_bufs(keys, alt);
    }
}

}  // namespace jas

namespace jas {

namespace {
// Fills src.tinfo for tiles of tile_keys entries (after checking its size).
void tile_samples(const KeySource &src, uint64_t Ncap, uint32_t tile_keys, const uint64_t *dN, hipStream_t s) {
    const uint64_t ntiles = onesweep::num_tiles(Ncap, tile_keys);
    if (!src.ids || !src.off || !src.tinfo || src.n < 1 || src.tinfo_words < 2 * ntiles)
        fail(JAS_EDEVICE, "sort from IDs: tile sample buffer does not cover the tiles");
    {
        JAS_TIMED("tile_samples", s);
        k_tile_samples<<<(uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(div_up(ntiles, 256), 4096)), 256, 0, s>>>(
            src.off, src.n, Ncap, tile_keys, src.tinfo, dN);
    }
    check_launch("tile samples");
}

// Keys per thread of a tile: 32, or 24 in the pass that forms the keys (it
// holds more, and 32 would spill), except where that leaves fewer than two
// tiles for each resident block (then 16: more, shorter tiles); 64 for 32-bit
// keys where that leaves two.  Two passes over 1.68 G pair words: 7.9 ms with 32,
// 8.0 with 40, 7.7 with 48, 7.6 with 56, 7.5 with 64 (5 registers spilled).
int tile_rounds(uint64_t N, bool from_ids, size_t key_bytes = 8) {
    const uint64_t two_tiles = (uint64_t)4 * 256 * kOsNT;
    if (N < two_tiles * 32) return 16;
    return from_ids ? 24 : key_bytes == 4 && N >= two_tiles * 64 ? 64 : 32;
}
// Most tiles of any pass of a sort of N keys.
uint64_t most_tiles(uint64_t N) { return onesweep::num_tiles(N, (uint32_t)kOsNT * tile_rounds(N, true)); }

// The look-back words of a sort: a ticket per pass, then the status words of
// two passes (a pass clears the other's while it runs, so only the first
// pass's and the tickets are cleared beforehand), or of one (cleared again
// before each pass: a launch more, 5 us, but half the bytes, so a caller's
// memory budget decides for it).
constexpr uint64_t kTicketWords = 64;
static_assert(kTicketWords >= kMaxPasses, "tickets");
uint64_t look_back_words(uint64_t ntiles, uint32_t radix, bool two = true) {
    return kTicketWords + (two ? 2 : 1) * onesweep::status_words(ntiles, radix);
}

// What every pass of one sort is launched with.
struct PassArgs {
    uint64_t N = 0;
    uint32_t *look_back = nullptr, *err = nullptr, radix = 256;
    const uint64_t *dN = nullptr, *gstart = nullptr;
    const KeySource *src = nullptr;  // null: the keys are in memory
    const void *first = nullptr;     // where the first pass reads them, if not in the sort's buffer
    bool two = true;                 // look_back holds the status words of two passes
    hipStream_t s = nullptr;
};

// Launches pass q on nbits bits from `bit` on; the first reads src.ids when
// the keys are formed from IDs.  Passes of at most 7 bits take a kernel that
// matches 7.
template <class K, int Rounds, int NB>
void onesweep_launch(const PassArgs &a, uint32_t q, const K *in, K *out, uint32_t bit, uint32_t nbits) {
    const uint32_t ntiles = (uint32_t)onesweep::num_tiles(a.N, (uint32_t)kOsNT * Rounds);
    // persistent blocks: two per CU (256 CUs) fit, never more than there are tiles
    const uint32_t grid = std::min<uint32_t>(ntiles, 256 * 2);
    uint32_t *st0 = a.look_back + kTicketWords, *st1 = st0 + onesweep::status_words(most_tiles(a.N), a.radix);
    uint32_t *st = a.two && (q & 1) ? st1 : st0, *next = a.two ? (q & 1 ? st0 : st1) : nullptr;
    uint32_t *ticket = a.look_back + q;
    const uint64_t *gs = a.gstart + (uint64_t)q * a.radix;
    if constexpr (sizeof(K) == 8 && Rounds != 32) {
        if (a.src && q == 0) {
            k_radix_onesweep<K, Rounds, NB, true><<<grid, kOsNT, 0, a.s>>>(
                reinterpret_cast<const K *>(a.src->ids), out, a.N, bit, nbits, gs, st, next, ticket, ntiles, a.err,
                a.dN, *a.src);
            return;
        }
    }
    if constexpr (Rounds != 24)
        k_radix_onesweep<K, Rounds, NB><<<grid, kOsNT, 0, a.s>>>(in, out, a.N, bit, nbits, gs, st, next, ticket, ntiles,
                                                                a.err, a.dN, KeySource{});
}
template <class K, int Rounds>
void onesweep_digits(const PassArgs &a, uint32_t q, const K *in, K *out, uint32_t bit, uint32_t nbits) {
    if constexpr (sizeof(K) == 8) {  // (pair words are sorted on at most 8 bits at a time)
        if (nbits > 8) return onesweep_launch<K, Rounds, 9>(a, q, in, out, bit, nbits);
    }
    if (nbits == 8) onesweep_launch<K, Rounds, 8>(a, q, in, out, bit, nbits);
    else onesweep_launch<K, Rounds, 7>(a, q, in, out, bit, nbits);
}
// Every pass; keys and alt are swapped as they go.
template <class K, class Swap>
void onesweep_passes(const PassArgs &a, uint32_t lo_bit, uint32_t hi_bit, uint32_t width, const char *name, K *keys,
                     K *alt, Swap swap) {
    if (a.src && (sizeof(K) != 8 || lo_bit < a.src->sbits)) fail(JAS_EDEVICE, "sort from IDs: bad digits or keys");
    const auto clear = [&](uint32_t *p, uint64_t len) {
        JAS_TIMED("fill_status", a.s);
        k_fill32<<<(uint32_t)std::min<uint64_t>(div_up(len, 256), 65536), 256, 0, a.s>>>(p, len);
        check_launch("look-back reset");
    };
    const uint64_t status = onesweep::status_words(most_tiles(a.N), a.radix);
    clear(a.look_back, kTicketWords + status);
    for (uint32_t q = 0; lo_bit + width * q < hi_bit; ++q) {
        const uint32_t bit = lo_bit + width * q, nbits = std::min(width, hi_bit - bit);
        if (!a.two && q > 0) clear(a.look_back + kTicketWords, status);
        {
            JAS_TIMED(name, a.s);
            const int rounds = tile_rounds(a.N, a.src && q == 0, sizeof(K));
            const K *in = a.first && q == 0 ? static_cast<const K *>(a.first) : keys;
            if (rounds == 64) onesweep_digits<K, sizeof(K) == 4 ? 64 : 32>(a, q, in, alt, bit, nbits);
            else if (rounds == 32) onesweep_digits<K, 32>(a, q, in, alt, bit, nbits);
            else if (rounds == 24) onesweep_digits<K, sizeof(K) == 8 ? 24 : 32>(a, q, in, alt, bit, nbits);
            else onesweep_digits<K, 16>(a, q, in, alt, bit, nbits);
        }
        check_launch("radix scatter (look-back)");
        std::swap(keys, alt);
        swap();
    }
}

// With src the keys are formed from CSR sets by the first pass (keys.p is
// not read); otherwise keys holds them.
template <class K>
bool onesweep_sort(DevBuf<K> &keys, DevBuf<K> &alt, uint64_t N, uint32_t lo_bit, uint32_t hi_bit, uint32_t width,
                   const unsigned long long *ghist, uint32_t *err, hipStream_t s, Budget *b, Arena *ar,
                   const char *name, const KeySource *src = nullptr, const K *first = nullptr) {
    if (N <= 1 || hi_bit <= lo_bit) return true;
    if (width < 1 || width > (sizeof(K) == 8 ? 9 : 8)) return false;
    const uint32_t npass = (hi_bit - lo_bit + width - 1) / width, radix = onesweep::radix_of(width);
    if (npass * radix > kMaxPasses * kRadix) return false;
    DevBuf<uint64_t> gstart, maxima;
    temp_buf(gstart, (uint64_t)kMaxPasses * kRadix, s, b, ar, "digit starts");
    temp_buf(maxima, kMaxPasses, s, b, ar, "digit maxima");
    digit_starts(ghist, npass, width, gstart.p, maxima.p, s);
    // no digit total is as large as the look-back counts' limit unless N is: only then they are read back
    const uint64_t limit = std::min<uint64_t>(kValMask, scatter_count_limit());
    if (N >= limit) {
        uint64_t hm[kMaxPasses];
        JAS_HIP(hipMemcpyAsync(hm, maxima.p, sizeof(uint64_t) * npass, hipMemcpyDeviceToHost, s));
        JAS_HIP(hipStreamSynchronize(s));
        for (uint32_t q = 0; q < npass; ++q)
            if (hm[q] >= limit) return false;
    }
    // What the kernel's indexing relies on (see onesweep_index.hpp): the key
    // buffers hold N keys, tiles are numbered in 32 bits and cover exactly
    // [0, N), the status array has a word for every (tile, digit) of two passes
    // (or of the one it is cleared for),
    // every pass has a row of digit starts, and no 30-bit status count can wrap
    // (checked above).
    const uint64_t ntiles = most_tiles(N);
    if (ntiles > 0xFFFFFFFFull) return false;
    DevBuf<uint32_t> look_back;
    PassArgs a;
    a.two = npass > 1 && !(b && b->limit);
    temp_buf(look_back, look_back_words(ntiles, radix, a.two), s, b, ar, "look-back status");
    if (keys.n < N || alt.n < N || look_back.n < look_back_words(ntiles, radix, a.two) ||
        gstart.n < (uint64_t)npass * radix)
        fail(JAS_EDEVICE, "single-pass scatter: buffer sizes do not cover its indexing");
    a.N = N;
    a.look_back = look_back.p;
    a.err = err;
    a.radix = radix;
    a.gstart = gstart.p;
    a.first = first;
    a.s = s;
    KeySource ks;
    DevBuf<uint32_t> tinfo;
    if (src) {
        ks = *src;
        temp_buf(tinfo, 2 * ntiles, s, b, ar, "tile samples");
        ks.tinfo = tinfo.p;
        ks.tinfo_words = tinfo.n;
        tile_samples(ks, N, (uint32_t)kOsNT * tile_rounds(N, true), nullptr, s);
        a.src = &ks;
    }
    onesweep_passes<K>(a, lo_bit, hi_bit, width, name, keys.p, alt.p, [&] { swap_bufs(keys, alt); });
    return true;
}
// The same passes for a planned encode: the key count is read from *dN
// (at most Ncap, the buffers' size) inside the kernels, every buffer is
// given, nothing is read back and nothing allocated.  A digit total too large
// for the 30-bit status counts sets bit 2 of err[0] (the result is then
// invalid; the caller reports it after the stream completes).
template <class K>
void onesweep_sort_planned(K *&keys, K *&alt, const uint64_t *dN, uint64_t Ncap, uint32_t lo_bit, uint32_t hi_bit,
                           uint32_t width, const unsigned long long *ghist, uint32_t *err, const OnesweepBufs &b,
                           hipStream_t s, const char *name, const KeySource *src = nullptr) {
    if (Ncap <= 1 || hi_bit <= lo_bit) return;
    const uint32_t npass = (hi_bit - lo_bit + width - 1) / width, radix = onesweep::radix_of(width);
    if (npass * radix > kMaxPasses * kRadix || width < 1 || width > (sizeof(K) == 8 ? 9 : 8))
        fail(JAS_EUNSUPPORTED, "planned sort: bad digit plan");
    const uint64_t ntiles = most_tiles(Ncap);
    if (b.status_words < look_back_words(ntiles, radix, false) || ntiles > 0xFFFFFFFFull)
        fail(JAS_EDEVICE, "planned sort: status buffer too small");
    {
        JAS_TIMED("digit_starts", s);
        k_digit_starts<<<npass, kOsNT, 0, s>>>(ghist, radix, b.gstart, b.maxima, err);
    }
    check_launch("digit starts");
    if (src) tile_samples(*src, Ncap, (uint32_t)kOsNT * tile_rounds(Ncap, true), dN, s);
    PassArgs a;
    a.N = Ncap;
    a.two = npass > 1 && b.status_words >= look_back_words(ntiles, radix);
    a.look_back = b.status;
    a.err = err;
    a.radix = radix;
    a.dN = dN;
    a.gstart = b.gstart;
    a.src = src;
    a.s = s;
    onesweep_passes<K>(a, lo_bit, hi_bit, width, name, keys, alt, [&] { std::swap(keys, alt); });
}

}  // namespace

void digit_starts(const unsigned long long *ghist, uint32_t npass, uint32_t width, uint64_t *starts, uint64_t *maxima,
                  hipStream_t s) {
    if (npass == 0) return;
    {
        JAS_TIMED("digit_starts", s);
        k_digit_starts<<<npass, kOsNT, 0, s>>>(ghist, onesweep::radix_of(width), starts, maxima, nullptr);
    }
    check_launch("digit starts");
}

uint64_t onesweep_tile_keys_from_ids(uint64_t N) { return (uint64_t)kOsNT * tile_rounds(N, true); }

uint64_t onesweep_look_back_words(uint64_t N, uint32_t width, bool two) {
    return look_back_words(most_tiles(N), onesweep::radix_of(width), two);
}

void radix_sort_onesweep_planned(uint64_t *&keys, uint64_t *&alt, const uint64_t *dN, uint64_t Ncap,
                                 uint32_t lo_bit, uint32_t hi_bit, uint32_t width, const unsigned long long *ghist,
                                 uint32_t *err, const OnesweepBufs &b, hipStream_t s, const KeySource *src) {
    onesweep_sort_planned<uint64_t>(keys, alt, dN, Ncap, lo_bit, hi_bit, width, ghist, err, b, s, "radix_onesweep",
                                    src);
}

void radix_sort_onesweep_u32_planned(uint32_t *&keys, uint32_t *&alt, const uint64_t *dN, uint64_t Ncap,
                                     uint32_t lo_bit, uint32_t hi_bit, uint32_t width,
                                     const unsigned long long *ghist, uint32_t *err, const OnesweepBufs &b,
                                     hipStream_t s) {
    onesweep_sort_planned<uint32_t>(keys, alt, dN, Ncap, lo_bit, hi_bit, width, ghist, err, b, s, "pair_sort");
}

bool radix_sort_onesweep(DevBuf<uint64_t> &keys, DevBuf<uint64_t> &alt, uint64_t N, uint32_t lo_bit,
                         uint32_t hi_bit, uint32_t width, const unsigned long long *ghist, uint32_t *err,
                         hipStream_t s, Budget *b, Arena *ar, const KeySource *src, const uint64_t *first) {
    return onesweep_sort<uint64_t>(keys, alt, N, lo_bit, hi_bit, width, ghist, err, s, b, ar, "radix_onesweep", src,
                                   first);
}

bool radix_sort_onesweep_u32(DevBuf<uint32_t> &keys, DevBuf<uint32_t> &alt, uint64_t N, uint32_t lo_bit,
                             uint32_t hi_bit, uint32_t width, const unsigned long long *ghist, uint32_t *err,
                             hipStream_t s, Budget *b, Arena *ar) {
    return onesweep_sort<uint32_t>(keys, alt, N, lo_bit, hi_bit, width, ghist, err, s, b, ar, "pair_sort");
}

}  // namespace jas
