// Encoding of the indicator matrix A (Sec. III-B).
//
// Input: CSR sets.  Keys (id << sbits) | sample are built in CSR order, which
// is already ascending in `sample`, so a stable sort on the ID bits alone
// leaves every ID's entries together with samples ascending.  The global sort
// (radix.hip) orders the keys by their top ID bits only; each range of whole
// buckets is finished here, in LDS (k_local_cls).
//
// After the sort (encode_sorted):
//   classify   first occurrence of a key = a distinct (ID, sample) pair, i.e. a
//              nonzero of A (repeats dropped: the (max, x) write of Sec. IV-A);
//              |X_i| = entries of sample i minus its repeats (column sums,
//              Eq. (4)); an ID's run of distinct pairs is one nonzero row of A
//              (the filter of Eq. (5)); rows with >= 2 pairs ("shared") are the
//              only rows off-diagonal B depends on, because a row with one
//              nonzero adds only to B_ii = |X_i|.
//   compaction shared rows are numbered in ID order by a prefix sum (Eq. (6)).
//   split      rows of degree >= dmin are bit-packed; rows of degree 2..dmin-1
//              are kept as row lists: their pairs, sorted by the smaller
//              sample, are counted per sample in the Gram step.
//   batches    packed rows are grouped by batch l = id >> batch_bits (Eq. (3));
//              inside a batch, row p (in ID order) is bit p % 64 of word row
//              p / 64, so words never straddle batches.
//   pack       one block per word row ORs the bits of its <= 64 rows into an
//              LDS row of n words and writes it out: W[w][i] is the word of
//              column i (the bitmask compression preceding Eq. (7)).
#include <algorithm>
#include <utility>

#include "device_util.hpp"
#include "jas_internal.hpp"
#include "onesweep_index.hpp"

namespace jas {
namespace {

constexpr int kNT = 256;
constexpr int kWaves = kNT / kWave;
constexpr int kRounds = 16;
constexpr uint32_t kTile = kNT * kRounds;  // 4096
constexpr uint64_t kChunk = 65536;         // elements per classify block
constexpr int32_t kHistMax = 16384;        // LDS column histogram up to this n
constexpr uint32_t kPackCols = 10112;      // LDS words per pack pass, at most (two blocks per CU)
constexpr uint32_t kPackLoads = 8;         // sample loads in flight per lane in k_pack
constexpr uint32_t kPackFlat = 6144;       // k_pack: word rows with at most this many entries deal them out one by one

// ---------------------------------------------------------------------------
// Keys of one chunk of entries per block, and the totals of every digit
// of every global sort pass (ghist, kGhistReplicas copies summed later, a row
// of 256 digits per pass, or 512 for 9-bit passes), which the single-pass
// scatter needs.  Pass q's digit is ID bits [idlo + width*q, idlo + width*(q+1)).  k_count_digits only counts (and
// checks the IDs): the sort's first pass then forms the keys itself.
template <bool kWrite>
__device__ __forceinline__ void build_keys_chunk(const uint64_t *__restrict__ ids, const uint64_t *__restrict__ off,
                                                 int32_t n, uint64_t N, uint32_t sbits, uint64_t hi_mask,
                                                 uint64_t *__restrict__ keys, uint32_t *err, uint32_t npass,
                                                 uint32_t idlo, uint32_t width,
                                                 unsigned long long *__restrict__ ghist,
                                                 const uint64_t *__restrict__ dsz, uint32_t chunk) {
    __shared__ int32_t s_lo, s_hi;
    __shared__ uint32_t gh[kMaxPasses * 256];
    const uint32_t tid = threadIdx.x;
    const uint32_t radix = onesweep::radix_of(width);  // npass * radix <= kMaxPasses * 256
    if (plan_aborted(dsz)) return;
    if (dsz) N = dsz[PZ_N];
    const uint64_t b0 = (uint64_t)blockIdx.x * chunk;
    if (b0 >= N) return;  // a planned launch covers the largest N
    const uint64_t b1 = min(N, b0 + chunk);
    constexpr uint32_t kAhead = 4;  // IDs in flight per thread: 1.78 G IDs 2.88 ms with one, 2.63 with 4, 2.68 with 8
    const uint32_t dmask = (1u << width) - 1u;
    for (uint32_t i = tid; i < npass * radix; i += kNT) gh[i] = 0;
    if (kWrite && tid == 0) {
        s_lo = find_sample(off, 0, n - 1, b0);
        s_hi = find_sample(off, s_lo, n - 1, b1 - 1);
    }
    __syncthreads();
    // A wave whose entries share a digit above the lowest (sets of ascending,
    // dense IDs) adds them with one atomic instead of 64 on one LDS word.  Each
    // wave decides once, from the top digit of its first 64 entries, whether
    // to look for such runs (IDs in no particular order never share it).
    bool agg = false;
    if (npass > 1) {
        const uint64_t t = b0 + tid;
        const uint32_t d = t < b1 ? (uint32_t)(ids[t] >> (idlo + width * (npass - 1))) & dmask : 0u;
        agg = __ballot(t < b1 && d == (uint32_t)__builtin_amdgcn_readfirstlane(d)) == __ballot(t < b1);
    }
    uint32_t bad = 0;
    int32_t lo = kWrite ? s_lo : 0;
    const auto take = [&](uint64_t t, uint64_t id) {
        bad |= (id & hi_mask) != 0;
        // the last pass sorts only the digit bits below U: with the others counted, an ID >= 2^U (refused later)
        // would be counted by another digit than it is sorted by, and places would be left unwritten
        id &= ~hi_mask;
        if constexpr (kWrite) {
            lo = find_sample(off, lo, s_hi, t);  // t only grows, so the search range only shrinks
            keys[t] = (id << sbits) | (uint64_t)lo;
        }
        if (agg) {  // wave-uniform
            const uint64_t active = __ballot(true);
            for (uint32_t q = 0; q < npass; ++q) {
                const uint32_t d = (uint32_t)(id >> (idlo + width * q)) & dmask;
                if (q > 0 && __ballot(d == (uint32_t)__builtin_amdgcn_readfirstlane(d)) == active) {
                    if (lane_id() == (uint32_t)__builtin_ctzll(active))
                        atomicAdd(&gh[q * radix + d], (uint32_t)__popcll(active));
                } else {
                    atomicAdd(&gh[q * radix + d], 1u);
                }
            }
        } else {
            for (uint32_t q = 0; q < npass; ++q)
                atomicAdd(&gh[q * radix + ((uint32_t)(id >> (idlo + width * q)) & dmask)], 1u);
        }
    };
    uint64_t t = b0 + tid;
    for (; t + (kAhead - 1) * kNT < b1; t += kAhead * kNT) {
        uint64_t id[kAhead];
#pragma unroll
        for (uint32_t u = 0; u < kAhead; ++u) id[u] = ids[t + u * kNT];
#pragma unroll
        for (uint32_t u = 0; u < kAhead; ++u) take(t + u * kNT, id[u]);
    }
    for (; t < b1; t += kNT) take(t, ids[t]);
    if (__ballot(bad) && lane_id() == 0) atomicOr(err, 1u);
    __syncthreads();
    unsigned long long *g = ghist + (uint64_t)(blockIdx.x % kGhistReplicas) * kMaxPasses * 256;
    for (uint32_t i = tid; i < npass * radix; i += kNT)
        if (gh[i]) atomicAdd(&g[i], (unsigned long long)gh[i]);
}

__global__ __launch_bounds__(kNT) void k_build_keys(const uint64_t *__restrict__ ids,
                                                     const uint64_t *__restrict__ off, int32_t n, uint64_t N,
                                                     uint32_t sbits, uint64_t hi_mask, uint64_t *__restrict__ keys,
                                                     uint32_t *err, uint32_t npass, uint32_t idlo, uint32_t width,
                                                     unsigned long long *__restrict__ ghist,
                                                     const uint64_t *__restrict__ dsz, uint32_t chunk) {
    build_keys_chunk<true>(ids, off, n, N, sbits, hi_mask, keys, err, npass, idlo, width, ghist, dsz, chunk);
}

__global__ __launch_bounds__(kNT) void k_count_digits(const uint64_t *__restrict__ ids, uint64_t N, uint64_t hi_mask,
                                                       uint32_t *err, uint32_t npass, uint32_t idlo, uint32_t width,
                                                       unsigned long long *__restrict__ ghist,
                                                       const uint64_t *__restrict__ dsz, uint32_t chunk) {
    build_keys_chunk<false>(ids, nullptr, 0, N, 0, hi_mask, nullptr, err, npass, idlo, width, ghist, dsz, chunk);
}

// Entries per block of the two kernels above: 2048 blocks are resident at once,
// and a block's threads take their entries one after another (about 0.55 us
// each), so fewer than 128 M entries are dealt out in shorter chunks.
// 638 K entries: 0.146 ms as 10 chunks of 65536, 0.012 ms as 312.  Longer chunks
// add fewer totals to memory.
uint32_t key_chunk(uint64_t N) {
    return (uint32_t)std::min<uint64_t>(std::max<uint64_t>(div_up(div_up(N, 2048), kNT) * kNT, 8 * kNT), kChunk);
}

__global__ void k_fill_u64(uint64_t *p, uint64_t len, uint64_t v) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < len; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// ---------------------------------------------------------------------------
// Classification of the sorted keys.  A block owns a chunk of kChunk keys and
// walks it in tiles of kTile; each tile is staged in LDS with one key of halo
// on each side, so the neighbours that decide an element come from LDS.
//   first    K[t] != K[t-1]: the first copy of a distinct (ID, sample) pair;
//   left     the previous distinct pair has the same ID (not the row's first);
//   right    the next distinct pair (after any copies of K[t]) has the same ID;
//   shared   first && (left || right): the row has >= 2 distinct pairs;
//   rowstart shared && !left;  newid = first && !left (one per nonzero row).
struct Cls {
    bool first, shared, rowstart, newid;
};

// L[0..cnt+1] = K[t0-1 .. t0+cnt] (out-of-range ends are complements of their
// neighbour so they compare unequal).  Element t0+i is L[i+1].
__device__ __forceinline__ void stage_tile(const uint64_t *__restrict__ K, uint64_t N, uint64_t t0, uint32_t cnt,
                                           uint64_t *L) {
    for (uint32_t i = threadIdx.x; i < cnt; i += kNT) L[i + 1] = K[t0 + i];
    if (threadIdx.x == 0) L[0] = t0 > 0 ? K[t0 - 1] : ~K[t0];
    if (threadIdx.x == 1) L[cnt + 1] = (t0 + cnt < N) ? K[t0 + cnt] : ~K[t0 + cnt - 1];
}

__device__ __forceinline__ Cls classify_lds(const uint64_t *__restrict__ K, uint64_t N, uint64_t t0, uint32_t cnt,
                                            const uint64_t *L, uint32_t i, uint32_t sbits) {
    Cls c;
    const uint64_t key = L[i + 1], prev = L[i];
    const uint64_t id = key >> sbits;
    const uint64_t t = t0 + i;
    c.first = (t == 0) || prev != key;
    const bool left = c.first && t > 0 && (prev >> sbits) == id;
    bool right = false;
    if (c.first) {
        // next distinct key: in the tile (or its halo), else (long runs of copies) in global memory
        uint32_t j = i + 2;
        while (j <= cnt + 1 && L[j] == key) ++j;
        uint64_t nxt;
        bool have = true;
        if (j <= cnt + 1) {
            nxt = L[j];
            have = t0 + (j - 1) < N;
        } else {
            uint64_t u = t0 + cnt + 1;
            while (u < N && K[u] == key) ++u;
            have = u < N;
            nxt = have ? K[u] : 0;
        }
        right = have && (nxt >> sbits) == id;
    }
    c.shared = c.first && (left || right);
    c.rowstart = c.shared && !left;
    c.newid = c.first && !left;
    return c;
}

__global__ __launch_bounds__(kNT) void k_cls_count(const uint64_t *__restrict__ K, uint64_t N, uint32_t sbits,
                                                    uint64_t smask, int32_t n, int lds_hist, uint32_t *cD,
                                                    uint32_t *cS, uint32_t *cR, unsigned long long *card,
                                                    unsigned long long *st) {
    extern __shared__ uint32_t hist[];
    __shared__ uint64_t L[kTile + 2];
    __shared__ uint64_t sh[kWaves];
    const uint32_t tid = threadIdx.x;
    if (lds_hist)
        for (int32_t i = tid; i < n; i += kNT) hist[i] = 0;
    const uint64_t c0 = (uint64_t)blockIdx.x * kChunk;
    const uint64_t c1 = min(N, c0 + kChunk);
    uint32_t nD = 0, nS = 0, nR = 0, nI = 0;
    for (uint64_t t0 = c0; t0 < c1; t0 += kTile) {
        const uint32_t cnt = (uint32_t)min((uint64_t)kTile, c1 - t0);
        __syncthreads();
        stage_tile(K, N, t0, cnt, L);
        __syncthreads();
        for (uint32_t i = tid; i < cnt; i += kNT) {
            const Cls c = classify_lds(K, N, t0, cnt, L, i, sbits);
            if (c.first) {
                ++nD;
                const uint32_t s = (uint32_t)(L[i + 1] & smask);
                if (s < (uint32_t)n) {
                    if (lds_hist) atomicAdd(&hist[s], 1u);
                    else atomicAdd(&card[s], 1ull);
                }
            }
            nS += c.shared;
            nR += c.rowstart;
            nI += c.newid;
        }
    }
    uint64_t tD, tS, tR, tI;
    block_excl_scan<kNT>(nD, sh, &tD);
    block_excl_scan<kNT>(nS, sh, &tS);
    block_excl_scan<kNT>(nR, sh, &tR);
    block_excl_scan<kNT>(nI, sh, &tI);
    if (tid == 0) {
        cD[blockIdx.x] = (uint32_t)tD;
        cS[blockIdx.x] = (uint32_t)tS;
        cR[blockIdx.x] = (uint32_t)tR;
        atomicAdd(&st[ST_PAIRS], (unsigned long long)tD);
        atomicAdd(&st[ST_ROWS], (unsigned long long)tI);
    }
    if (lds_hist)
        for (int32_t i = tid; i < n; i += kNT)
            if (hist[i]) atomicAdd(&card[i], (unsigned long long)hist[i]);
}

// Ordered compaction of the classified elements of one chunk: wave w of a
// tile owns its elements [w*1024, (w+1)*1024), 64 per round, in order.
__global__ __launch_bounds__(kNT) void k_cls_write(const uint64_t *__restrict__ K, uint64_t N, uint32_t sbits,
                                                    uint64_t smask, const uint64_t *oD, const uint64_t *oS,
                                                    const uint64_t *oR, uint64_t *Dout, uint32_t *Sout,
                                                    uint64_t *row_id, uint64_t *row_ptr) {
    __shared__ uint64_t L[kTile + 2];
    __shared__ uint32_t wc[3][kWaves];
    __shared__ uint64_t run[3];
    const uint32_t tid = threadIdx.x, lane = lane_id(), w = tid / kWave;
    const uint64_t lt = lanemask_lt();
    const uint64_t c0 = (uint64_t)blockIdx.x * kChunk;
    const uint64_t c1 = min(N, c0 + kChunk);
    if (tid == 0) {
        run[0] = oD[blockIdx.x];
        run[1] = oS[blockIdx.x];
        run[2] = oR[blockIdx.x];
    }
    for (uint64_t t0 = c0; t0 < c1; t0 += kTile) {
        const uint32_t cnt = (uint32_t)min((uint64_t)kTile, c1 - t0);
        __syncthreads();
        stage_tile(K, N, t0, cnt, L);
        __syncthreads();
        const uint32_t wb = w * (kTile / kWaves);
        uint32_t fD = 0, fS = 0, fR = 0;
        uint32_t nD = 0, nS = 0, nR = 0;
#pragma unroll 2
        for (int j = 0; j < kRounds; ++j) {
            const uint32_t i = wb + j * kWave + lane;
            bool d = false, s = false, r = false;
            if (i < cnt) {
                const Cls c = classify_lds(K, N, t0, cnt, L, i, sbits);
                d = c.first;
                s = c.shared;
                r = c.rowstart;
            }
            fD |= (uint32_t)d << j;
            fS |= (uint32_t)s << j;
            fR |= (uint32_t)r << j;
            nD += __popcll(__ballot(d));
            nS += __popcll(__ballot(s));
            nR += __popcll(__ballot(r));
        }
        if (lane == 0) {
            wc[0][w] = nD;
            wc[1][w] = nS;
            wc[2][w] = nR;
        }
        __syncthreads();
        uint64_t pD = run[0], pS = run[1], pR = run[2];
        for (uint32_t k = 0; k < w; ++k) {
            pD += wc[0][k];
            pS += wc[1][k];
            pR += wc[2][k];
        }
#pragma unroll
        for (int j = 0; j < kRounds; ++j) {
            const bool d = (fD >> j) & 1u, s = (fS >> j) & 1u, r = (fR >> j) & 1u;
            const uint64_t bd = __ballot(d), bs = __ballot(s), br = __ballot(r);
            const uint64_t posD = pD + __popcll(bd & lt);
            const uint64_t posS = pS + __popcll(bs & lt);
            const uint64_t posR = pR + __popcll(br & lt);
            if (d | s) {
                const uint64_t key = L[wb + j * kWave + lane + 1];
                if (d && Dout) Dout[posD] = key;
                if (s) Sout[posS] = (uint32_t)(key & smask);
                if (r) {
                    row_id[posR] = key >> sbits;
                    row_ptr[posR] = posS;
                }
            }
            pD += __popcll(bd);
            pS += __popcll(bs);
            pR += __popcll(br);
        }
        __syncthreads();
        if (tid == 0) {
            for (int k = 0; k < kWaves; ++k) {
                run[0] += wc[0][k];
                run[1] += wc[1][k];
                run[2] += wc[2][k];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Classification in LDS after a sort of the top ID bits only.
//
// The keys are ordered by bucket = key >> bsh (the top ID bits) and, inside a
// bucket, still in input order (every pass was stable, so entries of one ID
// are in ascending sample order).  Range c runs from the first bucket edge at
// or after c*stride to the first at or after (c+1)*stride (k_range_starts);
// the encoder tries the strides of kLocalStrides in turn until no range
// exceeds kLocalCapKeys, and launches the kernel built for kLocalShortCap keys
// when every range fits it, else the one for kLocalCapKeys.
// A range is made of whole buckets, so it holds whole rows of A and needs no
// halo.  One block loads a range (<= Cap keys) into LDS, finishes
// the sort there (stable LSD passes over the ID bits below the range's first
// bucket), classifies as k_cls_count/k_cls_write do, and writes its results
// at the range's own position (distinct keys in place over the range, shared
// pairs at the range start, rows at half the range start) with its counts;
// k_local_move then packs them after a scan of the counts.  A range longer
// than the cap (a bucket with very many keys) sets err bit 8 before any
// block writes; when it does at every try the caller sorts every ID bit
// and uses k_cls_count/k_cls_write.
constexpr int kLNT = 512;
constexpr int kLWaves = kLNT / kWave;

__device__ __forceinline__ uint64_t bucket_of(uint64_t key, uint32_t bsh) { return bsh >= 64 ? 0 : key >> bsh; }
__device__ __forceinline__ uint64_t div_up_dev(uint64_t a, uint64_t b) { return (a + b - 1) / b; }
__device__ __forceinline__ uint32_t dev_ceil_log2(uint64_t v) { return v <= 1 ? 0u : 64u - (uint32_t)__clzll(v - 1); }

// rs[c] = first bucket edge at or after c*stride, c in [0, nlc]; positions
// 0 and N are edges.  One wave per c, 256 keys per step.  An edge more than
// cap keys away is not looked for: rs[c] = ~0 and err |= 8.  Planned: nor is any
// edge when the ID check or the sort has failed (err bits 1, 2, 4, set by earlier
// launches): places of the keys may then be unwritten, and a range without a
// start is not classified.
__global__ __launch_bounds__(256) void k_range_starts(const uint64_t *__restrict__ K, uint64_t N, uint32_t bsh,
                                                       uint64_t stride, uint64_t nlc, uint64_t *__restrict__ rs,
                                                       uint32_t *err, const uint64_t *__restrict__ dsz,
                                                       uint32_t cap) {
    if (plan_aborted(dsz)) return;
    if (dsz) {
        N = dsz[PZ_N];
        nlc = div_up_dev(N, stride);
    }
    const uint64_t c = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const uint32_t lane = lane_id();
    if (c > nlc) return;  // whole waves
    if (dsz && (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 7u)) {
        if (lane == 0) rs[c] = ~0ull;
        return;
    }
    const uint64_t x = c * stride;
    if (x == 0 || x >= N) {
        if (lane == 0) rs[c] = min(x, N);
        return;
    }
    const uint64_t b0 = bucket_of(K[x - 1], bsh);
    for (uint64_t y = x; y < x + cap; y += 4 * kWave) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint64_t t = y + k * kWave + lane;
            const uint64_t m = __ballot(t >= N || bucket_of(K[t], bsh) != b0);
            if (m) {
                if (lane == 0) rs[c] = y + k * kWave + (uint64_t)__builtin_ctzll(m);
                return;
            }
        }
    }
    if (lane == 0) {
        rs[c] = ~0ull;
        atomicOr(err, 8u);
    }
}

// Checks every range (err |= 8 as above), whether it is longer than
// kLocalShortCap (err |= 128) and whether its keys fit 32 bits once made
// relative to the range's first bucket: ((id - rbase) << sbits) | sample, with
// rbase = first bucket << lowbits, needs lowbits + ceil_log2(the number of
// bucket values spanned) + sbits bits; err |= 16 where that exceeds 32.
// The flags of a thread's ranges are gathered first and set with one atomic
// per wave (every range may set bits 16 and 128).
__global__ void k_range_check(const uint64_t *__restrict__ K, const uint64_t *rs, uint64_t nlc, uint32_t bsh,
                              uint32_t lowbits, uint32_t sbits, uint32_t *err, const uint64_t *__restrict__ dsz,
                              uint64_t stride, uint32_t cap) {
    if (plan_aborted(dsz)) return;
    if (dsz) nlc = div_up_dev(dsz[PZ_N], stride);
    uint32_t f = 0;
    for (uint64_t c = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; c < nlc; c += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t a = rs[c], b = rs[c + 1];
        if (a == ~0ull || b == ~0ull || b < a || b - a > cap) {
            f |= 8u;
        } else if (b > a) {
            if (b - a > kLocalShortCap) f |= 128u;
            const uint64_t bf = bucket_of(K[a], bsh), bl = bucket_of(K[b - 1], bsh);
            if (lowbits + dev_ceil_log2(bl - bf + 1) + sbits > 32) f |= 16u;
        }
    }
    const uint64_t m8 = __ballot((f & 8u) != 0), m16 = __ballot((f & 16u) != 0), m128 = __ballot((f & 128u) != 0);
    if (lane_id() == 0 && (m8 | m16 | m128))
        atomicOr(err, (m8 ? 8u : 0u) | (m16 ? 16u : 0u) | (m128 ? 128u : 0u));
}

// KT is the LDS form of a key, relative to the range's first bucket:
// uint32_t when every range fits 32 bits (k_range_check), else uint64_t.
// Cap is the most keys of a range.  Blocks per CU (by LDS and registers): 4
// for 32-bit keys and Cap 4096, 3 for 32-bit keys and Cap 6144 or 64-bit keys
// and Cap 4096, 2 for 64-bit keys and Cap 6144; the register budget matches.
//
// The in-LDS sort bounds it, not the 8 bytes read per key.  Keys stay in
// registers from the load to the first pass and between passes; ranks come
// from ballots (VALU), which leaves LDS five operations per key and pass where
// finding the lanes of one digit through an LDS table took eight; passes of up
// to 9 bits take the ID bits in the fewest, equal parts (18 bits: two, where
// 8-bit passes took three).  1.78 G keys of 22 relative ID bits 18.2 -> 12.9 ms,
// 1.60 G of 15 bits 16.3 -> 11.2, 1.47 G of 18 bits 14.7 -> 9.1, 336 M of 9 bits
// 2.85 -> 1.63.
constexpr int local_cls_waves(size_t kt, uint32_t cap) { return kt == 4 ? (cap <= 4096 ? 8 : 6) : (cap <= 4096 ? 6 : 4); }
constexpr uint32_t kLDigits = 512;  // an LDS pass sorts at most 9 bits
typedef uint16_t __attribute__((may_alias)) u16_alias;

// Ranks of a wave's keys (R rounds of 64, of which `rounds` hold any) by digit
// (key >> dsh) & mask < 2^NB: lanes of a round with the same digit take
// consecutive slots after the digit's count so far in cnt (16 bits per digit),
// and the lowest of them adds the group to the count.  One wave's LDS
// operations run in order, so no round waits for another's.
template <int NB, uint32_t R, class KT>
__device__ __forceinline__ void rank_keys(const KT (&key)[R], uint32_t (&rank)[R], uint32_t rounds, uint32_t dsh,
                                          uint32_t mask, uint32_t *cnt) {
    uint32_t before[R];
#pragma unroll
    for (uint32_t j = 0; j < R; ++j) {
        if (j < rounds) {  // uniform
            const uint32_t d = (uint32_t)(key[j] >> dsh) & mask;
            const uint64_t peers = wave_match<NB>(d);
            before[j] = lanes_before(peers);
            rank[j] = __hip_atomic_load(&cnt[d >> 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >> (16 * (d & 1));
            if (before[j] == 0)
                __hip_atomic_fetch_add(&cnt[d >> 1], (uint32_t)__popcll(peers) << (16 * (d & 1)), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
#pragma unroll
    for (uint32_t j = 0; j < R; ++j)
        if (j < rounds) rank[j] = (rank[j] & 0xFFFFu) + before[j];
}

template <class KT, uint32_t Cap>
__global__ __launch_bounds__(kLNT) __attribute__((amdgpu_waves_per_eu(local_cls_waves(sizeof(KT), Cap)))) void k_local_cls(
    uint64_t *__restrict__ K, uint32_t sbits, uint64_t smask, uint32_t bsh, uint32_t lowbits,
    const uint64_t *__restrict__ rs, uint32_t nlc, uint32_t *__restrict__ cnt, int keep, uint32_t *__restrict__ Sg,
    uint64_t *__restrict__ rid_g, uint64_t *__restrict__ rptr_g, unsigned long long *__restrict__ dupc,
    unsigned long long *__restrict__ row_slots, uint32_t slots, const uint64_t *__restrict__ dsz, uint64_t stride,
    uint32_t *err) {
    static_assert(Cap <= kLocalCapKeys && Cap % kLNT == 0 && kLDigits == kLNT, "range cap");
    constexpr uint32_t kLRounds = Cap / kLNT;  // keys per thread
    __shared__ KT A[Cap];
    // per wave and digit d: a 16-bit count (then start) in half d & 1 of word
    // d >> 1; a wave adds to and reads only its own row
    __shared__ uint32_t wcnt[kLWaves][kLDigits / 2];
    __shared__ uint64_t sh[kLWaves];
    __shared__ uint32_t sh32[kLWaves];
    __shared__ uint32_t wc[3][kLWaves];
    const uint32_t tid = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(tid / kWave);
    const uint64_t lt = lanemask_lt();
    const uint32_t c = blockIdx.x;
    if (plan_aborted(dsz)) return;
    {
        // a planned launch covers the most ranges; the others count nothing,
        // and a range this kernel cannot hold is flagged and skipped
        const bool beyond = dsz && c >= div_up_dev(dsz[PZ_N], stride);
        const bool bad = !beyond && (rs[c] == ~0ull || rs[c + 1] == ~0ull || rs[c + 1] < rs[c] ||
                                     rs[c + 1] - rs[c] > Cap);
        if (beyond || bad) {
            if (tid == 0) {
                cnt[c] = 0;
                cnt[nlc + c] = 0;
                cnt[2 * (uint64_t)nlc + c] = 0;
                if (bad) atomicOr(err, 8u);
            }
            return;
        }
    }
    const uint64_t s0 = rs[c], s1 = rs[c + 1];
    const uint32_t L = (uint32_t)(s1 - s0);  // <= Cap (k_range_check)
    // wave w owns positions [w*seg, (w+1)*seg), 64 per round, in order
    const uint32_t seg = ((L + kLWaves - 1) / kLWaves + kWave - 1) / kWave * kWave;
    const uint32_t rounds = seg / kWave;
    const uint32_t wb = w * seg;
    // relative keys: key - kbase = ((id - rbase) << sbits) | sample < 2^(nb + sbits)
    uint64_t kbase = 0;
    uint32_t nb = 0;
    if (L > 0) {
        const uint64_t bf = bucket_of(K[s0], bsh), bl = bucket_of(K[s1 - 1], bsh);
        kbase = bf ? (bf << lowbits) << sbits : 0;  // bf > 0 only when lowbits < U
        // with no ID bits below the buckets (every ID bit sorted globally)
        // the range is sorted already: a bucket is one ID, its keys in sample order
        nb = lowbits == 0 ? 0u : lowbits + dev_ceil_log2(bl - bf + 1);
    }
    {
        // the wave's keys, all loads in flight at once.  Entries past the range's
        // end are all ones: they take the largest digit in every pass and come
        // last in it, so they stay past the range's keys (kLWaves * seg <= Cap).
        KT key[kLRounds];
        {
            uint64_t v[kLRounds];
            const uint64_t *src = K + s0 + wb;
#pragma unroll
            for (uint32_t j = 0; j < kLRounds; ++j)
                v[j] = wb + j * kWave + lane < L ? src[j * kWave + lane] : ~0ull;
#pragma unroll
            for (uint32_t j = 0; j < kLRounds; ++j)
                key[j] = wb + j * kWave + lane < L ? (KT)(v[j] - kbase) : ~(KT)0;
        }
        // --- finish the sort: stable LSD passes over the relative ID, of equal
        // width, at most 9 bits
        const uint32_t npass = L > 1 ? (nb + 8) / 9 : 0, width = npass ? (nb + npass - 1) / npass : 0;
        for (uint32_t p = 0; p < npass; ++p) {
            const uint32_t dsh = sbits + p * width, mask = (1u << width) - 1u;
            uint32_t rank[kLRounds];
#pragma unroll
            for (uint32_t i = 0; i < kLDigits / 2; i += kWave) wcnt[w][i + lane] = 0;
            if (width <= 7) rank_keys<7>(key, rank, rounds, dsh, mask, wcnt[w]);
            else if (width == 8) rank_keys<8>(key, rank, rounds, dsh, mask, wcnt[w]);
            else rank_keys<9>(key, rank, rounds, dsh, mask, wcnt[w]);
            __syncthreads();
            // thread tid owns digit tid: its count per wave becomes where the wave's keys of it start
            uint32_t n_d[kLWaves], tot = 0;
#pragma unroll
            for (int k = 0; k < kLWaves; ++k) {
                n_d[k] = reinterpret_cast<const u16_alias *>(wcnt[k])[tid];
                tot += n_d[k];
            }
            uint32_t run = wave_incl_scan_u32(tot);
            if (lane == kWave - 1) sh32[w] = run;
            __syncthreads();
            run -= tot;
            for (uint32_t k = 0; k < w; ++k) run += sh32[k];
#pragma unroll
            for (int k = 0; k < kLWaves; ++k) {
                reinterpret_cast<u16_alias *>(wcnt[k])[tid] = (uint16_t)run;
                run += n_d[k];
            }
            __syncthreads();
#pragma unroll
            for (uint32_t j = 0; j < kLRounds; ++j)
                if (j < rounds)
                    A[reinterpret_cast<const u16_alias *>(wcnt[w])[(uint32_t)(key[j] >> dsh) & mask] + rank[j]] = key[j];
            __syncthreads();
            if (p + 1 < npass) {
#pragma unroll
                for (uint32_t j = 0; j < kLRounds; ++j)
                    if (j < rounds) key[j] = A[wb + j * kWave + lane];
            }
        }
        if (npass == 0) {
#pragma unroll
            for (uint32_t j = 0; j < kLRounds; ++j)
                if (j < rounds) A[wb + j * kWave + lane] = key[j];
            __syncthreads();
        }
    }

    // --- classify (as classify_lds, with the whole row in LDS)
    uint32_t fD = 0, fS = 0, fR = 0;
    uint32_t nD = 0, nS = 0, nR = 0;
    uint64_t rows = 0;  // nonzero rows of A (distinct IDs) seen by this thread
    for (uint32_t j = 0; j < rounds; ++j) {
        const uint32_t t = wb + j * kWave + lane;
        bool d = false, sh_ = false, r = false;
        if (t < L) {
            const KT key = A[t], id = key >> sbits;
            const bool first = t == 0 || A[t - 1] != key;
            const bool left = first && t > 0 && (A[t - 1] >> sbits) == id;
            bool right = false;
            if (first) {
                uint32_t u = t + 1;
                while (u < L && A[u] == key) ++u;
                right = u < L && (A[u] >> sbits) == id;
            }
            d = first;
            sh_ = first && (left || right);
            r = sh_ && !left;
            rows += first && !left;
            if (!first && dupc) atomicAdd(&dupc[key & smask], 1ull);
        }
        fD |= (uint32_t)d << j;
        fS |= (uint32_t)sh_ << j;
        fR |= (uint32_t)r << j;
        nD += __popcll(__ballot(d));
        nS += __popcll(__ballot(sh_));
        nR += __popcll(__ballot(r));
    }
    if (lane == 0) {
        wc[0][w] = nD;
        wc[1][w] = nS;
        wc[2][w] = nR;
    }
    uint64_t all_rows;
    block_excl_scan<kLNT>(rows, sh, &all_rows);  // synchronises: wc is complete after it
    if (tid == 0) {
        uint32_t tD = 0, tS = 0, tR = 0;
        for (int k = 0; k < kLWaves; ++k) {
            tD += wc[0][k];
            tS += wc[1][k];
            tR += wc[2][k];
        }
        cnt[c] = tD;
        cnt[nlc + c] = tS;
        cnt[2 * (uint64_t)nlc + c] = tR;
        if (all_rows) atomicAdd(&row_slots[c % slots], (unsigned long long)all_rows);
    }

    // --- ordered writes at the range's own position (every read of the range is done)
    uint32_t pD = 0, pS = 0, pR = 0;
    for (uint32_t k = 0; k < w; ++k) {
        pD += wc[0][k];
        pS += wc[1][k];
        pR += wc[2][k];
    }
    const uint64_t r0 = s0 / 2;
    for (uint32_t j = 0; j < rounds; ++j) {
        const bool d = (fD >> j) & 1u, sh_ = (fS >> j) & 1u, r = (fR >> j) & 1u;
        const uint64_t bd = __ballot(d), bs = __ballot(sh_), br = __ballot(r);
        if (d | sh_) {
            const uint64_t key = kbase + (uint64_t)A[wb + j * kWave + lane];
            const uint32_t posS = pS + __popcll(bs & lt);
            if (d && keep) K[s0 + pD + __popcll(bd & lt)] = key;
            if (sh_) Sg[s0 + posS] = (uint32_t)(key & smask);
            if (r) {
                const uint64_t posR = r0 + pR + __popcll(br & lt);
                rid_g[posR] = key >> sbits;
                rptr_g[posR] = posS;
            }
        }
        pD += __popcll(bd);
        pS += __popcll(bs);
        pR += __popcll(br);
    }
}

// Launches the k_local_cls built for the key width and the range cap.
template <class... Args>
void launch_local_cls(bool wide, uint32_t cap, uint32_t grid, hipStream_t s, Args... args) {
    if (cap != kLocalShortCap && cap != kLocalCapKeys) fail(JAS_EDEVICE, "local classify: no kernel for this range cap");
    if (wide) {
        if (cap == kLocalShortCap) k_local_cls<uint64_t, kLocalShortCap><<<grid, kLNT, 0, s>>>(args...);
        else k_local_cls<uint64_t, kLocalCapKeys><<<grid, kLNT, 0, s>>>(args...);
    } else {
        if (cap == kLocalShortCap) k_local_cls<uint32_t, kLocalShortCap><<<grid, kLNT, 0, s>>>(args...);
        else k_local_cls<uint32_t, kLocalCapKeys><<<grid, kLNT, 0, s>>>(args...);
    }
}

// Packs the rows k_local_cls wrote per range (and, for the query index, the
// distinct keys): one block per range (grid-stride).  The shared pairs stay
// where the range wrote them (from its start, with gaps between ranges), so
// a row is row_deg entries of that array from row_ptr.
__global__ __launch_bounds__(256) void k_local_move(const uint64_t *__restrict__ rs, uint64_t nlc,
                                                     const uint64_t *__restrict__ oD, const uint64_t *__restrict__ oS,
                                                     const uint64_t *__restrict__ oR, const uint64_t *__restrict__ K,
                                                     const uint64_t *__restrict__ rid_g,
                                                     const uint64_t *__restrict__ rptr_g, uint64_t *__restrict__ Dk,
                                                     uint64_t *__restrict__ row_id, uint64_t *__restrict__ row_ptr,
                                                     uint32_t *__restrict__ row_deg, const uint64_t *__restrict__ dsz,
                                                     uint64_t stride) {
    if (plan_aborted(dsz)) return;
    if (dsz) nlc = div_up_dev(dsz[PZ_N], stride);
    for (uint64_t c = blockIdx.x; c < nlc; c += gridDim.x) {
        const uint64_t s0 = rs[c], r0 = s0 / 2;
        const uint64_t d0 = oD[c], nd = oD[c + 1] - d0;
        const uint64_t ns = oS[c + 1] - oS[c];
        const uint64_t w0 = oR[c], nr = oR[c + 1] - w0;
        for (uint64_t i = threadIdx.x; i < nr; i += blockDim.x) {
            row_id[w0 + i] = rid_g[r0 + i];
            const uint64_t a = rptr_g[r0 + i];
            row_ptr[w0 + i] = s0 + a;
            row_deg[w0 + i] = (uint32_t)((i + 1 < nr ? rptr_g[r0 + i + 1] : ns) - a);
        }
        if (Dk)
            for (uint64_t i = threadIdx.x; i < nd; i += blockDim.x) Dk[d0 + i] = K[s0 + i];
    }
}

// Degrees of contiguous rows: row_deg[r] = row_ptr[r + 1] - row_ptr[r].
__global__ void k_row_deg(const uint64_t *row_ptr, uint64_t R, uint32_t *row_deg) {
    for (uint64_t r = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; r < R; r += (uint64_t)gridDim.x * blockDim.x)
        row_deg[r] = (uint32_t)(row_ptr[r + 1] - row_ptr[r]);
}

// |X_i| = entries of sample i minus its repeated (ID, sample) entries; err |= 64
// when one reaches the limit (int32 B needs every |X_i| < 2^31).
__global__ void k_card_from_dups(const uint64_t *off, const unsigned long long *dupc, int32_t n, int64_t *card,
                                 int64_t limit, uint32_t *err) {
    bool over = false;
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const int64_t c = (int64_t)((off[i + 1] - off[i]) - dupc[i]);
        card[i] = c;
        over |= c >= limit;
    }
    if (__ballot(over) && lane_id() == 0) atomicOr(err, 64u);
}

// Row degree histogram (degrees are <= n): input of the degree threshold choice.
__global__ __launch_bounds__(kNT) void k_deg_hist(const uint32_t *row_deg, uint64_t R, uint32_t nb,
                                                   int lds, unsigned long long *hist) {
    extern __shared__ uint32_t h[];
    if (lds)
        for (uint32_t i = threadIdx.x; i < nb; i += kNT) h[i] = 0;
    __syncthreads();
    for (uint64_t r = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; r < R; r += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t d = min((uint64_t)row_deg[r], (uint64_t)(nb - 1));
        if (lds) atomicAdd(&h[d], 1u);
        else atomicAdd(&hist[d], 1ull);
    }
    __syncthreads();
    if (lds)
        for (uint32_t i = threadIdx.x; i < nb; i += kNT)
            if (h[i]) atomicAdd(&hist[i], (unsigned long long)h[i]);
}

// Rows: degree split.
// Row split by degree in two passes over tiles of kSplitTile rows (8
// consecutive rows per thread): k_row_count counts each tile's packed rows
// (degree >= dmin) and the list rows' pairs; after a scan of the tile counts
// k_row_split places every row: packed row r at its tile's offset plus the
// packed rows before it in the tile, list row r at r minus the packed rows
// before it.
constexpr uint32_t kSplitPer = 8;
constexpr uint64_t kSplitTile = (uint64_t)kNT * kSplitPer;
static_assert(kSplitTile == kSplitTilePub, "row split tile");

// The 8 degrees of rows [r0, r0 + 8) (two 16-byte loads when all exist; r0 is a
// multiple of 8, so they are aligned); rows past R read as degree 0.
__device__ __forceinline__ void load_degrees(const uint32_t *__restrict__ row_deg, uint64_t r0, uint64_t R,
                                             uint32_t (&d)[kSplitPer]) {
    if (r0 + kSplitPer <= R) {
        const uint4 a = *reinterpret_cast<const uint4 *>(row_deg + r0);
        const uint4 b = *reinterpret_cast<const uint4 *>(row_deg + r0 + 4);
        d[0] = a.x; d[1] = a.y; d[2] = a.z; d[3] = a.w;
        d[4] = b.x; d[5] = b.y; d[6] = b.z; d[7] = b.w;
    } else {
#pragma unroll
        for (uint32_t k = 0; k < kSplitPer; ++k) d[k] = r0 + k < R ? row_deg[r0 + k] : 0u;
    }
}

__global__ __launch_bounds__(kNT) void k_row_count(const uint32_t *__restrict__ row_deg, uint64_t R, uint32_t dmin,
                                                    uint32_t *__restrict__ tcnt, unsigned long long *pair_slots,
                                                    uint32_t slots, const uint64_t *__restrict__ dsz) {
    __shared__ uint64_t sh[kWaves], sh2[kWaves];
    if (plan_aborted(dsz)) return;
    if (dsz) R = dsz[PZ_R];  // tiles past R count nothing
    const uint64_t r0 = (uint64_t)blockIdx.x * kSplitTile + (uint64_t)threadIdx.x * kSplitPer;
    uint64_t nd = 0, lp = 0;
    uint32_t dg[kSplitPer];
    load_degrees(row_deg, r0, R, dg);
#pragma unroll
    for (uint32_t k = 0; k < kSplitPer; ++k) {
        if (r0 + k < R) {
            const uint64_t d = dg[k];
            if (d >= dmin) ++nd;
            else lp += d * (d - 1) / 2;
        }
    }
    // block sums of both (one pass: wave sums, then thread 0)
    const uint64_t wd = wave_incl_scan(nd), wp = wave_incl_scan(lp);
    if (lane_id() == kWave - 1) {
        sh[threadIdx.x / kWave] = wd;
        sh2[threadIdx.x / kWave] = wp;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t tot_d = 0, tot_p = 0;
#pragma unroll
        for (int k = 0; k < kWaves; ++k) {
            tot_d += sh[k];
            tot_p += sh2[k];
        }
        tcnt[blockIdx.x] = (uint32_t)tot_d;
        if (tot_p) atomicAdd(&pair_slots[blockIdx.x % slots], (unsigned long long)tot_p);
    }
}

__global__ __launch_bounds__(kNT) void k_row_split(const uint32_t *__restrict__ row_deg, uint64_t R, uint32_t dmin,
                                                    const uint64_t *__restrict__ toff, uint64_t *__restrict__ Drow,
                                                    uint64_t *__restrict__ Lrow, const uint64_t *__restrict__ dsz) {
    __shared__ uint64_t sh[kWaves];
    if (plan_aborted(dsz)) return;
    // planned: with every shared row of one form the maps are the identity
    // (the kernels that read them check the same sizes)
    if (dsz && (dsz[PZ_QD] == 0 || dsz[PZ_QL] == 0)) return;
    if (dsz) R = dsz[PZ_R];
    const uint64_t r0 = (uint64_t)blockIdx.x * kSplitTile + (uint64_t)threadIdx.x * kSplitPer;
    uint32_t flags = 0, nd = 0;
    uint32_t dg[kSplitPer];
    load_degrees(row_deg, r0, R, dg);
#pragma unroll
    for (uint32_t k = 0; k < kSplitPer; ++k) {
        if (r0 + k < R && dg[k] >= dmin) {
            flags |= 1u << k;
            ++nd;
        }
    }
    uint64_t tot;
    uint64_t pd = toff[blockIdx.x] + block_excl_scan<kNT>(nd, sh, &tot);  // packed rows before r0
#pragma unroll
    for (uint32_t k = 0; k < kSplitPer; ++k) {
        const uint64_t r = r0 + k;
        if (r < R) {
            if ((flags >> k) & 1u) Drow[pd++] = r;
            else Lrow[r - pd] = r;
        }
    }
}

// Whether the packed-row map Drow / the list-row map Lrow is read: a null map,
// or (planned) every shared row of that form, is the identity.
__device__ __forceinline__ bool packed_map_used(const uint64_t *Drow, const uint64_t *dsz) {
    return Drow && !(dsz && dsz[PZ_QL] == 0);
}
__device__ __forceinline__ bool list_map_used(const uint64_t *Lrow, const uint64_t *dsz) {
    return Lrow && !(dsz && dsz[PZ_QD] == 0);
}

// Batches of packed rows.  Drow maps packed row q to its shared row; null
// when every shared row is packed (q itself), here and in k_pack.
// (planned: flags for q < QD, zeros up to the capacity QDcap = the host QD)
__global__ void k_batch_flag(const uint64_t *Drow, const uint64_t *row_id, uint64_t QD, uint32_t bbits,
                             uint32_t *bs, const uint64_t *__restrict__ dsz) {
    if (plan_aborted(dsz)) return;
    const uint64_t qd = dsz ? dsz[PZ_QD] : QD;
    if (!packed_map_used(Drow, dsz)) Drow = nullptr;
    for (uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; q < QD; q += (uint64_t)gridDim.x * blockDim.x) {
        if (q >= qd) {
            bs[q] = 0;
            continue;
        }
        const uint64_t b = row_id[Drow ? Drow[q] : q] >> bbits;
        bs[q] = (q == 0) || b != (row_id[Drow ? Drow[q - 1] : q - 1] >> bbits);
    }
}

__global__ void k_batch_start(const uint32_t *bs, const uint64_t *bpos, uint64_t QD, uint64_t *bq,
                              const uint64_t *__restrict__ dsz) {
    if (plan_aborted(dsz)) return;
    if (dsz) QD = dsz[PZ_QD];
    for (uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; q < QD; q += (uint64_t)gridDim.x * blockDim.x)
        if (bs[q]) bq[bpos[q]] = q;
}

// Word rows of b = wb bits (32 or 64) per batch: ceil(rows / b).
// (planned: nb batches, zeros up to the capacity nbcap = the host nb)
__global__ void k_batch_words(const uint64_t *bq, uint64_t nb, uint32_t wb, uint64_t *nw,
                              const uint64_t *__restrict__ dsz) {
    if (plan_aborted(dsz)) return;
    const uint64_t nbv = dsz ? dsz[PZ_NB] : nb;
    for (uint64_t b = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; b < nb; b += (uint64_t)gridDim.x * blockDim.x)
        nw[b] = b < nbv ? (bq[b + 1] - bq[b] + wb - 1) / wb : 0;
}

// Word row w (of wb bits) holds packed rows [wq0[w], wq1[w]): bit p % wb of
// row p / wb of its batch.
__global__ void k_word_rows(uint64_t QD, const uint64_t *bpos, const uint64_t *bq, const uint64_t *wbase, uint32_t wb,
                            uint64_t *wq0, uint64_t *wq1, const uint64_t *__restrict__ dsz) {
    if (plan_aborted(dsz)) return;
    if (dsz) QD = dsz[PZ_QD];
    for (uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; q < QD; q += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t b = bpos[q + 1] - 1;  // batch of packed row q
        const uint64_t p = q - bq[b];        // position inside the batch
        if (p % wb == 0) {
            const uint64_t w = wbase[b] + p / wb;
            wq0[w] = q;
            wq1[w] = min(q + wb, bq[b + 1]);
        }
    }
}

// G waves per 64-bit row of W: OR the bits of its <= 64 rows into an LDS
// row of words and write it out.  With b = 64 a row of W is one word row;
// with b = 32 it holds word rows 2w (bits 0..31) and 2w + 1 (bits 32..63),
// each a 32-bit word per column, so the Gram kernels read both as one 64-bit
// step (the AND + popcount, or the dot product, of a 64-bit element is the
// sum over its two halves).  Hw = word rows of b bits.  With a single batch
// (null wq0) word row w simply holds packed rows [w * b, (w + 1) * b) of the QD
// there are.
//
// W's bytes bound it once the waits are out of the way, which is what the split
// is for.  Every wave has the rows in its lanes (lane t: the row of bit t), so
// nothing is passed through LDS but the words and a bitmap of where the rows'
// entries start, and the next word row's are read while this one is packed.  An
// entry's row is the number of starts at or before it.  Words are cleared as
// they are written out.  Short word rows are a wave's work alone, without block
// barriers; long ones are spread over a block large enough that two fill a CU.
// 1.25 M rows of 1024 words (456 entries each): 7.9 ms with a block of 256
// threads for each and its entries' rows spelled out in LDS, 3.5 ms now (10.2 GB
// written); 65517 of 10112 (5960): 4.0, 2.1 ms (5.3 GB); 65536 of 4096 (17900):
// 1.9 both ways; 1090 of 128: 0.033, 0.010 ms.
template <int G>
__global__ __launch_bounds__(G < 4 ? 256 : G * kWave) void k_pack(
    uint64_t *__restrict__ W, uint64_t ldw, uint64_t H, uint64_t Hw, uint32_t wb, const uint64_t *__restrict__ wq0,
    const uint64_t *__restrict__ wq1, uint64_t QD, const uint64_t *__restrict__ Drow,
    const uint64_t *__restrict__ row_ptr, const uint32_t *__restrict__ row_deg, const uint32_t *__restrict__ S,
    uint32_t cols, unsigned long long *word_slots, uint32_t slots, const uint64_t *__restrict__ dsz) {
    constexpr uint32_t kTeam = G * kWave, kTeams = kTeam < 256 ? 256 / kTeam : 1;
    extern __shared__ __attribute__((aligned(16))) unsigned long long lds[];
    if (plan_aborted(dsz)) return;
    const uint32_t team = threadIdx.x / kTeam, tid = threadIdx.x % kTeam, lane = lane_id(), wv = tid / kWave;
    unsigned long long *lw = lds + team * cols;
    unsigned long long *starts = lds + kTeams * cols + team * (kPackFlat / 64 + 1);  // bitmap of the rows' first entries
    uint32_t *starts32 = reinterpret_cast<uint32_t *>(starts);
    uint32_t *zsh = starts32 + kPackFlat / 32;  // nonzero words of the row (b = 32: of each half)
    const auto sync = [] {
        if constexpr (G == 1) {
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else {
            __syncthreads();
        }
    };
    // planned: H is the capacity; rows from the actual count on are written as
    // zeros (they add nothing to the Gram product)
    const uint64_t Hv = dsz ? dsz[PZ_H] : H;
    if (!packed_map_used(Drow, dsz)) Drow = nullptr;
    if (dsz) Hw = dsz[PZ_HW];
    uint64_t next_base = 0;
    uint32_t next_deg = 0;
    const auto read_rows = [&](uint64_t w) {
        next_deg = 0;
        if (w >= Hv) return;
        const uint64_t ww = wb == 64 ? w : 2 * w + (lane >> 5);
        if (ww >= Hw) return;
        const uint64_t q0 = wq0 ? wq0[ww] : ww * wb, q1 = wq0 ? wq1[ww] : min(q0 + wb, QD);
        const uint64_t q = q0 + (wb == 64 ? lane : lane & 31);
        if (q >= q1) return;
        const uint64_t r = Drow ? Drow[q] : q;
        next_base = row_ptr[r];
        next_deg = row_deg[r];
    };
    // starts: bits of the rows in next_deg (wave 0)
    const auto mark_next = [&] {
        const uint32_t inc = wave_incl_scan_u32(next_deg), at = inc - next_deg;
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1);
        if (next_deg && total <= kPackFlat) atomicOr(&starts32[at >> 5], 1u << (at & 31));
    };
    const uint64_t step = (uint64_t)gridDim.x * kTeams;
    uint64_t w = (uint64_t)blockIdx.x * kTeams + team;
    read_rows(w);
    for (uint32_t i = tid; i < cols; i += kTeam) lw[i] = 0;
    for (uint32_t i = tid; i < kPackFlat / 64 + 1; i += kTeam) starts[i] = 0;
    sync();
    if (wv == 0) mark_next();
    sync();
    unsigned long long nnz_acc = 0, f_acc = 0;  // this team's totals (its first thread)
    for (; w < H; w += step) {
        if (w >= Hv) {
            for (uint64_t i = tid; i < ldw; i += kTeam) W[w * ldw + i] = 0;
            continue;
        }
        const uint64_t base = next_base;
        const uint32_t deg = next_deg;
        read_rows(w + step);
        const uint32_t inc = wave_incl_scan_u32(deg), first = inc - deg;
        const uint32_t P = (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1);
        const uint64_t delta = base - first;  // S position of entry f of this lane's row: delta + f
        // rows fill the lanes from 0 on, or of each half (b = 32)
        const uint32_t low = (uint32_t)__popc((uint32_t)__ballot(deg > 0));
        uint32_t z0 = 0, z1 = 0;
        for (uint64_t c0 = 0; c0 < ldw; c0 += cols) {
            const uint32_t cn = (uint32_t)min((uint64_t)cols, ldw - c0);
            if (P <= kPackFlat) {
                // kPackLoads entries per lane in flight before their ORs; a sample
                // of ~0u lies past every chunk
                for (uint32_t c = wv; c * kWave < P; c += G * kPackLoads) {
                    uint32_t v[kPackLoads], row[kPackLoads];
#pragma unroll
                    for (uint32_t u = 0; u < kPackLoads; ++u) {
                        const uint32_t f0 = (c + u * G) * kWave, f = f0 + lane;
                        v[u] = ~0u;
                        row[u] = 0;
                        if (f0 < P) {  // wave-uniform
                            const uint64_t m = starts[f0 / kWave];
                            uint32_t t = (uint32_t)__popcll(__ballot(deg > 0 && first < f0)) + lanes_before(m) +
                                         (uint32_t)((m >> lane) & 1) - 1;
                            t += t >= low ? kWave / 2 - low : 0;
                            const uint64_t at = __shfl(delta, (int)t, kWave) + f;
                            row[u] = t;
                            if (f < P) v[u] = S[at];
                        }
                    }
#pragma unroll
                    for (uint32_t u = 0; u < kPackLoads; ++u)
                        if (v[u] >= c0 && v[u] < c0 + cn) atomicOr(&lw[v[u] - c0], 1ull << row[u]);
                }
            } else {
                // many entries: the lanes of a wave walk one row at a time
                for (uint32_t t = wv; t < kWave; t += G) {
                    const uint64_t rb = __shfl(base, (int)t, kWave);
                    const uint32_t dg = __shfl(deg, (int)t, kWave);
                    for (uint32_t e0 = lane; e0 < dg; e0 += kWave * kPackLoads) {
                        uint32_t v[kPackLoads];
#pragma unroll
                        for (uint32_t u = 0; u < kPackLoads; ++u) {
                            const uint32_t e = e0 + u * kWave;
                            v[u] = e < dg ? S[rb + e] : ~0u;
                        }
#pragma unroll
                        for (uint32_t u = 0; u < kPackLoads; ++u)
                            if (v[u] >= c0 && v[u] < c0 + cn) atomicOr(&lw[v[u] - c0], 1ull << t);
                    }
                }
            }
            sync();
            if (wv == 0 && c0 + cn == ldw) {  // the bitmap is the next row's from here on
                if (deg && P <= kPackFlat) starts32[first >> 5] = 0;
                mark_next();
            }
            // a wave's 128 words of a round are all below cn or all past it
            for (uint32_t i = 2 * tid; i < cn; i += 2 * kTeam) {
                const ulonglong2 v = *reinterpret_cast<const ulonglong2 *>(lw + i);
                *reinterpret_cast<ulonglong2 *>(lw + i) = ulonglong2{0, 0};
                *reinterpret_cast<ulonglong2 *>(W + w * ldw + c0 + i) = v;
                if (wb == 64) {
                    z0 += (uint32_t)(__popcll(__ballot(v.x != 0)) + __popcll(__ballot(v.y != 0)));
                } else {
                    z0 += (uint32_t)(__popcll(__ballot((uint32_t)v.x != 0)) + __popcll(__ballot((uint32_t)v.y != 0)));
                    z1 += (uint32_t)(__popcll(__ballot((v.x >> 32) != 0)) + __popcll(__ballot((v.y >> 32) != 0)));
                }
            }
            if (G > 1 && c0 + cn == ldw && lane == 0) {
                if (z0) atomicAdd(&zsh[0], z0);
                if (z1) atomicAdd(&zsh[1], z1);
            }
            sync();
        }
        if (tid == 0) {
            unsigned long long a = z0, b = z1;
            if (G > 1) {  // (added to again only after the next row's first barrier)
                a = zsh[0];
                b = zsh[1];
                zsh[0] = zsh[1] = 0;
            }
            nnz_acc += a + b;
            f_acc += a * (a + 1) / 2 + b * (b + 1) / 2;
        }
    }
    if (tid == 0 && nnz_acc) {
        const uint32_t slot = (blockIdx.x * kTeams + team) % slots;
        atomicAdd(&word_slots[slot], nnz_acc);
        atomicAdd(&word_slots[slots + slot], f_acc);
    }
}

// Row lists: CSR of the rows of degree 2..dmin-1.  Lrow maps list row j to
// its shared row; null when every shared row is a list row (j itself), here
// and in k_list_wave_pairs and k_pair_emit.
__global__ void k_list_deg(const uint64_t *Lrow, const uint32_t *row_deg, uint64_t QL, uint64_t *deg) {
    for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < QL; j += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t r = Lrow ? Lrow[j] : j;
        deg[j] = row_deg[r];
    }
}

__global__ void k_list_gather(const uint64_t *Lrow, const uint64_t *row_ptr, const uint32_t *row_deg, const uint32_t *S,
                              const uint64_t *lptr, uint64_t QL, uint32_t *lsmp) {
    for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < QL; j += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t r = Lrow ? Lrow[j] : j;
        const uint64_t a0 = row_ptr[r], d = row_deg[r], o = lptr[j];
        for (uint64_t k = 0; k < d; ++k) lsmp[o + k] = S[a0 + k];
    }
}

// Row lists as pairs for the Gram step: every pair (a, b), a < b, of every
// list row as the 32-bit word (a << 16) | b, then sorted by a (single-pass
// scatters over the bits of a), so that the Gram step reads each sample's
// pairs as one contiguous run (the row-by-row form of B = A^T A over the row
// lists).  wnp[g] = pairs of list rows [64g, 64g + 64): one wave per group,
// which is also one wave's share of the emission below.
__global__ void k_list_wave_pairs(const uint64_t *Lrow, const uint32_t *row_deg, uint64_t QL, uint64_t *wnp,
                                  const uint64_t *__restrict__ dsz) {
    if (plan_aborted(dsz)) return;
    // planned: QL is the capacity; groups past the actual rows count nothing
    const uint64_t nw = (QL + kWave - 1) / kWave;
    if (dsz) QL = dsz[PZ_QL];
    if (!list_map_used(Lrow, dsz)) Lrow = nullptr;
    const uint32_t lane = lane_id();
    for (uint64_t g = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave; g < nw;
         g += ((uint64_t)gridDim.x * blockDim.x) / kWave) {
        const uint64_t j = g * kWave + lane;
        uint64_t np = 0;
        if (j < QL) {
            const uint64_t r = Lrow ? Lrow[j] : j;
            const uint64_t d = row_deg[r];
            np = d * (d - 1) / 2;
        }
        const uint64_t inc = wave_incl_scan(np);
        if (lane == kWave - 1) wnp[g] = inc;
    }
}

// A wave takes 64 consecutive rows; their pairs fill one contiguous stretch of
// the output (the rows' pair counts scanned), row by row, each row's pairs in
// order.  It works through them a few rows at a time, as many as fit its LDS
// (kEmitIn entries, kEmitStage pairs): the entries are read into LDS, the pairs
// formed there and copied out with 16-byte stores.
//
// Forming them is what bounds it, not the 4 bytes per pair, so a lane forms four
// consecutive output words whatever the rows' lengths.  The pairs of one smaller
// entry are a run of words; each run's start is marked with its position and
// entry, and a running maximum over the marks (in the lane, then over the wave)
// tells every word its run, hence both of its entries.  Marks of earlier parts
// need no clearing: a mark's top bits number its part, and the first word of
// every part is marked.  Only the marking goes row by row, a lane for each.
// 1.68 G pairs of 33.5 M rows of about 10: 6.35 ms with a lane per output word
// that solved for its row and pair (some 140 instructions), 2.7 ms now; 1.85 G of
// 196 M rows of 2 to 20: 5.28 ms with a lane per row where the pairs fitted,
// 3.9 ms.
//
// A row too long for the stage is written straight to memory, lanes along the
// pairs of entries k and d - 1 - k.  Per-block LDS totals of the sort digits
// (digit q = bits [16 + width*q, 16 + width*(q+1)) of the word) are counted by
// the lane that has the entry.
// With few rows (gridDim.y > 1) that many waves take the same 64 rows and deal
// these parts among them: 1231 rows of degree 60 to 67 (2.6 M pairs) fill 20
// waves, 1.79 ms, and 0.075 ms shared.
// (both: sizes from 512 and 256 to 2048 and 512 measured on the two above)
constexpr uint32_t kEmitStage = 896;  // pairs per wave, at a time
constexpr uint32_t kEmitIn = 384;     // entries per wave, at a time
constexpr uint32_t kMarkEntry = 9, kMarkPart = 21;  // a mark: part << 21 | word << 9 | entry
constexpr uint32_t kMarkParts = (1u << (32 - kMarkPart)) - 1;
static_assert(kEmitIn <= 1u << kMarkEntry && kEmitStage + 3 < 1u << (kMarkPart - kMarkEntry), "marks");
constexpr uint32_t kPairPasses = 2;   // 16 sample bits, 8-bit digits

// Pairs of a row of d entries whose smaller entry comes before entry i.
__device__ __forceinline__ uint32_t pairs_before(uint32_t d, uint32_t i) { return i * (2 * d - i - 1) / 2; }

__global__ __launch_bounds__(256) void k_pair_emit(const uint64_t *__restrict__ Lrow,
                                                    const uint64_t *__restrict__ row_ptr,
                                                    const uint32_t *__restrict__ row_deg,
                                                    const uint32_t *__restrict__ ls, uint64_t QL,
                                                    const uint64_t *__restrict__ wpo,
                                                    uint32_t *__restrict__ pairs, uint32_t npass, uint32_t width,
                                                    unsigned long long *__restrict__ ghist,
                                                    const uint64_t *__restrict__ dsz) {
    constexpr uint32_t kWavesHere = 256 / kWave;
    __shared__ uint32_t gh[kPairPasses][256];
    __shared__ uint32_t entb[kWavesHere][kEmitIn];
    __shared__ __attribute__((aligned(16))) uint32_t markb[kWavesHere][kEmitStage + 4];
    if (plan_aborted(dsz)) return;
    if (dsz) QL = dsz[PZ_QL];
    if (!list_map_used(Lrow, dsz)) Lrow = nullptr;
    const uint32_t tid = threadIdx.x, lane = lane_id(), w = tid / kWave;
    const uint32_t dmask = (1u << width) - 1u;
#pragma unroll
    for (int k = 0; k < (int)kPairPasses; ++k) gh[k][tid] = 0;
    __syncthreads();
    uint32_t *ent = entb[w], *mark = markb[w];
    uint32_t marked = kMarkParts;  // parts marked since the marks were cleared (at first: not cleared yet)
    const auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    const auto count = [&](uint32_t a, uint32_t c) {
        for (uint32_t q = 0; q < npass; ++q) atomicAdd(&gh[q][(a >> (width * q)) & dmask], c);
    };
    for (uint64_t r0 = ((uint64_t)blockIdx.x * kWavesHere + w) * kWave; r0 < QL; r0 += (uint64_t)gridDim.x * 256) {
        const uint64_t r = r0 + lane;
        uint64_t e0 = 0;
        uint32_t deg = 0;
        if (r < QL) {
            const uint64_t rr = Lrow ? Lrow[r] : r;
            e0 = row_ptr[rr];
            deg = row_deg[rr];
        }
        // the wave's first pair (wpo: scan of the 64-row groups' pair counts); a
        // list row has at most n <= kSampleMajorMaxN entries, so 64 rows hold
        // fewer than 2^32 pairs
        const uint64_t base = wpo[r0 / kWave];
        const uint32_t np = deg > 1 ? deg * (deg - 1) / 2 : 0;
        const uint32_t pin = wave_incl_scan_u32(np), ein = wave_incl_scan_u32(deg);
        uint32_t b = 0, pb = 0, eb = 0, part = 0;  // rows, pairs, entries and parts before the part in hand
        while (b < kWave) {
            const uint64_t fit = __ballot(lane >= b && pin - pb <= kEmitStage && ein - eb <= kEmitIn);
            const uint32_t c = (uint32_t)__popcll(fit);
            if (c == 0) {  // row b alone, straight to memory
                const uint32_t d = __shfl(deg, (int)b, kWave);
                const uint32_t *s = ls + __shfl(e0, (int)b, kWave);
                uint32_t *out = pairs + base + pb;
                for (uint32_t k = (blockIdx.y + part) % gridDim.y; 2 * k < d; k += gridDim.y) {
                    const uint32_t m = d - 1 - k, len = k == m ? m : d - 1;
                    const uint32_t a1 = s[k], a2 = s[m];
                    if (lane < 2 && (lane == 0 || k != m)) count(lane ? a2 : a1, lane ? k : m);
                    uint32_t *o1 = out + pairs_before(d, k), *o2 = out + pairs_before(d, m);
                    for (uint32_t u = lane; u < len; u += kWave) {
                        const uint32_t v = s[u + 1 + (u < m ? k : 0)];
                        if (u < m) o1[u] = a1 << 16 | v;
                        else o2[u - m] = a2 << 16 | v;
                    }
                }
            } else if (part % gridDim.y == blockIdx.y) {
                const uint32_t end = b + c;
                // the entries: one span of the sample array (the rows ascend), or,
                // where rows of other kinds or the ends of ranges leave gaps that
                // do not fit, row after row
                const uint64_t span0 = __shfl(e0, (int)b, kWave);
                const uint32_t lastrow = (uint32_t)(min(r0 + end, QL) - 1 - r0);
                const uint64_t span = __shfl(e0 + deg, (int)lastrow, kWave) - span0;
                const bool whole = span <= kEmitIn;  // wave-uniform
                const bool mine = lane >= b && lane < end && r < QL;
                uint32_t at = whole ? (uint32_t)(e0 - span0) : ein - deg - eb;
                if (whole) {
                    for (uint32_t k = lane; k < (uint32_t)span; k += kWave) ent[k] = ls[span0 + k];
                } else if (mine) {
                    for (uint32_t k = 0; k < deg; k += 4) {
                        uint32_t v[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) v[u] = k + u < deg ? ls[e0 + k + u] : 0u;
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            if (k + u < deg) ent[at + k + u] = v[u];
                    }
                }
                if (marked == kMarkParts) {
                    for (uint32_t k = lane; k < kEmitStage + 4; k += kWave) mark[k] = 0;
                    marked = 0;
                }
                wave_sync();
                const uint32_t gen = ++marked << kMarkPart;
                // words are numbered from the 16-byte boundary before the first
                const uint64_t first = base + pb;
                const uint32_t shift = (uint32_t)first & 3u;
                if (mine) {
                    uint32_t o = pin - np - pb + shift;
                    for (uint32_t i = 0; i + 1 < deg; ++i) {
                        mark[o] = gen | o << kMarkEntry | (at + i);
                        count(ent[at + i], deg - 1 - i);
                        o += deg - 1 - i;
                    }
                }
                wave_sync();
                const uint32_t stop = shift + __shfl(pin, (int)end - 1, kWave) - pb;
                uint32_t *out = pairs + (first - shift);
                uint32_t carry = 0;
                for (uint32_t o0 = 0; o0 < stop; o0 += 4 * kWave) {
                    const uint32_t o = o0 + 4 * lane;
                    uint4 m = o < stop ? *reinterpret_cast<const uint4 *>(mark + o) : uint4{0, 0, 0, 0};
                    m.y = max(m.x, m.y);
                    m.z = max(m.y, m.z);
                    m.w = max(m.z, m.w);
                    const uint32_t all = wave_incl_max(m.w);
                    const uint32_t before = max(carry, wave_shift_up(all));
                    carry = max(carry, (uint32_t)__builtin_amdgcn_readlane((int)all, kWave - 1));
                    const auto word = [&](uint32_t v, uint32_t at_o) {
                        v = max(v, before);
                        const uint32_t e = v & ((1u << kMarkEntry) - 1u);
                        const uint32_t start = (v >> kMarkEntry) & ((1u << (kMarkPart - kMarkEntry)) - 1u);
                        return ent[e] << 16 | ent[min(e + 1 + (at_o - start), kEmitIn - 1)];
                    };
                    const uint4 v{word(m.x, o), word(m.y, o + 1), word(m.z, o + 2), word(m.w, o + 3)};
                    if (o >= shift && o + 4 <= stop) {
                        *reinterpret_cast<uint4 *>(out + o) = v;
                    } else {
                        if (o >= shift && o < stop) out[o] = v.x;
                        if (o + 1 >= shift && o + 1 < stop) out[o + 1] = v.y;
                        if (o + 2 >= shift && o + 2 < stop) out[o + 2] = v.z;
                        if (o + 3 >= shift && o + 3 < stop) out[o + 3] = v.w;
                    }
                }
                wave_sync();
            }
            const uint32_t done = c ? c : 1;
            b += done;
            ++part;
            pb = __shfl(pin, (int)b - 1, kWave);
            eb = __shfl(ein, (int)b - 1, kWave);
        }
    }
    __syncthreads();
    unsigned long long *g = ghist + (uint64_t)(blockIdx.x % kGhistReplicas) * kMaxPasses * 256;
    for (uint32_t q = 0; q < npass; ++q)
        if (gh[q][tid]) atomicAdd(&g[q * 256 + tid], (unsigned long long)gh[q][tid]);
}

// Query index: bucket[b] = first distinct key whose ID has top bits >= b.
__global__ void k_bucket(const uint64_t *D, uint64_t ND, uint32_t sbits, uint32_t shift, uint64_t nbk,
                         uint64_t *bucket) {
    for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t <= ND; t += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t bk = t < ND ? ((D[t] >> sbits) >> shift) : nbk;
        const int64_t prev = t == 0 ? -1 : (int64_t)((D[t - 1] >> sbits) >> shift);
        for (int64_t b = prev + 1; b <= (int64_t)bk; ++b) bucket[b] = t;
    }
}

// --- planned encode: sizes after each scan, checked against the capacities.
// One thread each; a size above its capacity sets PZ_ABORT (every later
// kernel of the encode then returns at once) and err bit 32.  (k_plan_begin:
// the other threads clear the counters.)
__global__ void k_plan_begin(const uint64_t *off, int32_t n, uint64_t Ncap, uint64_t *dsz, uint32_t *err, Clear c) {
    for (int k = 0; k < Clear::kMax; ++k)
        for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < c.words[k];
             i += (uint64_t)gridDim.x * blockDim.x)
            c.p[k][i] = 0;
    if (blockIdx.x || threadIdx.x) return;
    uint64_t N = n > 0 ? off[n] : 0;
    for (int k = 0; k < PZ_COUNT; ++k) dsz[k] = 0;
    err[0] = 0;
    if (N > Ncap) {  // nothing is encoded (the sort sees no keys either)
        dsz[PZ_ABORT] = 1;
        dsz[PZ_OVER] = PZ_N + 1;
        dsz[PZ_OVER_VALUE] = N;
        err[0] = 32u;
        N = 0;
    }
    dsz[PZ_N] = N;
}

__global__ void k_plan_rows(const uint64_t *offR, const uint64_t *offS, uint64_t nlc_cap, uint64_t Rcap,
                            uint64_t *rptr, uint64_t *dsz, uint32_t *err) {
    if (dsz[PZ_ABORT]) return;
    const uint64_t R = offR[nlc_cap], NS = offS[nlc_cap];
    if (R > Rcap) {
        dsz[PZ_ABORT] = 1;
        dsz[PZ_OVER] = PZ_R + 1;
        dsz[PZ_OVER_VALUE] = R;
        atomicOr(err, 32u);
        return;
    }
    dsz[PZ_R] = R;
    rptr[R] = NS;
}

__global__ void k_plan_split(const uint64_t *toff, uint64_t tile_cap, uint64_t QDcap, uint64_t QLcap, uint64_t *dsz,
                             uint32_t *err) {
    if (dsz[PZ_ABORT]) return;
    const uint64_t QD = toff[tile_cap], QL = dsz[PZ_R] - QD;
    if (QD > QDcap || QL > QLcap) {
        dsz[PZ_ABORT] = 1;
        dsz[PZ_OVER] = QD > QDcap ? PZ_QD + 1 : PZ_QL + 1;
        dsz[PZ_OVER_VALUE] = QD > QDcap ? QD : QL;
        atomicOr(err, 32u);
        return;
    }
    dsz[PZ_QD] = QD;
    dsz[PZ_QL] = QL;
}

__global__ void k_plan_batches(const uint64_t *bpos, uint64_t QDcap, uint64_t *bq, uint64_t *dsz) {
    if (dsz[PZ_ABORT]) return;
    const uint64_t nb = bpos[QDcap];  // the flags past QD are zero
    dsz[PZ_NB] = nb;
    bq[nb] = dsz[PZ_QD];
}

__global__ void k_plan_words(const uint64_t *wbase, uint64_t QDcap, uint32_t wb, uint64_t Hwcap, uint64_t Hcap,
                             uint64_t *dsz, uint32_t *err) {
    if (dsz[PZ_ABORT]) return;
    const uint64_t Hw = wbase[QDcap], H = wb == 64 ? Hw : (Hw + 1) / 2;
    if (Hw > Hwcap || H > Hcap) {
        dsz[PZ_ABORT] = 1;
        dsz[PZ_OVER] = PZ_HW + 1;
        dsz[PZ_OVER_VALUE] = Hw;
        atomicOr(err, 32u);
        return;
    }
    dsz[PZ_HW] = Hw;
    dsz[PZ_H] = H;
}

__global__ void k_plan_pairs(const uint64_t *npo, uint64_t gcap, uint64_t Pcap, uint64_t *dsz, uint32_t *err) {
    if (dsz[PZ_ABORT]) return;
    const uint64_t P = npo[gcap];
    if (P > Pcap) {
        dsz[PZ_ABORT] = 1;
        dsz[PZ_OVER] = PZ_P + 1;
        dsz[PZ_OVER_VALUE] = P;
        atomicOr(err, 32u);
        return;
    }
    dsz[PZ_P] = P;
}

// k_pack with a wave, 4 or 8 waves per row of W: a wave where the row is short
// and there are rows enough to fill the chip (16 waves per CU), 8 where its
// words leave room for few blocks per CU (16 measured the same).  Column chunks
// are of equal size (multiples of 128 words).
template <int G>
void launch_pack_waves(uint64_t H, uint32_t cols, hipStream_t s, uint64_t *W, uint64_t ldw, uint64_t Hw, uint32_t wb,
                       const uint64_t *wq0, const uint64_t *wq1, uint64_t QD, const uint64_t *Drow,
                       const uint64_t *row_ptr, const uint32_t *row_deg, const uint32_t *S, unsigned long long *word_slots,
                       uint32_t slots, const uint64_t *dsz) {
    constexpr uint32_t threads = std::max(256, G * kWave), teams = threads / (G * kWave);
    const size_t lds = teams * ((size_t)cols + kPackFlat / 64 + 1) * sizeof(uint64_t);
    const uint32_t blocks = (uint32_t)std::min<uint64_t>(div_up(H, (uint64_t)teams), G == 1 ? 2048 : 4096);
    if (lds > 65536)
        JAS_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&k_pack<G>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    k_pack<G><<<blocks, threads, lds, s>>>(W, ldw, H, Hw, wb, wq0, wq1, QD, Drow, row_ptr, row_deg, S, cols, word_slots,
                                           slots, dsz);
}

void launch_pack(uint64_t *W, uint64_t ldw, uint64_t H, uint64_t Hw, uint32_t wb, const uint64_t *wq0,
                 const uint64_t *wq1, uint64_t QD, const uint64_t *Drow, const uint64_t *row_ptr,
                 const uint32_t *row_deg, const uint32_t *S, unsigned long long *word_slots, uint32_t slots,
                 const uint64_t *dsz, hipStream_t s) {
    const uint64_t nchunk = div_up(ldw, (uint64_t)kPackCols);
    const uint32_t cols = (uint32_t)(div_up(div_up(ldw, nchunk), 128) * 128);
    const auto go = [&](auto launch) {
        launch(H, cols, s, W, ldw, Hw, wb, wq0, wq1, QD, Drow, row_ptr, row_deg, S, word_slots, slots, dsz);
    };
    if (ldw <= 1024 && H >= 4096) go(launch_pack_waves<1>);
    else if (ldw <= 1024) go(launch_pack_waves<4>);
    else go(launch_pack_waves<8>);
}

// Grid of k_pair_emit over QL list rows: a wave per 64 rows, and as many waves
// sharing the same rows as bring the chip to about 8192 waves.
dim3 pair_emit_grid(uint64_t QL) {
    const uint64_t waves = div_up(QL, (uint64_t)kWave);
    return dim3((uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(div_up(QL, 256), 8192)),
                (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(8192 / std::max<uint64_t>(waves, 1), 64)));
}

template <class F>
void launch_1d(uint64_t work, hipStream_t s, F f) {
    const uint64_t blocks = std::min<uint64_t>(std::max<uint64_t>(div_up(work, 256), 1), 65536);
    f((uint32_t)blocks, s);
}

uint64_t to_host_u64(const uint64_t *dptr, hipStream_t s) {
    uint64_t v = 0;
    read_back(ReadBack().add(dptr), &v, s);
    return v;
}

}  // namespace

void build_keys(const uint64_t *ids, const uint64_t *offsets, int32_t n, uint64_t N, uint32_t sbits, uint32_t U,
                const SortPlan &plan, uint64_t *keys, uint32_t *err, unsigned long long *ghist, hipStream_t s) {
    if (N == 0) return;
    const uint64_t hi_mask = U >= 64 ? 0 : ~((uint64_t(1) << U) - 1);
    const uint32_t chunk = key_chunk(N);
    const uint64_t blocks = div_up(N, (uint64_t)chunk);
    if (blocks > 0xFFFFFFFFull) fail(JAS_EUNSUPPORTED, "too many IDs");
    if (keys) {
        JAS_TIMED("build_keys", s);
        k_build_keys<<<(uint32_t)blocks, kNT, 0, s>>>(ids, offsets, n, N, sbits, hi_mask, keys, err, plan.npass,
                                                      U - plan.top_bits, plan.width, ghist, nullptr, chunk);
    } else {
        JAS_TIMED("count_digits", s);
        k_count_digits<<<(uint32_t)blocks, kNT, 0, s>>>(ids, N, hi_mask, err, plan.npass, U - plan.top_bits,
                                                        plan.width, ghist, nullptr, chunk);
    }
    check_launch("build keys");
}

namespace {
// The ranges k_local_cls finishes: their starts rs[0 .. nlc], the most keys of
// one (cap, one of the kernel's), and the flags of k_range_check (bit 8: no
// stride gives ranges that fit LDS; bit 16: their keys need 64 bits).
struct Ranges {
    uint64_t nlc = 0, stride = 0, err = 8;
    uint32_t cap = kLocalCapKeys;
    uint32_t sort_err = 0;
};
constexpr uint64_t kMinStride = kLocalStrides[sizeof(kLocalStrides) / sizeof(kLocalStrides[0]) - 1];

// Clears `clear` too, and reads sort_err (if given) along with its own flags:
// keys out of order only make it find ranges that nothing then uses.
Ranges find_ranges(const uint64_t *keys, uint64_t N, uint32_t bsh, uint32_t lowbits, uint32_t sbits,
                   DevBuf<uint64_t> &rs, DevBuf<uint64_t> &flags, Clear clear, const uint32_t *sort_err, hipStream_t s,
                   Budget *tb) {
    Ranges r;
    rs.alloc(div_up(N, kMinStride) + 1, s, tb, true, "range starts");
    flags.alloc(1, s, tb, true, "range error flag");
    uint32_t *err = reinterpret_cast<uint32_t *>(flags.p);
    // with every ID bit sorted globally the ranges need no LDS passes, and
    // longer ranges (fewer blocks) pay: 4096 is tried first
    const uint64_t strides[] = {kLocalWideStride, kLocalStrides[0], kLocalStrides[1]};
    for (const uint64_t stride : strides) {
        if (stride == kLocalWideStride && lowbits != 0) continue;
        r.nlc = div_up(N, stride);
        clear_words(clear.add(flags.p, 1), s);
        clear = Clear();
        {
            JAS_TIMED("range_starts", s);
            k_range_starts<<<(uint32_t)div_up(r.nlc + 1, 256 / kWave), 256, 0, s>>>(keys, N, bsh, stride, r.nlc, rs.p,
                                                                                     err, nullptr, r.cap);
            k_range_check<<<(uint32_t)std::min<uint64_t>(div_up(r.nlc, 256), 4096), 256, 0, s>>>(
                keys, rs.p, r.nlc, bsh, lowbits, sbits, err, nullptr, 0, r.cap);
        }
        check_launch("range starts");
        uint64_t got[2] = {0, 0};
        ReadBack rb;
        rb.add(flags.p);
        if (sort_err) rb.add(sort_err);
        read_back(rb, got, s);
        r.err = got[0];
        r.sort_err = (uint32_t)got[1];
        if (r.sort_err) break;
        if ((r.err & 8u) == 0) {
            r.cap = r.err & 128u ? kLocalCapKeys : kLocalShortCap;
            r.stride = stride;
            break;
        }
    }
    return r;
}
}  // namespace

uint64_t distinct_sorted(DevBuf<uint64_t> &keys, DevBuf<uint64_t> &alt, uint64_t N, uint32_t U, const SortPlan &plan,
                         hipStream_t s) {
    if (div_up(N, kMinStride) > 0xFFFFFFFFull || keys.n < N || alt.n < N) return ~0ull;
    const uint32_t lowbits = U - plan.top_bits;
    DevBuf<uint64_t> rs, flags;
    const Ranges rg = find_ranges(keys.p, N, lowbits, lowbits, 0, rs, flags, Clear(), nullptr, s, nullptr);
    if (rg.err & 8u) return ~0ull;
    DevBuf<unsigned long long> rows;
    DevBuf<uint32_t> cnt;
    DevBuf<uint64_t> off, zero, tmp;
    rows.alloc(kStatSlots, s, nullptr, true, "row counters");
    cnt.alloc(3 * rg.nlc, s, nullptr, true, "range counts");
    off.alloc(rg.nlc + 1, s, nullptr, true, "range offsets");
    zero.alloc(rg.nlc + 1, s, nullptr, true, "range offsets");
    tmp.alloc(scan_tmp_elems(rg.nlc), s, nullptr, true, "scan scratch");
    {
        // without sample bits no two distinct keys share an ID: no rows, no shared pairs
        JAS_TIMED(rg.err & 16u ? "local_cls_wide" : "local_cls", s);
        launch_local_cls((rg.err & 16u) != 0, rg.cap, (uint32_t)rg.nlc, s, keys.p, 0u, (uint64_t)0, lowbits, lowbits,
                         (const uint64_t *)rs.p, (uint32_t)rg.nlc, cnt.p, 1, (uint32_t *)nullptr, (uint64_t *)nullptr,
                         (uint64_t *)nullptr, (unsigned long long *)nullptr, rows.p, kStatSlots, (const uint64_t *)nullptr,
                         (uint64_t)0, reinterpret_cast<uint32_t *>(flags.p));
    }
    check_launch("local distinct");
    scan_excl_u32(cnt.p, off.p, rg.nlc, tmp.p, s);
    {
        JAS_TIMED("local_move", s);
        k_fill_u64<<<(uint32_t)std::min<uint64_t>(div_up(rg.nlc + 1, 256), 4096), 256, 0, s>>>(zero.p, rg.nlc + 1, 0);
        k_local_move<<<(uint32_t)std::min<uint64_t>(rg.nlc, 65536), 256, 0, s>>>(
            rs.p, rg.nlc, off.p, zero.p, zero.p, keys.p, nullptr, nullptr, alt.p, nullptr, nullptr, nullptr, nullptr, 0);
    }
    check_launch("local move");
    return to_host_u64(off.p + rg.nlc, s);
}

namespace {
// Scans of the three counts of len ranges or chunks: one launch or two, or, within
// a memory limit, one after another in a third of the scratch.
void scan_counts(const DevBuf<uint32_t> &cnt, uint64_t len, DevBuf<uint64_t> &offD, DevBuf<uint64_t> &offS,
                 DevBuf<uint64_t> &offR, DevBuf<uint64_t> &tmp, hipStream_t s, Budget *tb) {
    const bool limited = tb && tb->limit;
    tmp.alloc(scan_tmp_elems(len, limited ? 1 : kScanRows), s, tb, true, "scan scratch");
    uint64_t *const out[kScanRows] = {offD.p, offS.p, offR.p};
    if (!limited) return scan_excl_u32_rows(cnt.p, len, out, len, tmp.p, s);
    for (uint32_t y = 0; y < kScanRows; ++y) scan_excl_u32(cnt.p + y * len, out[y], len, tmp.p, s);
}
}  // namespace

void encode_sorted(jas_db *db, DevBuf<uint64_t> &keys, DevBuf<uint64_t> &alt, uint64_t N, const SortPlan &plan,
                   const uint64_t *offsets, const uint32_t *sort_err, hipStream_t s, Budget *tb) {
    const int32_t n = db->n;
    const uint32_t sbits = db->sbits;
    const uint64_t smask = sbits ? ((uint64_t(1) << sbits) - 1) : 0;
    const bool keep = db->flags & JAS_KEEP_IDS;
    const bool query_only = db->flags & JAS_QUERY_ONLY;  // no packed words or row lists

    DevBuf<unsigned long long> st;
    const uint32_t slots = stat_slots(N, tb && tb->limit);
    st.alloc(stat_words(slots), s, tb, true, "encode counters");
    Clear clear;  // by the first launch below
    clear.add(st.p, st.n);
    const auto check_sort = [](uint32_t e) {
        if (e & 1u) fail(JAS_EINVAL, "jas_encode: an ID is >= 2^universe_bits");
        if (e) fail(JAS_EDEVICE, "jas_encode: the radix sort's look-back waited too long (result discarded)");
    };
    // |X_i|, all checked against the limit by the kernels that write it
    db->card.alloc(std::max<int32_t>(n, 1), s, &db->budget, false, "card");
    const auto check_card = [&](bool over) {
        if (!over) return;
        std::vector<int64_t> hc((size_t)n);
        JAS_HIP(hipMemcpyAsync(hc.data(), db->card.p, sizeof(int64_t) * n, hipMemcpyDeviceToHost, s));
        JAS_HIP(hipStreamSynchronize(s));
        const uint64_t lim = card_limit();
        for (int32_t i = 0; i < n; ++i)
            if ((uint64_t)hc[i] >= lim)
                fail(JAS_EOVERFLOW, "sample " + std::to_string(i) + " has " + std::to_string(hc[i]) +
                                        " distinct IDs (limit " + std::to_string(lim - 1) + ")");
    };

    // Outputs of the classification: distinct keys (query index), shared
    // pairs S in row order, and per shared row its ID and first pair.  (The keys,
    // and the pair words below, are the call's until the db takes them: on an
    // error they go back to the cache in stream order, not as idle.)
    uint64_t NDk = 0, NS = 0, R = 0;
    DevBuf<uint64_t> Dk, rid_own, rptr_own;
    DevBuf<uint32_t> rdeg_own;
    DevBuf<uint32_t> S_own;
    uint32_t *Sp = nullptr;
    uint64_t *ridp = nullptr, *rptrp = nullptr;
    uint32_t *rdegp = nullptr;
    bool done = N == 0;
    if (done) clear_words(clear.add(db->card.p, std::max<int32_t>(n, 1)), s);
    bool checked = done;  // sort_err

    // --- classify each range of whole buckets in LDS ------------------------
    if (!done && div_up(N, kMinStride) <= 0xFFFFFFFFull && alt.n >= N + 2) {
        const uint32_t lowbits = db->U - plan.top_bits;
        const uint32_t bsh = sbits + lowbits;
        DevBuf<uint64_t> rs, flags;
        DevBuf<unsigned long long> dupc;  // repeat counts per sample
        dupc.alloc(std::max<int32_t>(n, 1), s, tb, true, "repeat counts");
        clear.add(dupc.p, std::max<int32_t>(n, 1));
        const Ranges rg = find_ranges(keys.p, N, bsh, lowbits, sbits, rs, flags, clear, sort_err, s, tb);
        check_sort(rg.sort_err);
        checked = true;
        clear = Clear();
        uint32_t *errL = reinterpret_cast<uint32_t *>(flags.p);
        const uint64_t nlc = rg.nlc;
        const uint32_t cap = rg.cap;
        uint64_t herr = rg.err;
        db->trace.stride = rg.stride;
        db->trace.lcap = cap;
        if ((herr & 8u) == 0) {
            DevBuf<uint32_t> cnt;
            DevBuf<uint64_t> rid_g, offD, offS, offR, stmp;
            cnt.alloc(3 * nlc, s, tb, true, "range counts");
            rid_g.alloc(N / 2 + 1, s, tb, true, "row ids (by range)");
            // shared pairs at the range starts in the first half of the free sort
            // buffer, row pointers (relative to the range) after it
            uint32_t *Sg = reinterpret_cast<uint32_t *>(alt.p);
            uint64_t *rptr_g = alt.p + div_up(N, 2);
            {
                JAS_TIMED(herr & 16u ? "local_cls_wide" : "local_cls", s);
                launch_local_cls((herr & 16u) != 0, cap, (uint32_t)nlc, s, keys.p, sbits, smask, bsh, lowbits,
                                 (const uint64_t *)rs.p, (uint32_t)nlc, cnt.p, keep ? 1 : 0, Sg, rid_g.p, rptr_g,
                                 dupc.p, st.p + stat_rows(slots), slots, (const uint64_t *)nullptr, (uint64_t)0, errL);
            }
            check_launch("local classify");
            if (n > 0) {
                JAS_TIMED("card", s);
                k_card_from_dups<<<(uint32_t)std::min<uint64_t>(div_up(n, 256), 1024), 256, 0, s>>>(
                    offsets, dupc.p, n, db->card.p, (int64_t)card_limit(), errL);
            }
            check_launch("column sums");
            offD.alloc(nlc + 1, s, tb, true, "range offsets");
            offS.alloc(nlc + 1, s, tb, true, "range offsets");
            offR.alloc(nlc + 1, s, tb, true, "range offsets");
            scan_counts(cnt, nlc, offD, offS, offR, stmp, s, tb);
            uint64_t t3[4];
            read_back(ReadBack().add(offD.p + nlc).add(offS.p + nlc).add(offR.p + nlc).add(flags.p), t3, s);
            herr = t3[3];
            if (herr & 8u) fail(JAS_EDEVICE, "local classify: a range exceeds the kernel's capacity");
            check_card((herr & 64u) != 0);
            NDk = t3[0];
            NS = t3[1];
            R = t3[2];
            cnt.release();
            stmp.release();
            dupc.release();
            flags.release();
            if (!keep) keys.release();
            db->trace.local = true;
            db->trace.wide = (herr & 16u) != 0;
            db->trace.nlc = nlc;
            if (keep) Dk.alloc(NDk, s, &db->budget, true, "query index keys");
            rid_own.alloc(R, s, tb, true, "row ids");
            rptr_own.alloc(R + 1, s, tb, true, "row pointers");
            rdeg_own.alloc(R + 1, s, tb, true, "row degrees");
            Sp = Sg;  // the shared pairs stay in the ranges' stretches
            ridp = rid_own.p;
            rptrp = rptr_own.p;
            rdegp = rdeg_own.p;
            {
                JAS_TIMED("local_move", s);
                k_local_move<<<(uint32_t)std::min<uint64_t>(nlc, 65536), 256, 0, s>>>(
                    rs.p, nlc, offD.p, offS.p, offR.p, keys.p, rid_g.p, rptr_g, keep ? Dk.p : nullptr, ridp, rptrp,
                    rdegp, nullptr, 0);
            }
            check_launch("local move");
            keys.release();
            done = true;
        }
    }

    // --- otherwise: sort every ID bit, classify with neighbours in global memory
    if (!done) {
        JAS_HOST_TIMED("classify_fallback");
        if (!checked) {
            uint64_t e = 0;
            read_back(ReadBack().add(sort_err), &e, s);
            check_sort((uint32_t)e);
        }
        clear_words(clear.add(db->card.p, std::max<int32_t>(n, 1)), s);
        {
            RadixWork rw;
            radix_sort_u64(keys, alt, N, sbits, sbits + db->U, rw, s, tb);
        }
        const uint64_t *K = keys.p;
        const uint64_t nch = div_up(N, kChunk);
        DevBuf<uint32_t> cnt;
        DevBuf<uint64_t> offD, offS, offR, stmp;
        cnt.alloc(3 * nch, s, tb, true, "classify counts");
        const int lds_hist = n <= kHistMax;
        const size_t shmem = lds_hist ? (size_t)n * sizeof(uint32_t) : 0;
        {
            JAS_TIMED("cls_count", s);
            k_cls_count<<<(uint32_t)nch, kNT, shmem, s>>>(K, N, sbits, smask, n, lds_hist, cnt.p, cnt.p + nch,
                                                          cnt.p + 2 * nch,
                                                          reinterpret_cast<unsigned long long *>(db->card.p), st.p);
        }
        check_launch("classify count");
        offD.alloc(nch + 1, s, tb, true, "classify offsets");
        offS.alloc(nch + 1, s, tb, true, "classify offsets");
        offR.alloc(nch + 1, s, tb, true, "classify offsets");
        scan_counts(cnt, nch, offD, offS, offR, stmp, s, tb);
        uint64_t t3[3];
        read_back(ReadBack().add(offD.p + nch).add(offS.p + nch).add(offR.p + nch), t3, s);
        check_card(true);  // (looks at every sum)
        NDk = t3[0];
        NS = t3[1];
        R = t3[2];
        if (keep) Dk.alloc(NDk, s, &db->budget, true, "query index keys");
        S_own.alloc(NS, s, tb, true, "shared pairs");
        rid_own.alloc(R, s, tb, true, "row ids");
        rptr_own.alloc(R + 1, s, tb, true, "row pointers");
        Sp = S_own.p;
        ridp = rid_own.p;
        rptrp = rptr_own.p;
        {
            JAS_TIMED("cls_write", s);
            k_cls_write<<<(uint32_t)nch, kNT, 0, s>>>(K, N, sbits, smask, offD.p, offS.p, offR.p,
                                                      keep ? Dk.p : nullptr, Sp, ridp, rptrp);
        }
        check_launch("classify write");
    }
    if (!rdegp) {  // the global classification wrote the rows contiguously
        if (N > 0) {
            JAS_TIMED("fill_u64", s);
            k_fill_u64<<<1, 1, 0, s>>>(rptrp + R, 1, NS);
        }
        check_launch("fill");
        rdeg_own.alloc(R + 1, s, tb, true, "row degrees");
        rdegp = rdeg_own.p;
        launch_1d(std::max<uint64_t>(R, 1), s, [&](uint32_t b, hipStream_t st_) {
            JAS_TIMED("row_deg", st_);
            k_row_deg<<<b, 256, 0, st_>>>(rptrp, R, rdegp);
        });
        check_launch("row degrees");
    }

    // --- split rows by degree ------------------------------------------------
    uint64_t QD = 0, QL = 0, P = 0, list_pairs = 0;
    bool sized = false;  // QD and P come from the degree histogram, not from the device
    DevBuf<uint64_t> Drow, Lrow;
    if (R > 0 && !query_only && db->dmin == 0) {
        // choose the degree threshold from the row degree histogram
        JAS_HOST_TIMED("choose_dmin");
        const uint32_t nb = (uint32_t)n + 2;
        DevBuf<unsigned long long> hist;
        hist.alloc(nb, s, tb, true, "degree histogram");
        clear_words(Clear().add(hist.p, nb), s);
        const int lds = nb <= 16384;
        const uint32_t blocks = (uint32_t)std::min<uint64_t>(div_up(R, 256), 2048);
        {
            JAS_TIMED("deg_hist", s);
            k_deg_hist<<<blocks, kNT, lds ? nb * sizeof(uint32_t) : 0, s>>>(rdegp, R, nb, lds, hist.p);
        }
        check_launch("degree histogram");
        std::vector<uint64_t> hh(nb);
        JAS_HIP(hipMemcpyAsync(hh.data(), hist.p, nb * sizeof(uint64_t), hipMemcpyDeviceToHost, s));
        JAS_HIP(hipStreamSynchronize(s));
        size_t free_b = 0, total_b = 0;
        if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) {
            (void)hipGetLastError();
            free_b = 0;
        }
        uint64_t cap = free_b ? (uint64_t)free_b / 2 : ~0ull;
        if (tb->limit) cap = std::min<uint64_t>(cap, tb->limit / 2);
        const uint32_t bb = db->batch_bits, U = db->U;
        const uint64_t nbatches = (U - bb >= 63) ? ~0ull : (uint64_t(1) << (U - bb));
        db->dmin = choose_dense_min_degree(hh, (uint32_t)n, nbatches, cap);
        for (uint64_t d = 0; d < nb; ++d) {
            if (d >= db->dmin) QD += hh[d];
            else if (d > 1) P += hh[d] * (d * (d - 1) / 2);
        }
        QL = R - QD;
        list_pairs = P;
        sized = true;
    }
    db->stats.dense_min_degree = db->dmin;
    if (R > 0 && !query_only && !(sized && (QD == 0 || QL == 0))) {
        const uint64_t nt = div_up(R, kSplitTile);
        if (nt > 0xFFFFFFFFull) fail(JAS_EUNSUPPORTED, "too many rows");
        DevBuf<uint32_t> tcnt;
        DevBuf<uint64_t> toff, tmp;
        tcnt.alloc(nt, s, tb, true, "row tile counts");
        toff.alloc(nt + 1, s, tb, true, "row tile offsets");
        tmp.alloc(scan_tmp_elems(nt), s, tb, true, "scan scratch");
        {
            JAS_TIMED("row_count", s);
            k_row_count<<<(uint32_t)nt, kNT, 0, s>>>(rdegp, R, db->dmin, tcnt.p,
                                                      st.p + stat_lists(slots), slots, nullptr);
        }
        check_launch("row count");
        scan_excl_u32(tcnt.p, toff.p, nt, tmp.p, s);
        if (!sized) {
            QD = to_host_u64(toff.p + nt, s);
            QL = R - QD;
        }
        // when every shared row is of one form the split is the identity: the
        // kernels take a null Drow / Lrow as row q = q
        if (QD > 0 && QL > 0) {
            Drow.alloc(QD, s, tb, true, "packed rows");
            Lrow.alloc(QL, s, tb, true, "list rows");
            {
                JAS_TIMED("row_split", s);
                k_row_split<<<(uint32_t)nt, kNT, 0, s>>>(rdegp, R, db->dmin, toff.p, Drow.p, Lrow.p, nullptr);
            }
            check_launch("row split");
        }
    }

    // only the batches of packed rows are told apart by the rows' IDs
    if (QD == 0 || db->batch_bits >= db->U) rid_own.release();

    // --- row lists, first part -------------------------------------------------
    // Up to kSampleMajorMaxN samples: the rows' pairs, sorted by their smaller
    // sample, straight from the shared pairs.  Otherwise (or if that sort
    // cannot run) the rows as a CSR of samples, summed pair by pair.  The
    // pairs are emitted and sorted on a side stream while the packed rows are
    // packed on s (the two read the same rows and write different arrays); s
    // waits for the side stream before anything of the pair path is freed or
    // read.
    db->n_list = QL;
    bool pairs_done = false;
    const bool pair_form = QL > 0 && n <= kSampleMajorMaxN;
    DevBuf<uint64_t> npo;
    DevBuf<uint32_t> pk, palt, perr;
    DevBuf<unsigned long long> pgh;
    uint32_t psb = 0, pwidth = 0;
    hipStream_t s2 = nullptr;
    StreamJoin join;  // after the buffers: on an error s waits for s2 before they are freed
    if (pair_form) {
        // pairs per group of 64 list rows (one wave of the emission), scanned
        const uint64_t nw = div_up(QL, (uint64_t)kWave);
        DevBuf<uint64_t> np, tmp2;
        np.alloc(nw, s, tb, true, "row group pair counts");
        launch_1d(QL, s, [&](uint32_t b, hipStream_t st_) {
            {
                JAS_TIMED("list_npairs", st_);
                k_list_wave_pairs<<<b, 256, 0, st_>>>(Lrow.p, rdegp, QL, np.p, nullptr);
            }
        });
        check_launch("row pair counts");
        npo.alloc(nw + 1, s, tb, true, "row group pair offsets");
        tmp2.alloc(scan_tmp_elems(nw), s, tb, true, "scan scratch");
        scan_excl_u64(np.p, npo.p, nw, tmp2.p, s);
        if (!sized) P = to_host_u64(npo.p + nw, s);
        np.release();
        tmp2.release();
        psb = std::max<uint32_t>(1, ceil_log2_u64((uint64_t)n));
        const uint32_t npass = (psb + 7) / 8;
        pwidth = (psb + npass - 1) / npass;
        if (npass > kPairPasses) fail(JAS_EUNSUPPORTED, "row-list pairs: too many sample bits");
        pk.alloc(P + 2, s, &db->budget, true, "row-list pairs");
        palt.alloc(P + 2, s, tb, true, "row-list pairs (second buffer)");
        pgh.alloc(digit_words(npass, pwidth), s, tb, true, "pair digit totals");
        perr.alloc(2, s, tb, true, "pair sort flag");
        s2 = side_stream();
        stream_after(s2, s);  // everything the pair path reads is on s so far
        join.waiter = s;
        join.on = s2;
        join.armed = true;
        clear_words(Clear().add(pgh.p, pgh.n).add(perr.p, 1), s2);
        {
            JAS_TIMED("pair_emit", s2);
            k_pair_emit<<<pair_emit_grid(QL), 256, 0, s2>>>(
                Lrow.p, rptrp, rdegp, Sp, QL, npo.p, pk.p, npass, pwidth, pgh.p, nullptr);
        }
        check_launch("pair emit");
    }

    // --- packed rows: batches, word rows, pack -------------------------------
    const uint64_t ldw = div_up((uint64_t)std::max<int32_t>(n, 1), 128) * 128;
    const uint32_t wb = db->word_bits;
    uint64_t nb = 0, H = 0, Hw = 0;  // rows of W (64-bit), word rows of wb bits
    if (QD > 0) {
        DevBuf<uint32_t> bs;
        DevBuf<uint64_t> bpos, bq, nw, wbase, tmp, wq0, wq1;
        if (db->batch_bits >= db->U) {
            // a single batch: its word rows need no table (six launches and two
            // waits fewer, 0.1 ms of a small call)
            nb = 1;
            Hw = div_up(QD, (uint64_t)wb);
        } else {
            bs.alloc(QD, s, tb, true, "batch flags");
            const uint32_t bbits = db->batch_bits;
            launch_1d(QD, s, [&](uint32_t b, hipStream_t st_) {
                {
                    JAS_TIMED("batch_flag", st_);
                    k_batch_flag<<<b, 256, 0, st_>>>(Drow.p, ridp, QD, bbits, bs.p, nullptr);
                }
            });
            check_launch("batch flags");
            bpos.alloc(QD + 1, s, tb, true, "batch scan");
            tmp.alloc(scan_tmp_elems(QD), s, tb, true, "scan scratch");
            scan_excl_u32(bs.p, bpos.p, QD, tmp.p, s);
            nb = to_host_u64(bpos.p + QD, s);
            bq.alloc(nb + 1, s, tb, true, "batch starts");
            launch_1d(QD, s, [&](uint32_t b, hipStream_t st_) { { JAS_TIMED("batch_start", st_); k_batch_start<<<b, 256, 0, st_>>>(bs.p, bpos.p, QD, bq.p, nullptr); } });
            {
                JAS_TIMED("fill_u64", s);
                k_fill_u64<<<1, 1, 0, s>>>(bq.p + nb, 1, QD);
            }
            check_launch("batch starts");
            nw.alloc(nb, s, tb, true, "batch words");
            launch_1d(nb, s, [&](uint32_t b, hipStream_t st_) { { JAS_TIMED("batch_words", st_); k_batch_words<<<b, 256, 0, st_>>>(bq.p, nb, wb, nw.p, nullptr); } });
            check_launch("batch words");
            wbase.alloc(nb + 1, s, tb, true, "word bases");
            tmp.release();
            tmp.alloc(scan_tmp_elems(nb), s, tb, true, "scan scratch");
            scan_excl_u64(nw.p, wbase.p, nb, tmp.p, s);
            Hw = to_host_u64(wbase.p + nb, s);
            wq0.alloc(Hw, s, tb, true, "word rows");
            wq1.alloc(Hw, s, tb, true, "word rows");
            launch_1d(QD, s, [&](uint32_t b, hipStream_t st_) {
                {
                    JAS_TIMED("word_rows", st_);
                    k_word_rows<<<b, 256, 0, st_>>>(QD, bpos.p, bq.p, wbase.p, wb, wq0.p, wq1.p, nullptr);
                }
            });
            check_launch("word rows");
            bs.release();
            bpos.release();
            bq.release();
            nw.release();
            wbase.release();
            tmp.release();
        }
        H = wb == 64 ? Hw : div_up(Hw, 2);
        db->W.alloc(H * ldw, s, &db->budget, false, "packed words");
        {
            JAS_TIMED("pack", s);
            launch_pack(db->W.p, ldw, H, Hw, wb, wq0.p, wq1.p, QD, Drow.p, rptrp, rdegp, Sp, st.p + stat_words_of(slots),
                        slots, nullptr, s);
        }
        check_launch("pack");
    }
    db->H = H;

    // --- row lists, second part: the pair sort (side stream), then s waits --
    uint64_t hst[kStatWords];
    bool have_st = false;  // hst holds the final counters
    if (pair_form) {
        const bool ok = radix_sort_onesweep_u32(pk, palt, P, 16, 16 + psb, pwidth, pgh.p, perr.p, s2, tb);
        JAS_HIP(hipStreamSynchronize(s2));
        stream_after(s, s2);
        join.armed = false;
        uint64_t got[1 + kStatWords];
        read_back(ReadBack().add(perr.p).add(st.p, (uint32_t)st.n), got, s);
        std::copy(got + 1, got + 1 + st.n, hst);
        have_st = true;
        if (ok && (uint32_t)got[0] == 0) {
            db->n_lpairs = P;
            db->pairs = std::move(pk);
            db->pairs.owned_by_db = true;
            pairs_done = true;
            db->trace.pairs = true;
            db->trace.P = P;
        }
    }
    if (QL > 0 && !pairs_done) {
        db->list_ptr.alloc(QL + 1, s, &db->budget, false, "row list pointers");
        DevBuf<uint64_t> deg, tmp;
        deg.alloc(QL, s, tb, true, "row list degrees");
        launch_1d(QL, s, [&](uint32_t b, hipStream_t st_) { { JAS_TIMED("list_deg", st_); k_list_deg<<<b, 256, 0, st_>>>(Lrow.p, rdegp, QL, deg.p); } });
        check_launch("list degrees");
        tmp.alloc(scan_tmp_elems(QL), s, tb, true, "scan scratch");
        scan_excl_u64(deg.p, db->list_ptr.p, QL, tmp.p, s);
        db->list_nnz = to_host_u64(db->list_ptr.p + QL, s);
        db->list_smp.alloc(db->list_nnz, s, &db->budget, false, "row list samples");
        launch_1d(QL, s, [&](uint32_t b, hipStream_t st_) {
            {
                JAS_TIMED("list_gather", st_);
                k_list_gather<<<b, 256, 0, st_>>>(Lrow.p, rptrp, rdegp, Sp, db->list_ptr.p, QL, db->list_smp.p);
            }
        });
        check_launch("list gather");
    } else {
        db->list_ptr.alloc(1, s, &db->budget, false, "row list pointers");
        {
            JAS_TIMED("fill_u64", s);
            k_fill_u64<<<1, 1, 0, s>>>(db->list_ptr.p, 1, 0);
        }
        db->list_nnz = 0;
        db->list_smp.alloc(1, s, &db->budget, false, "row list samples");
    }

    // --- query index -----------------------------------------------------------
    if (keep) {
        db->n_keys = NDk;
        uint32_t ib = ceil_log2_u64(div_up(std::max<uint64_t>(NDk, 1), 32));
        ib = std::max<uint32_t>(1, std::min<uint32_t>(ib, std::min<uint32_t>(db->U, 26)));
        db->ibits = ib;
        const uint64_t nbk = uint64_t(1) << ib;
        db->bucket.alloc(nbk + 1, s, &db->budget, false, "query buckets");
        if (NDk == 0) {
            {
                JAS_TIMED("fill_u64", s);
                k_fill_u64<<<64, 256, 0, s>>>(db->bucket.p, nbk + 1, 0);
            }
            db->keys.alloc(1, s, &db->budget, false, "query index keys");
        } else {
            launch_1d(NDk + 1, s, [&](uint32_t b, hipStream_t st_) {
                {
                    JAS_TIMED("bucket", st_);
                    k_bucket<<<b, 256, 0, st_>>>(Dk.p, NDk, sbits, db->U - ib, nbk, db->bucket.p);
                }
            });
            db->keys = std::move(Dk);
            db->keys.owned_by_db = true;
        }
        check_launch("query buckets");
    }

    // --- stats -----------------------------------------------------------------
    if (!have_st) read_back(ReadBack().add(st.p, (uint32_t)st.n), hst, s);
    add_slots(hst, slots);
    if (sized) hst[ST_LISTPAIRS] = list_pairs;
    jas_encode_stats &o = db->stats;
    db->trace.N = N;
    db->trace.ND = NDk;
    db->trace.NS = NS;
    db->trace.R = R;
    db->trace.QD = QD;
    db->trace.QL = QL;
    db->trace.nb = nb;
    db->trace.Hw = Hw;
    db->trace.H = H;
    o.n_ids = N;
    o.n_pairs = NDk;
    o.n_rows = hst[ST_ROWS];
    o.n_shared_rows = R;
    o.n_packed_rows = QD;
    o.n_list_rows = QL;
    o.n_batches = nb;
    o.n_word_rows = Hw;
    o.word_bits = wb;
    o.w_rows = H;
    o.w_stride = ldw;
    o.n_list_pairs = db->n_lpairs;
    o.nnz_words = hst[ST_NNZW];
    o.word_pairs_F = hst[ST_F];
    o.list_pairs = hst[ST_LISTPAIRS];
    o.device_bytes = db->budget.held;
    set_tile_stats(o, (uint64_t)n);
}

// The encode of a plan: the common path of jas_encode (single-pass scatters
// on the top ID bits, ranges finished in LDS with the planned stride and key
// width, the planned degree threshold, row lists as sorted pair words), every
// size read from device memory and every buffer the plan's own.  Nothing is
// read back and nothing allocated, so the whole sequence can be captured in a
// HIP graph; what the eager path would have done differently (a fallback) or
// a size above its capacity is flagged in p.err and reported afterwards.
void encode_planned(PlanState &p, const uint64_t *ids, const uint64_t *offsets, hipStream_t s) {
    const int32_t n = p.n;
    const uint32_t sbits = p.sbits, U = p.U;
    const uint64_t smask = sbits ? ((uint64_t(1) << sbits) - 1) : 0;
    uint64_t *dsz = p.dsz.p;
    uint32_t *err = p.err.p;
    const uint64_t Ncap = p.Ncap;
    {
        JAS_TIMED("plan_sizes", s);
        Clear c;
        c.add(p.ghist.p, p.ghist.n);
        c.add(p.st.p, p.st.n);
        c.add(p.dupc.p, (uint64_t)std::max<int32_t>(n, 1));
        if (p.QLcap > 0) c.add(p.gh.p, p.gh.n);
        k_plan_begin<<<256, 256, 0, s>>>(offsets, n, Ncap, dsz, err, c);
    }
    check_launch("plan begin");
    // keys and the global sort on the top ID bits
    const uint64_t hi_mask = U >= 64 ? 0 : ~((uint64_t(1) << U) - 1);
    const uint32_t chunk = key_chunk(Ncap), key_blocks = (uint32_t)div_up(Ncap, (uint64_t)chunk);
    if (p.sort.top_bits > 0) {  // the sort's first pass forms the keys
        JAS_TIMED("count_digits", s);
        k_count_digits<<<key_blocks, kNT, 0, s>>>(ids, Ncap, hi_mask, err, p.sort.npass,
                                                                       U - p.sort.top_bits, p.sort.width, p.ghist.p,
                                                                       dsz, chunk);
    } else {
        JAS_TIMED("build_keys", s);
        k_build_keys<<<key_blocks, kNT, 0, s>>>(ids, offsets, n, Ncap, sbits, hi_mask, p.keys.p,
                                                                     err, p.sort.npass, U - p.sort.top_bits,
                                                                     p.sort.width, p.ghist.p, dsz, chunk);
    }
    check_launch("build keys (planned)");
    uint64_t *K = p.keys.p, *F = p.alt.p;
    if (p.sort.top_bits > 0) {
        OnesweepBufs ob;
        ob.gstart = p.os_gstart.p;
        ob.maxima = p.os_maxima.p;
        ob.status = p.os_status.p;
        ob.status_words = p.os_status.n;
        KeySource src;
        src.ids = ids;
        src.off = offsets;
        src.n = n;
        src.sbits = sbits;
        src.tinfo = p.os_tinfo.p;
        src.tinfo_words = p.os_tinfo.n;
        const uint32_t lo = sbits + U - p.sort.top_bits, hi = sbits + U;
        radix_sort_onesweep_planned(K, F, dsz + PZ_N, Ncap, lo, hi, p.sort.width, p.ghist.p, err, ob, s, &src);
    }
    // ranges of whole buckets, finished in LDS
    const uint32_t lowbits = U - p.sort.top_bits;
    const uint32_t bsh = sbits + lowbits;
    const uint64_t nlc = p.nlc_cap;
    {
        JAS_TIMED("range_starts", s);
        k_range_starts<<<(uint32_t)div_up(nlc + 1, 256 / kWave), 256, 0, s>>>(K, Ncap, bsh, p.stride, nlc, p.rs.p,
                                                                               err, dsz, p.lcap);
        k_range_check<<<(uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(div_up(nlc, 256), 4096)), 256, 0, s>>>(
            K, p.rs.p, nlc, bsh, lowbits, sbits, err, dsz, p.stride, p.lcap);  // bit 16 matters only to narrow plans
    }
    check_launch("range starts (planned)");
    uint32_t *Sg = reinterpret_cast<uint32_t *>(F);
    uint64_t *rptr_g = F + div_up(Ncap, 2);
    {
        JAS_TIMED(p.wide ? "local_cls_wide" : "local_cls", s);
        launch_local_cls(p.wide, p.lcap, (uint32_t)nlc, s, K, sbits, smask, bsh, lowbits, (const uint64_t *)p.rs.p,
                         (uint32_t)nlc, p.cnt.p, 0, Sg, p.rid_g.p, rptr_g, p.dupc.p, p.st.p + stat_rows(p.slots), p.slots, dsz,
                         p.stride, err);
    }
    check_launch("local classify (planned)");
    scan_excl_u32_rows(p.cnt.p, nlc, {p.offD.p, p.offS.p, p.offR.p}, nlc, p.stmp.p, s);
    {
        JAS_TIMED("plan_sizes", s);
        k_plan_rows<<<1, 1, 0, s>>>(p.offR.p, p.offS.p, nlc, p.Rcap, p.rptr.p, dsz, err);
    }
    {
        JAS_TIMED("local_move", s);
        k_local_move<<<(uint32_t)std::min<uint64_t>(nlc, 65536), 256, 0, s>>>(
            p.rs.p, nlc, p.offD.p, p.offS.p, p.offR.p, K, p.rid_g.p, rptr_g, nullptr, p.rid.p, p.rptr.p, p.rdeg.p, dsz,
            p.stride);
    }
    {
        JAS_TIMED("card", s);
        k_card_from_dups<<<(uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(div_up(n, 256), 1024)), 256, 0, s>>>(
            offsets, p.dupc.p, n, p.card.p, (int64_t)card_limit(), err);
    }
    check_launch("local move (planned)");
    // rows by degree
    {
        JAS_TIMED("row_count", s);
        k_row_count<<<(uint32_t)p.tile_cap, kNT, 0, s>>>(p.rdeg.p, p.Rcap, p.dmin, p.tcnt.p,
                                                            p.st.p + stat_lists(p.slots), p.slots, dsz);
    }
    scan_excl_u32(p.tcnt.p, p.toff.p, p.tile_cap, p.stmp.p, s);
    {
        JAS_TIMED("plan_sizes", s);
        k_plan_split<<<1, 1, 0, s>>>(p.toff.p, p.tile_cap, p.QDcap, p.QLcap, dsz, err);
    }
    {
        JAS_TIMED("row_split", s);
        k_row_split<<<(uint32_t)p.tile_cap, kNT, 0, s>>>(p.rdeg.p, p.Rcap, p.dmin, p.toff.p, p.Drow.p, p.Lrow.p, dsz);
    }
    check_launch("row split (planned)");
    // packed rows
    if (p.QDcap > 0) {
        const uint64_t QDc = p.QDcap;
        launch_1d(QDc, s, [&](uint32_t b, hipStream_t st_) {
            JAS_TIMED("batch_flag", st_);
            k_batch_flag<<<b, 256, 0, st_>>>(p.Drow.p, p.rid.p, QDc, p.batch_bits, p.bs.p, dsz);
        });
        scan_excl_u32(p.bs.p, p.bpos.p, QDc, p.stmp.p, s);
        {
            JAS_TIMED("plan_sizes", s);
            k_plan_batches<<<1, 1, 0, s>>>(p.bpos.p, QDc, p.bq.p, dsz);
        }
        launch_1d(QDc, s, [&](uint32_t b, hipStream_t st_) {
            JAS_TIMED("batch_start", st_);
            k_batch_start<<<b, 256, 0, st_>>>(p.bs.p, p.bpos.p, QDc, p.bq.p, dsz);
            k_batch_words<<<b, 256, 0, st_>>>(p.bq.p, QDc, p.word_bits, p.nw.p, dsz);
        });
        scan_excl_u64(p.nw.p, p.wbase.p, QDc, p.stmp.p, s);
        {
            JAS_TIMED("plan_sizes", s);
            k_plan_words<<<1, 1, 0, s>>>(p.wbase.p, QDc, p.word_bits, p.Hwcap, p.Hcap, dsz, err);
        }
        launch_1d(QDc, s, [&](uint32_t b, hipStream_t st_) {
            JAS_TIMED("word_rows", st_);
            k_word_rows<<<b, 256, 0, st_>>>(QDc, p.bpos.p, p.bq.p, p.wbase.p, p.word_bits, p.wq0.p, p.wq1.p, dsz);
        });
        {
            JAS_TIMED("pack", s);
            launch_pack(p.W.p, p.ldw, p.Hcap, p.Hwcap, p.word_bits, p.wq0.p, p.wq1.p, p.QDcap, p.Drow.p, p.rptr.p,
                        p.rdeg.p, reinterpret_cast<const uint32_t *>(F), p.st.p + stat_words_of(p.slots), p.slots, dsz, s);
        }
        check_launch("pack (planned)");
    }
    // row lists as pair words sorted by the smaller sample
    if (p.QLcap > 0) {
        const uint64_t QLc = p.QLcap;
        launch_1d(QLc, s, [&](uint32_t b, hipStream_t st_) {
            JAS_TIMED("list_npairs", st_);
            k_list_wave_pairs<<<b, 256, 0, st_>>>(p.Lrow.p, p.rdeg.p, QLc, p.np.p, dsz);
        });
        scan_excl_u64(p.np.p, p.npo.p, p.gcap, p.stmp.p, s);
        {
            JAS_TIMED("plan_sizes", s);
            k_plan_pairs<<<1, 1, 0, s>>>(p.npo.p, p.gcap, p.Pcap, dsz, err);
        }
        {
            JAS_TIMED("pair_emit", s);
            k_pair_emit<<<pair_emit_grid(QLc), 256, 0, s>>>(
                p.Lrow.p, p.rptr.p, p.rdeg.p, reinterpret_cast<const uint32_t *>(F), QLc, p.npo.p, p.pk.p,
                p.pair_npass, p.pair_width, p.gh.p, dsz);
        }
        check_launch("pair emit (planned)");
        OnesweepBufs ob;
        ob.gstart = p.os2_gstart.p;
        ob.maxima = p.os2_maxima.p;
        ob.status = p.os2_status.p;
        ob.status_words = p.os2_status.n;
        uint32_t *a = p.pk.p, *b = p.palt.p;
        radix_sort_onesweep_u32_planned(a, b, dsz + PZ_P, p.Pcap, 16, 16 + p.pair_bits, p.pair_width, p.gh.p, err,
                                        ob, s);
        if (a != p.pairs_final) fail(JAS_EDEVICE, "planned pair sort ended in an unexpected buffer");
    }
}

}  // namespace jas
