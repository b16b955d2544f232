// Query x database similarity: Eq. (1) with i over query sets, j over the
// encoded samples.
//
// The query block of B is B_qj = sum_k q_k a_kj over rows k of A.  Each distinct
// ID of a query set is looked up in the database's sorted distinct keys (a
// table of start positions by the ID's top bits, then a search from the place
// the ID's next bits point to), and every database sample holding that ID gains
// 1.  A block accumulates its part of one query's row of B in LDS before adding
// it to global memory.
//
// Query sets become sets in one of two ways.  Requests of small sets go set by
// set through hash tables in LDS (k_query_small): a set's IDs are dealt to its
// blocks by a hash, each block drops the repeats of its share and looks the
// rest up, all in one launch.  Larger ones are made sets like the database: keys
// (q << U) | id, a stable radix sort, repeats dropped where equal keys meet
// (k_qlookup).
#include <algorithm>

#include "device_util.hpp"
#include "jas_internal.hpp"

namespace jas {
namespace {

constexpr int kNT = 256;
constexpr uint64_t kQChunk = 2048;  // query entries per block (more blocks than CUs for typical requests)
constexpr int32_t kHistMax = 16384;
constexpr uint64_t kMaxBlocks = uint64_t(1) << 22;  // of a launch (2^32 threads are too many)
constexpr uint32_t kWalk = 512;  // database entries of one ID a thread reads before it leaves the rest to its block

// Small sets: IDs per block on average (16 to 512, for about kSmallBlocks
// blocks), slots of a block's table (at least four times as many: a
// share is binomial, so at most a few dozen slots in a row are taken unless IDs are
// chosen against the hash; an ID that finds kProbes taken leaves the request to
// the sorted path), and the largest set and request taken.
constexpr uint32_t kMinShareLog = 4, kShareLog = 9, kSlots = 2048, kProbes = 128, kSmallBlocks = 512;
constexpr uint64_t kSpareBlocks = 1024;  // blocks without a share that may be launched: half of what runs at once
constexpr uint64_t kSmallSet = 32768, kSmallIds = uint64_t(1) << 20;

// Keys (q << U) | id of 4096 entries per block, and the totals of every
// 8-bit digit of the keys (kGhistReplicas copies) for the single-pass sort.
__global__ __launch_bounds__(kNT) void k_qkeys(const uint64_t *__restrict__ ids, const uint64_t *__restrict__ off,
                                                int32_t nq, uint64_t N, uint32_t U, uint64_t *__restrict__ keys,
                                                uint32_t *err, uint32_t npass, unsigned long long *__restrict__ ghist) {
    __shared__ int32_t s_lo, s_hi;
    __shared__ uint32_t gh[kMaxPasses][256];
    const uint64_t b0 = (uint64_t)blockIdx.x * 4096;
    const uint64_t b1 = min(N, b0 + 4096);
#pragma unroll
    for (int k = 0; k < kMaxPasses; ++k) gh[k][threadIdx.x] = 0;
    if (threadIdx.x == 0) {
        s_lo = find_sample(off, 0, nq - 1, b0);
        s_hi = find_sample(off, s_lo, nq - 1, b1 - 1);
    }
    __syncthreads();
    const uint64_t hi_mask = ~((uint64_t(1) << U) - 1);
    uint32_t bad = 0;
    for (uint64_t t = b0 + threadIdx.x; t < b1; t += kNT) {
        const int32_t q = find_sample(off, s_lo, s_hi, t);
        const uint64_t id = ids[t];
        bad |= (id & hi_mask) != 0;
        const uint64_t key = ((uint64_t)q << U) | (id & ~hi_mask);
        keys[t] = key;
        for (uint32_t p = 0; p < npass; ++p) atomicAdd(&gh[p][(uint32_t)(key >> (8 * p)) & 255u], 1u);
    }
    if (__ballot(bad) && lane_id() == 0) atomicOr(err, 1u);
    __syncthreads();
    if (ghist) {
        unsigned long long *g = ghist + (uint64_t)(blockIdx.x % kGhistReplicas) * kMaxPasses * 256;
        for (uint32_t p = 0; p < npass; ++p)
            if (gh[p][threadIdx.x]) atomicAdd(&g[p * 256 + threadIdx.x], (unsigned long long)gh[p][threadIdx.x]);
    }
}

__global__ void k_qblocks(const uint64_t *off, int32_t nq, uint64_t *nb) {
    for (int32_t q = blockIdx.x * blockDim.x + threadIdx.x; q < nq; q += gridDim.x * blockDim.x)
        nb[q] = (off[q + 1] - off[q] + kQChunk - 1) / kQChunk;
}

// B = 0 and words[0 .. nwords) = 0.
__global__ void k_query_zero(int32_t *B, uint64_t len, uint32_t *words, uint64_t nwords) {
    const uint64_t step = (uint64_t)gridDim.x * blockDim.x, i0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (uint64_t i = i0; i < len; i += step) B[i] = 0;
    for (uint64_t i = i0; i < nwords; i += step) words[i] = 0;
}

// The database's side of a lookup.
struct Index {
    const uint64_t *keys, *bucket;
    uint64_t n_keys;
    uint32_t U, ibits, sbits, n;
};

// First position in ix.keys whose ID is >= id (among those of id's bucket, or
// one past them).  A bucket holds about 32 keys, 256 bytes; the search starts
// where the ID's bits below the bucket's point to.
__device__ __forceinline__ uint64_t first_at(const Index &ix, uint64_t id) {
    const uint32_t shift = ix.U - ix.ibits;
    const uint64_t bk = id >> shift;
    return lower_bound_from(ix.keys, ix.bucket[bk], ix.bucket[bk + 1], id << ix.sbits,
                            shift ? id << (64 - shift) : 0);
}

// What a block keeps while it looks its IDs up.
struct LongRuns {
    uint64_t at[kNT], id[kNT];  // entries of an ID from position `at` on, left to the block
    uint32_t count;
};

// Looks up one ID per thread (have = false: none) and adds 1 to the counter of
// every database sample holding it: in the LDS row hist, or (hist null) in row
// B_q.  A thread reads up to kWalk entries of its ID itself; the rest of a longer
// run (an ID many samples hold: a power-law graph's hubs have 60,000 of 2^20
// vertices, which one thread read in 10 to 22 ms) is read by the whole block,
// eight entries per thread in flight.  Every thread
// of the block calls it.
__device__ __forceinline__ void count_holders(const Index &ix, uint64_t id, bool have, uint32_t *hist, int32_t *B_q,
                                              LongRuns &lr) {
    const uint64_t smask = ix.sbits ? (uint64_t(1) << ix.sbits) - 1 : 0;
    const auto add = [&](uint64_t key) {
        const uint32_t s = (uint32_t)(key & smask);
        if (hist) atomicAdd(&hist[s], 1u);
        else atomicAdd(&B_q[s], 1);
    };
    if (have) {
        uint64_t u = first_at(ix, id);
        const uint64_t end = min(ix.n_keys, u + kWalk);
        bool in = true;
        while (in && u < end) {
            uint64_t d[4];
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) d[k] = u + k < end ? ix.keys[u + k] : ~0ull;
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) {
                in = in && u + k < end && (d[k] >> ix.sbits) == id;
                if (in) add(d[k]);
            }
            u += 4;
        }
        if (in && end < ix.n_keys) {  // every entry up to `end` held the ID
            const uint32_t e = atomicAdd(&lr.count, 1u);
            lr.at[e] = end;
            lr.id[e] = id;
        }
    }
    __syncthreads();
    const uint32_t nl = lr.count;
    for (uint32_t e = 0; e < nl; ++e) {
        const uint64_t rid = lr.id[e];
        for (uint64_t u = lr.at[e] + threadIdx.x;; u += 8 * kNT) {
            uint64_t d[8];
#pragma unroll
            for (uint32_t k = 0; k < 8; ++k) d[k] = u + k * kNT < ix.n_keys ? ix.keys[u + k * kNT] : ~0ull;
            bool in = false;
#pragma unroll
            for (uint32_t k = 0; k < 8; ++k) {
                in = u + k * kNT < ix.n_keys && (d[k] >> ix.sbits) == rid;
                if (in) add(d[k]);
            }
            if (!in) break;  // the run ends before this thread's last entry
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) lr.count = 0;
    __syncthreads();
}

// Sorted path: a block per slice of kQChunk keys of one query (bo: the slices
// before each query's), in turn where the grid is smaller.
__global__ __launch_bounds__(kNT) void k_qlookup(const uint64_t *__restrict__ K, const uint64_t *__restrict__ qoff,
                                                  int32_t nq, const uint64_t *__restrict__ bo, Index ix, int lds,
                                                  int32_t *__restrict__ B, unsigned long long *__restrict__ qcard) {
    extern __shared__ uint32_t hist[];
    __shared__ uint64_t sh[kNT / kWave];
    __shared__ LongRuns lr;
    const uint32_t tid = threadIdx.x;
    const uint64_t slices = bo[nq], umask = (uint64_t(1) << ix.U) - 1;
    for (uint64_t b = blockIdx.x; b < slices; b += gridDim.x) {
        int32_t lo = 0, hi = nq - 1;
        while (lo < hi) {
            const int32_t mid = lo + (hi - lo + 1) / 2;
            if (bo[mid] <= b) lo = mid;
            else hi = mid - 1;
        }
        const int32_t q = lo;
        const uint64_t qs = qoff[q];
        const uint64_t t0 = qs + (b - bo[q]) * kQChunk;
        const uint64_t t1 = min(qoff[q + 1], t0 + kQChunk);
        if (lds)
            for (uint32_t i = tid; i < ix.n; i += kNT) hist[i] = 0;
        if (tid == 0) lr.count = 0;
        __syncthreads();
        uint32_t cnt = 0;
        for (uint64_t t = t0 + tid; t - tid < t1; t += kNT) {  // uniform
            bool have = t < t1;
            uint64_t key = 0;
            if (have) {
                key = K[t];
                have = t == qs || K[t - 1] != key;  // else a repeat inside this query set
            }
            cnt += have;
            count_holders(ix, key & umask, have && ix.n_keys > 0, lds ? hist : nullptr, B + (uint64_t)q * ix.n, lr);
        }
        uint64_t tot;
        block_excl_scan<kNT>(cnt, sh, &tot);
        if (tid == 0 && tot) atomicAdd(&qcard[q], (unsigned long long)tot);
        if (lds)
            for (uint32_t i = tid; i < ix.n; i += kNT)
                if (hist[i]) atomicAdd(&B[(uint64_t)q * ix.n + i], (int32_t)hist[i]);
        __syncthreads();  // the row is cleared again
    }
}

// Small sets: query q has P blocks, or with P = 0 those from small_block(q) on, one
// for each share of its IDs; block p takes the IDs whose hash falls in share p, drops repeats
// through a hash table in LDS and looks the others up.
// err |= 1 for an ID >= 2^U, |= 8 when a table is too full (the sorted path then
// runs instead).
// (q + its first ID / share leaves a query 1 + floor(end / share) - floor(start /
// share) blocks, at least as many as it has shares, so the grid is the number of
// queries plus that of shares however unequal the sets are.  As many blocks for
// each as the longest has, 20,000 sets of which one has 32,768 IDs took 3.5 ms,
// and with more sets the grid passed a launch's 2^32 threads.)
__device__ __host__ __forceinline__ uint64_t small_block(uint64_t q, uint64_t start, uint32_t log_share) {
    return q + (start >> log_share);
}

__global__ __launch_bounds__(kNT) void k_query_small(const uint64_t *__restrict__ ids,
                                                      const uint64_t *__restrict__ qoff, int32_t nq, uint32_t P, uint32_t log_share,
                                                      Index ix, int lds, int32_t *__restrict__ B, unsigned long long *__restrict__ qcard,
                                                      uint32_t *err) {
    extern __shared__ uint32_t hist[];
    __shared__ unsigned long long slot[kSlots];
    __shared__ uint16_t found[kSlots];  // slots in use
    __shared__ uint32_t nfound;
    __shared__ LongRuns lr;
    const uint32_t tid = threadIdx.x;
    int32_t q = 0;
    uint32_t p = 0;
    if (P) {
        q = (int32_t)(blockIdx.x / P);
        p = blockIdx.x % P;
    } else {
        // the last query whose blocks start here or before; as many blocks as the grid has
        // more than there are queries are in front of it at most.  Each wave looks at 64
        // of the rest at once
        q = max((int32_t)(blockIdx.x - (gridDim.x - (uint32_t)nq)), 0);
        for (int32_t left = min(nq, (int32_t)blockIdx.x + 1) - q; left > 1;) {
            const int32_t step = (left + kWave - 1) / kWave, o = step * (int32_t)(tid % kWave);
            const uint64_t before = __ballot(o < left && small_block(q + o, qoff[o < left ? q + o : q], log_share) <= blockIdx.x);
            const int32_t first = step * (__popcll(before) - 1);
            q += first;
            left = min(step, left - first);
        }
        p = blockIdx.x - (uint32_t)small_block(q, qoff[q], log_share);
    }
    const uint64_t qs = qoff[q];
    const uint32_t len = (uint32_t)(qoff[q + 1] - qs);
    const uint32_t parts = (len + (1u << log_share) - 1) >> log_share;
    if (p >= parts) return;
    constexpr unsigned long long kEmpty = ~0ull;  // no ID: U <= 63
    for (uint32_t i = tid; i < kSlots; i += kNT) slot[i] = kEmpty;
    if (lds)
        for (uint32_t i = tid; i < ix.n; i += kNT) hist[i] = 0;
    if (tid == 0) {
        nfound = 0;
        lr.count = 0;
    }
    __syncthreads();
    uint32_t bad = 0;
    // (a thread that found the table too full stops: the sorted path takes the
    // request.  8194 IDs chosen for one share: 7.4 ms with every slot looked at for
    // each ID, 0.44 ms so, the sorted path and all)
    for (uint32_t i0 = tid; i0 < len && !(bad & 8u); i0 += 8 * kNT) {
        uint64_t v[8];
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) v[u] = i0 + u * kNT < len ? ids[qs + i0 + u * kNT] : 0;
#pragma unroll
        for (uint32_t u = 0; u < 8; ++u) {
            const uint64_t id = v[u];
            if (id >> ix.U) {  // refused, and not looked up: it has no bucket
                bad |= 1u;
                continue;
            }
            // a multiplicative hash (Knuth): its high half picks the block, both halves the slot
            const uint64_t h = (id ^ (id >> 32)) * 0x9E3779B97F4A7C15ull;
            if (i0 + u * kNT >= len || (uint32_t)(((h >> 32) * parts) >> 32) != p) continue;
            uint32_t s = ((uint32_t)h ^ (uint32_t)(h >> 32)) % kSlots, probes = 0;
            for (;;) {
                const unsigned long long old = atomicCAS(&slot[s], kEmpty, (unsigned long long)id);
                if (old == kEmpty) {
                    found[atomicAdd(&nfound, 1u)] = (uint16_t)s;
                    break;
                }
                if (old == id) break;  // a repeat
                if (++probes == kProbes) {
                    bad |= 8u;
                    break;
                }
                s = (s + 1) % kSlots;
            }
        }
    }
    if (bad) atomicOr(err, bad);
    __syncthreads();
    const uint32_t nf = nfound;
    if (tid == 0 && nf) atomicAdd(&qcard[q], (unsigned long long)nf);
    for (uint32_t i = tid; i - tid < nf; i += kNT)  // uniform
        count_holders(ix, i < nf ? slot[found[i]] : 0, i < nf && ix.n_keys > 0, lds ? hist : nullptr,
                      B + (uint64_t)q * ix.n, lr);
    if (lds)
        for (uint32_t i = tid; i < ix.n; i += kNT)
            if (hist[i]) atomicAdd(&B[(uint64_t)q * ix.n + i], (int32_t)hist[i]);
}

__global__ void k_qfinalize(const int32_t *__restrict__ B, const unsigned long long *__restrict__ qcard,
                            const int64_t *__restrict__ card, int32_t nq, uint32_t n, int64_t *__restrict__ q_card,
                            int64_t *__restrict__ den, double *__restrict__ J) {
    const uint64_t total = (uint64_t)nq * n;
    for (uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; p < total; p += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t q = p / n, j = p % n;
        const int64_t b = B[p];
        const int64_t c = (int64_t)qcard[q] + card[j] - b;
        if (den) den[p] = c;
        if (J) J[p] = c == 0 ? 1.0 : (double)b / (double)c;
        if (q_card && j == 0) q_card[q] = (int64_t)qcard[q];
    }
}

}  // namespace

uint64_t query_workspace_bytes(const jas_db *db, int32_t nq, uint64_t n_q_ids) {
    (void)db;
    // keys and second buffer, the per-pass fallback's counts, look-back status
    // (two of 1 KiB per 8192 keys), digit totals and starts, per-query blocks
    const uint64_t nk = std::max<uint64_t>(n_q_ids, 1);
    return 2 * 8 * nk + radix_work_bytes(n_q_ids) + 2 * (nk / 8192 + 1) * 1024 + 512 + 2 * (uint64_t)kGhistReplicas * 8 * 256 * 8 +
           8 * (uint64_t)(nq + 1) * 4 + scan_tmp_elems(nq) * 8 + 4096;
}

void query(const jas_db *db, const uint64_t *q_ids, const uint64_t *q_offsets, int32_t nq,
           const std::vector<uint64_t> &hoff, hipStream_t s, int32_t *B, int64_t *q_card, int64_t *den, double *J,
           Arena *ar) {
    const uint32_t n = (uint32_t)db->n;
    const uint32_t U = db->U;
    const uint32_t qbits = ceil_log2_u64((uint64_t)std::max<int32_t>(nq, 1));
    if (U + qbits > 64) fail(JAS_EINVAL, "universe_bits + ceil(log2 nq) exceeds 64");
    if (nq == 0) return;
    const uint64_t NQ = hoff[nq], len = (uint64_t)nq * n;
    uint64_t longest = 0;
    for (int32_t q = 0; q < nq; ++q) longest = std::max(longest, hoff[q + 1] - hoff[q]);
    Index ix;
    ix.keys = db->keys.p;
    ix.bucket = db->bucket.p;
    ix.n_keys = n > 0 ? db->n_keys : 0;  // without a database side only |Q| is needed
    ix.U = U;
    ix.ibits = db->ibits;
    ix.sbits = db->sbits;
    ix.n = n;
    const int lds = (int32_t)n <= kHistMax && ix.n_keys > 0;
    const size_t row = lds ? n * sizeof(uint32_t) : 0;
    // |Q| per query, then the error flag and the digit totals of the sorted path
    const uint64_t nhist = (uint64_t)kGhistReplicas * kMaxPasses * 256;
    DevBuf<unsigned long long> qc;
    temp_buf(qc, (uint64_t)nq + 1 + nhist, s, nullptr, ar, "query counters");
    uint32_t *err = reinterpret_cast<uint32_t *>(qc.p + nq);
    unsigned long long *ghist = qc.p + nq + 1;
    const auto zero = [&](uint64_t words64) {
        JAS_TIMED("query_zero", s);
        const uint64_t w = std::max<uint64_t>(len, 2 * words64);
        k_query_zero<<<(uint32_t)std::min<uint64_t>(div_up(w, 256), 65536), 256, 0, s>>>(
            B, len, reinterpret_cast<uint32_t *>(qc.p), 2 * words64);
        check_launch("zero query block");
    };
    const auto finish = [&] {
        if (n > 0) {
            JAS_TIMED("qfinalize", s);
            const uint64_t blocks = std::min<uint64_t>(div_up(std::max<uint64_t>(len, nq), 256), 65536);
            k_qfinalize<<<(uint32_t)blocks, 256, 0, s>>>(B, qc.p, db->card.p, nq, n, q_card, den, J);
            check_launch("query finalize");
        } else if (q_card) {
            JAS_HIP(hipMemcpyAsync(q_card, qc.p, sizeof(int64_t) * nq, hipMemcpyDeviceToDevice, s));
        }
        uint32_t h = 0;
        JAS_HIP(hipMemcpyAsync(&h, err, 4, hipMemcpyDeviceToHost, s));
        JAS_HIP(hipStreamSynchronize(s));
        if (h & 1u) fail(JAS_EINVAL, "a query ID is >= 2^universe_bits");
        return h;
    };
    // Small sets: one launch instead of a sort's ten (one set of 10,000 IDs
    // against 4096 samples of 390,000: 300 us sorted, 80 us so).  Every block
    // reads its set's IDs, so the limits keep that reading below what the sort
    // costs (32 sets of up to a million IDs, sorted: 960 us, of which the lookups'
    // scattered lines take 570 at 4 TB/s and the sort 270).
    if (longest <= kSmallSet && NQ <= kSmallIds) {
        zero((uint64_t)nq + 1);
        if (NQ > 0) {
            uint32_t log_share = kMinShareLog;
            while (log_share < kShareLog && (uint64_t)kSmallBlocks << log_share < NQ) ++log_share;
            // a number for every set where that is hardly more blocks: no search (16 sets,
            // hubs among them: 414 us for 424)
            const uint64_t packed = small_block((uint64_t)nq - 1, NQ, log_share) + 1;
            const uint64_t per = (longest + (uint64_t(1) << log_share) - 1) >> log_share;
            const uint32_t P = (uint64_t)nq * per <= packed + kSpareBlocks ? (uint32_t)per : 0;
            const uint64_t blocks = P ? (uint64_t)nq * P : packed;
            if (blocks <= kMaxBlocks) {
                {
                    JAS_TIMED("query_small", s);
                    k_query_small<<<(uint32_t)blocks, kNT, row, s>>>(q_ids, q_offsets, nq, P, log_share, ix, lds, B, qc.p, err);
                }
                check_launch("small queries");
                if (!(finish() & 8u)) return;
            }
        } else {
            finish();
            return;
        }
    }
    // the sort, then the lookups; should the sort's look-back have given up,
    // all again with per-pass histograms
    DevBuf<uint64_t> keys, alt, nb, bo, tmp;
    temp_buf(keys, NQ, s, nullptr, ar, "query keys");
    temp_buf(alt, NQ, s, nullptr, ar, "query keys");
    temp_buf(nb, nq, s, nullptr, ar, "query blocks");
    temp_buf(bo, nq + 1, s, nullptr, ar, "query blocks");
    temp_buf(tmp, scan_tmp_elems(nq), s, nullptr, ar, "scan scratch");
    {
        JAS_TIMED("qblocks", s);
        k_qblocks<<<(uint32_t)div_up(nq, 256), 256, 0, s>>>(q_offsets, nq, nb.p);
    }
    scan_excl_u64(nb.p, bo.p, nq, tmp.p, s);
    const uint64_t lookup_blocks = std::min(div_up(NQ, kQChunk) + (uint64_t)nq, kMaxBlocks);  // the most slices there can be
    const uint64_t kb = div_up(NQ, 4096);
    const uint32_t kbits = U + qbits, npass = (kbits + 7) / 8;
    for (const bool single : {true, false}) {
        zero((uint64_t)nq + 1 + (single ? nhist : 0));
        {
            JAS_TIMED("qkeys", s);
            k_qkeys<<<(uint32_t)kb, kNT, 0, s>>>(q_ids, q_offsets, nq, NQ, U, keys.p, err, single ? npass : 0,
                                                  single ? ghist : nullptr);
        }
        check_launch("query keys");
        if (single) {
            if (!radix_sort_onesweep(keys, alt, NQ, 0, kbits, 8, ghist, err, s, nullptr, ar)) continue;
        } else {
            RadixWork rw;
            radix_sort_u64(keys, alt, NQ, 0, kbits, rw, s, nullptr, ar);
        }
        {
            JAS_TIMED("qlookup", s);
            k_qlookup<<<(uint32_t)lookup_blocks, kNT, row, s>>>(keys.p, q_offsets, nq, bo.p, ix, lds, B, qc.p);
        }
        check_launch("query lookup");
        if (!(finish() & 2u)) return;
    }
}

}  // namespace jas
