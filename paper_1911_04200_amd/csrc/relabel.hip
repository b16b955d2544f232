// Exact relabelling of IDs by rank: every ID becomes its position among the
// distinct IDs of the array.  Equal IDs stay equal and distinct ones stay
// distinct, so every |X_i cap X_j| (and with it B, C and J) is unchanged,
// while the universe shrinks from U bits to ceil(log2 D) bits (D distinct
// IDs).  It lets long k-mers (k = 31: IDs below 2^62, Sec. II-B) go through
// the encoder, whose keys (ID << ceil(log2 n)) | sample must fit 64 bits.
//
//   1. the IDs sorted by their top bits (single-pass scatters) and each range
//      of whole buckets finished in LDS, as the encoder does, which leaves the
//      distinct IDs, ascending; where a bucket is too large for that, the IDs
//      sorted on every bit, then head flags, a scan and compaction;
//   2. a table of 64-byte lines, one per value of the top `ibits` ID bits: where
//      the IDs with those bits start among the distinct IDs, and 16 more bits of
//      each; for every input ID its line gives its rank.
// Bits above the highest one in which two IDs differ are left out of both (the
// digit totals of the first sort show when that can matter).
// 134 M k-mers of 62 bits (k = 31), 39 M distinct: 20.8 ms with a sort on every
// bit (eight passes, 4.9 ms), flags and compaction (2.4) and ranks by binary
// search (12.2); now 11.9 ms: two passes (1.2), ranges (3.9, their LDS passes over
// 47 bits), lines (0.3) and ranks (5.6, scattered 64-byte reads).
#include <algorithm>

#include "device_util.hpp"
#include "jas_internal.hpp"

namespace jas {
namespace {

constexpr int kNT = 256;

__global__ void k_zero_u64(uint64_t *p, uint64_t len) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < len; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}
__global__ void k_zero_u32(uint32_t *p) { *p = 0; }

__global__ __launch_bounds__(kNT) void k_id_digits(const uint64_t *__restrict__ ids, uint64_t N, uint64_t mask,
                                                    uint32_t npass, unsigned long long *__restrict__ ghist) {
    __shared__ uint32_t gh[kMaxPasses][256];
#pragma unroll
    for (int k = 0; k < kMaxPasses; ++k) gh[k][threadIdx.x] = 0;
    __syncthreads();
    for (uint64_t i = (uint64_t)blockIdx.x * kNT + threadIdx.x; i < N; i += (uint64_t)gridDim.x * kNT) {
        const uint64_t id = ids[i] & mask;
        for (uint32_t q = 0; q < npass; ++q) atomicAdd(&gh[q][(uint32_t)(id >> (8 * q)) & 255u], 1u);
    }
    __syncthreads();
    unsigned long long *g = ghist + (uint64_t)(blockIdx.x % kGhistReplicas) * kMaxPasses * 256;
    for (uint32_t q = 0; q < npass; ++q)
        if (gh[q][threadIdx.x]) atomicAdd(&g[q * 256 + threadIdx.x], (unsigned long long)gh[q][threadIdx.x]);
}

// diff |= the bits in which some ID differs from the first.
__global__ __launch_bounds__(kNT) void k_id_diff(const uint64_t *__restrict__ ids, uint64_t N, unsigned long long *diff) {
    unsigned long long d = 0;
    const uint64_t first = ids[0];
    for (uint64_t i = (uint64_t)blockIdx.x * kNT + threadIdx.x; i < N; i += (uint64_t)gridDim.x * kNT) d |= ids[i] ^ first;
#pragma unroll
    for (int k = 1; k < kWave; k <<= 1) d |= __shfl_xor(d, k, kWave);
    if (lane_id() == 0 && d) atomicOr(diff, d);
}

// head[i] = 1 where sorted[i] starts a new value
__global__ void k_heads(const uint64_t *__restrict__ sorted, uint64_t N, uint32_t *__restrict__ head) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (uint64_t)gridDim.x * blockDim.x)
        head[i] = i == 0 || sorted[i] != sorted[i - 1];
}

__global__ void k_compact_heads(const uint64_t *__restrict__ sorted, uint64_t N, const uint32_t *__restrict__ head,
                                const uint64_t *__restrict__ pos, uint64_t *__restrict__ distinct) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (uint64_t)gridDim.x * blockDim.x)
        if (head[i]) distinct[pos[i]] = sorted[i];
}

// bucket[b] = first distinct ID whose top bits ((id & mask) >> shift) are >= b,
// b in [0, nbk].  A thread writes the entries between its ID's bucket and the one
// before; where there are more than a few, its wave writes them (2^21 entries
// between two groups of IDs: 67 ms by one thread, 1.1 so).
__global__ void k_rank_buckets(const uint64_t *__restrict__ distinct, uint64_t D, uint64_t mask, uint32_t shift,
                               uint64_t nbk, uint64_t *__restrict__ bucket) {
    constexpr int64_t kFew = 16;
    const uint32_t lane = lane_id();
    const auto of = [&](uint64_t t) { return shift >= 64 ? 0 : (int64_t)((distinct[t] & mask) >> shift); };
    const uint64_t step = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t - lane <= D; t += step) {  // wave-uniform
        int64_t from = 0, to = -1;
        if (t <= D) {
            from = t == 0 ? 0 : of(t - 1) + 1;
            to = t < D ? of(t) : (int64_t)nbk;
        }
        for (uint64_t many = __ballot(to - from >= kFew); many; many &= many - 1) {
            const int l = __builtin_ctzll(many);
            const int64_t a = __shfl(from, l, kWave), z = __shfl(to, l, kWave);
            for (int64_t b = a + lane; b <= z; b += kWave) bucket[b] = t - lane + l;
        }
        if (to - from < kFew)
            for (int64_t b = from; b <= to; ++b) bucket[b] = t;
    }
}

// The ranks of N IDs in no particular order cost one scattered read each, so
// what a rank needs is put in one 64-byte line: the word start | count << 48 and,
// in ascending order, the 16 ID bits below the bucket's of up to 28 IDs.  A
// search of the 8-byte IDs through a bucket table read two to three 128-byte
// lines (134 M IDs, 39 M distinct: 11.1 ms, 5.6 now).  A bucket with more IDs is
// marked by the count kFullLine and searched in the distinct IDs.
constexpr uint32_t kLineIds = 28, kLineWords = 8;  // 8-byte words of a line
constexpr uint64_t kFullLine = 0xFFFF, kStartMask = (uint64_t(1) << 48) - 1;
// Buckets of up to this many IDs are searched from the place an ID's bits point
// to; in larger ones (crowded IDs, seldom evenly spread) halving takes half the
// steps a guess that is far off does (33 M ranks in two buckets: 11.1 and 6.0 ms).
constexpr uint64_t kNear = 256;

// The 16 bits of id below its bucket's (all of them, if shift <= 16).
// (shift < 64 takes only bits that the mask leaves)
__device__ __forceinline__ uint32_t line_bits(uint64_t id, uint32_t shift) {
    const uint64_t low = shift >= 64 ? id : id & ((uint64_t(1) << shift) - 1);
    return (uint32_t)(shift > 16 ? low >> (shift - 16) : low);
}

// Eight threads per line: word 0 and the seven words of four IDs each.
__global__ void k_rank_lines(const uint64_t *__restrict__ distinct, const uint64_t *__restrict__ bucket, uint64_t nbk,
                             uint32_t shift, uint64_t *__restrict__ lines) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nbk * kLineWords;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t b = i / kLineWords, start = bucket[b], cnt = bucket[b + 1] - start;
        const uint32_t w = (uint32_t)(i % kLineWords);
        uint64_t v = 0;
        if (w == 0) {
            v = start | (cnt > kLineIds ? kFullLine : cnt) << 48;
        } else {
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) {
                const uint64_t e = 4 * (w - 1) + k;
                // past the last ID: above every ID's bits, or equal (then never before it)
                v |= (uint64_t)(e < cnt ? line_bits(distinct[start + e], shift) : 0xFFFFu) << (16 * k);
            }
        }
        lines[i] = v;
    }
}

// out[i] = rank of ids[i] among the distinct IDs (out may be ids); every ID is
// one of them, so the only one of the bucket with its 16 bits needs no look at
// the distinct IDs themselves.  The line is read whole, at once: it is gone from
// the cache when a second read of it would follow.
// 134 M IDs, 39 M distinct: 6.2 ms with the line's first word, then the one the
// ID was expected in, then the ID itself; 5.6 ms so.  (Half the lines, 18 IDs each
// on average: 7.9, too many are full.)
__global__ void k_rank(const uint64_t *ids, uint64_t N, const uint64_t *__restrict__ distinct,
                       const uint64_t *__restrict__ bucket, const uint64_t *__restrict__ lines, uint64_t mask,
                       uint32_t shift, uint64_t *out) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t id = ids[i], b = shift >= 64 ? 0 : (id & mask) >> shift;
        const uint4 *line = reinterpret_cast<const uint4 *>(lines + b * kLineWords);
        const uint4 q[4] = {line[0], line[1], line[2], line[3]};
        const uint64_t head = (uint64_t)q[0].y << 32 | q[0].x, start = head & kStartMask, cnt = head >> 48;
        if (cnt == kFullLine) {
            uint64_t lo = start, hi = bucket[b + 1];
            if (hi - lo <= kNear) {
                lo = lower_bound_from(distinct, lo, hi, id, shift ? id << (64 - shift) : 0);
            } else {
                while (lo < hi) {
                    const uint64_t m = lo + (hi - lo) / 2;
                    if (distinct[m] < id) lo = m + 1;
                    else hi = m;
                }
            }
            out[i] = lo;
            continue;
        }
        const uint32_t r = line_bits(id, shift);
        uint32_t below = 0, upto = 0;
        const auto take = [&](uint32_t v) {
            below += (uint32_t)((v & 0xFFFFu) < r) + (uint32_t)((v >> 16) < r);
            upto += (uint32_t)((v & 0xFFFFu) <= r) + (uint32_t)((v >> 16) <= r);
        };
        take(q[0].z);
        take(q[0].w);
#pragma unroll
        for (int k = 1; k < 4; ++k) {
            take(q[k].x);
            take(q[k].y);
            take(q[k].z);
            take(q[k].w);
        }
        uint64_t pos = start + below;
        // IDs that agree in the 16 bits too: compared whole
        if (shift > 16 && upto - below > 1)
            while (pos + 1 < start + cnt && distinct[pos] < id) ++pos;
        out[i] = pos;
    }
}

uint32_t grid_for(uint64_t work) {
    return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(div_up(work, 256), 65536));
}

}  // namespace

namespace {
// The distinct IDs by a sort on each of their low U bits (mask; the others are the
// same in every ID): returns their number, in alt.
uint64_t distinct_full_sort(const uint64_t *ids, uint64_t N, uint32_t U, uint64_t mask, DevBuf<uint64_t> &keys,
                            DevBuf<uint64_t> &alt, unsigned long long *ghist, uint32_t *err, hipStream_t s) {
    const uint32_t npass = (U + 7) / 8;
    {
        JAS_TIMED("relabel_digits", s);
        k_zero_u64<<<64, 256, 0, s>>>(reinterpret_cast<uint64_t *>(ghist), (uint64_t)kGhistReplicas * kMaxPasses * 256);
        k_id_digits<<<(uint32_t)std::min<uint64_t>(div_up(N, 256 * 16), 8192), kNT, 0, s>>>(ids, N, mask, npass, ghist);
    }
    check_launch("relabel digits");
    uint32_t herr = 0;
    bool sorted = radix_sort_onesweep(keys, alt, N, 0, U, 8, ghist, err, s, nullptr, nullptr, nullptr, ids);
    if (sorted) {
        JAS_HIP(hipMemcpyAsync(&herr, err, 4, hipMemcpyDeviceToHost, s));
        JAS_HIP(hipStreamSynchronize(s));
        sorted = herr == 0;
    }
    if (!sorted) {  // digit totals too large for the single-pass form, or its look-back gave up
        JAS_HIP(hipMemcpyAsync(keys.p, ids, N * 8, hipMemcpyDeviceToDevice, s));
        RadixWork rw;
        radix_sort_u64(keys, alt, N, 0, U, rw, s, nullptr);
    }
    DevBuf<uint32_t> head;
    DevBuf<uint64_t> pos, tmp;
    head.alloc(N, s, nullptr, true, "relabel heads");
    pos.alloc(N + 1, s, nullptr, true, "relabel positions");
    tmp.alloc(scan_tmp_elems(N), s, nullptr, true, "scan scratch");
    {
        JAS_TIMED("relabel_unique", s);
        k_heads<<<grid_for(N), 256, 0, s>>>(keys.p, N, head.p);
    }
    scan_excl_u32(head.p, pos.p, N, tmp.p, s);
    {
        JAS_TIMED("relabel_unique", s);
        k_compact_heads<<<grid_for(N), 256, 0, s>>>(keys.p, N, head.p, pos.p, alt.p);
    }
    check_launch("relabel unique");
    uint64_t D = 0;
    JAS_HIP(hipMemcpyAsync(&D, pos.p + N, 8, hipMemcpyDeviceToHost, s));
    JAS_HIP(hipStreamSynchronize(s));
    return D;
}
}  // namespace

uint64_t relabel(const uint64_t *ids, uint64_t N, uint32_t U, hipStream_t s, uint64_t *out) {
    if (N == 0) return 0;
    DevBuf<uint32_t> err;
    err.alloc(2, s, nullptr, true, "relabel error flag");
    DevBuf<unsigned long long> ghist;
    ghist.alloc((uint64_t)kGhistReplicas * kMaxPasses * 256, s, nullptr, true, "relabel digit totals");
    DevBuf<uint64_t> dig, diff;
    dig.alloc((uint64_t)kMaxPasses * 257, s, nullptr, true, "relabel digit starts");
    diff.alloc(1, s, nullptr, true, "relabel ID difference");
    uint64_t *maxima = dig.p + (uint64_t)kMaxPasses * 256;
    uint32_t bits = U;  // the IDs are the same above these
    SortPlan plan;
    bool crowded = false;
    for (bool again = false;; again = true) {
        plan = sort_plan(N, bits, 0);
        clear_words(Clear().add(ghist.p, (uint64_t)kGhistReplicas * kMaxPasses * 256).add(err.p, 1).add(diff.p, 1), s);
        build_keys(ids, nullptr, 0, N, 0, bits, plan, nullptr, err.p, ghist.p, s);
        digit_starts(ghist.p, plan.npass, plan.width, dig.p, maxima, s);
        uint64_t got[1 + kMaxPasses];
        read_back(ReadBack().add(err.p).add(maxima, kMaxPasses), got, s);
        if (!again && got[0]) fail(JAS_EINVAL, "jas_relabel: an ID is >= 2^universe_bits");
        // some bucket of the sorted bits surely exceeds an LDS range when the
        // IDs of one top digit do on average
        const uint32_t below = plan.npass ? plan.width * (plan.npass - 1) : 0;
        crowded = plan.npass && got[plan.npass] > (uint64_t)kLocalCapKeys << below;
        if (!crowded || again) break;
        {
            JAS_TIMED("relabel_diff", s);
            k_id_diff<<<(uint32_t)std::min<uint64_t>(div_up(N, 256 * 16), 4096), kNT, 0, s>>>(
                ids, N, reinterpret_cast<unsigned long long *>(diff.p));
        }
        check_launch("relabel difference");
        uint64_t d = 0;
        read_back(ReadBack().add(diff.p), &d, s);
        const uint32_t used = d ? 64 - (uint32_t)__builtin_clzll(d) : 1;
        if (used >= bits) break;
        bits = used;
    }
    const uint64_t mask = bits >= 64 ? ~0ull : (uint64_t(1) << bits) - 1;
    clear_words(Clear().add(err.p, 1), s);  // (of the ID check against fewer bits)
    uint32_t herr = 0;
    DevBuf<uint64_t> keys, alt;
    keys.alloc(N, s, nullptr, true, "relabel keys");
    alt.alloc(N, s, nullptr, true, "relabel keys (second buffer)");
    uint64_t D = ~0ull;
    if (plan.top_bits == 0) {  // one range holds everything
        JAS_HIP(hipMemcpyAsync(keys.p, ids, N * 8, hipMemcpyDeviceToDevice, s));
        D = distinct_sorted(keys, alt, N, bits, plan, s);
    } else if (!crowded && radix_sort_onesweep(keys, alt, N, bits - plan.top_bits, bits, plan.width, ghist.p, err.p, s,
                                               nullptr, nullptr, nullptr, ids)) {
        JAS_HIP(hipMemcpyAsync(&herr, err.p, 4, hipMemcpyDeviceToHost, s));
        JAS_HIP(hipStreamSynchronize(s));
        if (!herr) D = distinct_sorted(keys, alt, N, bits, plan, s);
        else k_zero_u32<<<1, 1, 0, s>>>(err.p);  // the sort's look-back gave up
    }
    if (D == ~0ull) D = distinct_full_sort(ids, N, bits, mask, keys, alt, ghist.p, err.p, s);
    // buckets of 5 to 10 distinct IDs where the lines, which take the place of
    // the sorted keys, allow it (2^ib lines of 64 bytes in 8 N bytes)
    uint32_t ib = std::min<uint32_t>(ceil_log2_u64(div_up(D, 10)), bits);
    while (ib > 0 && ((uint64_t)kLineWords << ib) > N) --ib;
    const uint32_t shift = bits - ib;
    const uint64_t nbk = uint64_t(1) << ib;
    DevBuf<uint64_t> bucket, small;
    bucket.alloc(nbk + 1, s, nullptr, true, "relabel buckets");
    if (N < kLineWords) small.alloc(kLineWords, s, nullptr, true, "relabel line");
    uint64_t *lines = N < kLineWords ? small.p : keys.p;
    {
        JAS_TIMED("relabel_lines", s);
        k_rank_buckets<<<grid_for(D + 1), 256, 0, s>>>(alt.p, D, mask, shift, nbk, bucket.p);
        k_rank_lines<<<grid_for(nbk * kLineWords), 256, 0, s>>>(alt.p, bucket.p, nbk, shift, lines);
    }
    {
        JAS_TIMED("relabel_rank", s);
        k_rank<<<grid_for(N), 256, 0, s>>>(ids, N, alt.p, bucket.p, lines, mask, shift, out);
    }
    check_launch("relabel rank");
    JAS_HIP(hipStreamSynchronize(s));
    return D;
}

}  // namespace jas
