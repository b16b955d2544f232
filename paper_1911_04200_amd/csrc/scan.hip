// Exclusive prefix sums over device arrays (reduce-then-scan, no inter-block
// waiting): each block sums 4096 entries, then scans them from the sum of the
// blocks before it.
#include <algorithm>

#include "device_util.hpp"
#include "jas_internal.hpp"

namespace jas {
namespace {

constexpr int kNT = 256;
constexpr int kItems = 16;
constexpr uint64_t kBlock = (uint64_t)kNT * kItems;
// Up to this many blocks, each adds up the sums before it by itself (a few loads
// per thread); past it the sums are scanned first.  A scan is then one launch
// (one block) or two instead of two or five of about 4.5 us each (a planned
// encode of 22 M IDs, with 6 calls: 1.14 to 1.06 ms), and the entries are read
// twice and written once instead of written, read and written again.
constexpr uint64_t kDirect = 2048;

// Arrays scanned by one launch (blockIdx.y): in + y * stride to out[y].
struct Outs {
    uint64_t *p[kScanRows];
};

__device__ __forceinline__ uint64_t block_sum(uint64_t v, uint64_t *sh) {
    v = wave_incl_scan(v);
    if (lane_id() == kWave - 1) sh[threadIdx.x / kWave] = v;
    __syncthreads();
    uint64_t t = 0;
#pragma unroll
    for (int k = 0; k < kNT / kWave; ++k) t += sh[k];
    __syncthreads();
    return t;
}

template <class T>
__global__ __launch_bounds__(kNT) void k_scan_sums(const T *__restrict__ in, uint64_t stride, uint64_t len,
                                                   uint64_t *__restrict__ sums) {
    __shared__ uint64_t sh[kNT / kWave];
    const T *p = in + blockIdx.y * stride;
    const uint64_t b0 = (uint64_t)blockIdx.x * kBlock;
    uint64_t s = 0;
#pragma unroll
    for (int m = 0; m < kItems; ++m) {
        const uint64_t idx = b0 + (uint64_t)m * kNT + threadIdx.x;
        s += idx < len ? (uint64_t)p[idx] : 0;
    }
    s = block_sum(s, sh);
    if (threadIdx.x == 0) sums[(uint64_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
}

// starts[b]: sum of the blocks before b, or (null) sums holds every block's own.
template <class T>
__global__ __launch_bounds__(kNT) void k_scan_block(const T *__restrict__ in, uint64_t stride, Outs outs, uint64_t len,
                                                    const uint64_t *__restrict__ sums,
                                                    const uint64_t *__restrict__ starts) {
    __shared__ uint64_t stage[kBlock];
    __shared__ uint64_t sh[kNT / kWave];
    const T *p = in + blockIdx.y * stride;
    uint64_t *out = outs.p[blockIdx.y];
    const uint64_t b0 = (uint64_t)blockIdx.x * kBlock;
    const uint32_t tid = threadIdx.x;
    // coalesced load into LDS
#pragma unroll
    for (int m = 0; m < kItems; ++m) {
        const uint64_t idx = b0 + (uint64_t)m * kNT + tid;
        stage[m * kNT + tid] = idx < len ? (uint64_t)p[idx] : 0;
    }
    uint64_t before = 0;
    if (starts) {
        before = starts[blockIdx.x];
    } else if (blockIdx.x > 0) {
        const uint64_t *sy = sums + (uint64_t)blockIdx.y * gridDim.x;
        for (uint32_t b = tid; b < blockIdx.x; b += kNT) before += sy[b];
        before = block_sum(before, sh);
    }
    __syncthreads();
    // each thread owns kItems consecutive entries
    uint64_t v[kItems];
    uint64_t s = 0;
#pragma unroll
    for (int m = 0; m < kItems; ++m) {
        v[m] = stage[tid * kItems + m];
        s += v[m];
    }
    uint64_t tot;
    uint64_t run = before + block_excl_scan<kNT>(s, sh, &tot);
#pragma unroll
    for (int m = 0; m < kItems; ++m) {
        stage[tid * kItems + m] = run;
        run += v[m];
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < kItems; ++m) {
        const uint64_t idx = b0 + (uint64_t)m * kNT + tid;
        if (idx < len) out[idx] = stage[m * kNT + tid];
    }
    if (tid == 0 && blockIdx.x == gridDim.x - 1) out[len] = before + tot;
}

template <class T>
void scan_impl(const T *in, uint64_t stride, const Outs &outs, uint32_t rows, size_t len, uint64_t *tmp,
               hipStream_t s) {
    const uint64_t nb = std::max<uint64_t>(div_up(len, kBlock), 1);  // an empty array's total is 0
    if (nb > kDirect && rows > 1) {
        for (uint32_t y = 0; y < rows; ++y) scan_impl<T>(in + y * stride, 0, Outs{{outs.p[y]}}, 1, len, tmp, s);
        return;
    }
    const dim3 grid((uint32_t)nb, rows);
    uint64_t *sums = tmp, *starts = nullptr;  // rows * nb
    if (nb > 1) {
        JAS_TIMED("scan_sums", s);
        k_scan_sums<T><<<grid, kNT, 0, s>>>(in, stride, len, sums);
        check_launch("scan sums");
    }
    if (nb > kDirect) {
        starts = tmp + nb;  // nb + 1
        scan_impl<uint64_t>(sums, 0, Outs{{starts}}, 1, nb, starts + nb + 1, s);
    }
    {
        JAS_TIMED("scan_block", s);
        k_scan_block<T><<<grid, kNT, 0, s>>>(in, stride, outs, len, sums, starts);
    }
    check_launch("scan block");
}

}  // namespace

size_t scan_tmp_elems(size_t len, uint32_t rows) {
    const size_t nb = div_up(len, kBlock);
    const size_t direct = rows * std::max<size_t>(std::min<size_t>(nb, kDirect), 1);
    return nb > kDirect ? std::max(direct, 2 * nb + 1 + scan_tmp_elems(nb)) : direct;
}

void scan_excl_u32(const uint32_t *in, uint64_t *out, size_t len, uint64_t *tmp, hipStream_t s) {
    scan_impl<uint32_t>(in, 0, Outs{{out}}, 1, len, tmp, s);
}

void scan_excl_u32_rows(const uint32_t *in, uint64_t stride, uint64_t *const (&out)[kScanRows], size_t len,
                        uint64_t *tmp, hipStream_t s) {
    Outs o;
    std::copy(out, out + kScanRows, o.p);
    scan_impl<uint32_t>(in, stride, o, kScanRows, len, tmp, s);
}

void scan_excl_u64(const uint64_t *in, uint64_t *out, size_t len, uint64_t *tmp, hipStream_t s) {
    scan_impl<uint64_t>(in, 0, Outs{{out}}, 1, len, tmp, s);
}

}  // namespace jas
