// Device memory cache of libjas.
//
// Every device buffer the library uses comes from here.  A freed block is
// kept, tagged with the stream that last used it and its event, recorded on that
// stream (an event is made once per block: creating and destroying one per
// free cost more than recording it); a later request reuses it on the same
// stream directly, or on another stream after making that stream wait for the
// event.  Steady-state calls thus never reach hipMalloc/hipFree, whose cost for
// multi-GB buffers is large and erratic.  jas_trim() hands the cached blocks
// back to the device.
#include <algorithm>
#include <map>
#include <mutex>
#include <vector>

#include "jas_internal.hpp"

namespace jas {
namespace {

struct Block {
    void *p;
    size_t bytes;
    hipStream_t s;
    hipEvent_t ev;  // made when the block is first freed
    bool pending;   // ev marks work that may still use the block
    int device;
};

std::mutex g_mu;
std::multimap<size_t, Block> g_free;  // by size
std::map<void *, Block> g_live;       // outstanding blocks by address
uint64_t g_cached = 0, g_in_use = 0;

size_t round_size(size_t bytes) {
    if (bytes < (1u << 20)) return (bytes + 511) & ~size_t(511);
    return (bytes + (2u << 20) - 1) & ~size_t((2u << 20) - 1);
}

void release_all_locked() {
    (void)hipDeviceSynchronize();
    for (auto &kv : g_free) {
        if (kv.second.ev) (void)hipEventDestroy(kv.second.ev);
        (void)hipFree(kv.second.p);
    }
    g_free.clear();
    g_cached = 0;
    (void)hipGetLastError();
}

}  // namespace

void *cache_alloc(size_t bytes, hipStream_t s, const char *what) {
    const size_t need = round_size(bytes ? bytes : 1);
    int dev = 0;
    JAS_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_mu);
    const size_t cap = need < (64u << 20) ? 2 * need : need + need / 4;
    for (auto it = g_free.lower_bound(need); it != g_free.end() && it->first <= cap; ++it) {
        Block b = it->second;
        if (b.device != dev) continue;
        g_free.erase(it);
        if (b.pending && b.s != s) {
            const hipError_t e = hipStreamWaitEvent(s, b.ev, 0);
            if (e != hipSuccess) {
                g_free.emplace(b.bytes, b);
                check_hip(e, "hipStreamWaitEvent");
            }
        }
        b.pending = false;
        b.s = s;
        g_cached -= b.bytes;
        g_in_use += b.bytes;
        g_live[b.p] = b;
        return b.p;
    }
    void *p = nullptr;
    hipError_t e;
    {
        JAS_HOST_TIMED("malloc");
        e = hipMalloc(&p, need);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        release_all_locked();
        e = hipMalloc(&p, need);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            fail(JAS_ENOMEM, std::string("device allocation of ") + std::to_string(need) + " bytes for " + what +
                                 " failed: " + hipGetErrorString(e));
        }
    }
    g_in_use += need;
    g_live[p] = Block{p, need, s, nullptr, false, dev};
    return p;
}

void cache_free(void *p, bool synced) {
    if (!p) return;
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_live.find(p);
    if (it == g_live.end()) return;
    Block b = it->second;
    g_live.erase(it);
    b.pending = false;
    if (!synced) {
        if ((!b.ev && hipEventCreateWithFlags(&b.ev, hipEventDisableTiming) != hipSuccess) ||
            hipEventRecord(b.ev, b.s) != hipSuccess) {
            // cannot tag the block: wait for its stream instead
            (void)hipGetLastError();
            if (b.ev) (void)hipEventDestroy(b.ev);
            b.ev = nullptr;
            (void)hipStreamSynchronize(b.s);
        } else {
            b.pending = true;
        }
    }
    g_in_use -= b.bytes;
    g_cached += b.bytes;
    g_free.emplace(b.bytes, b);
}

namespace {
// Pinned blocks of read_back, for any device.  One is in use per call that
// waits for its words; at most kKeptBlocks idle ones are kept.
constexpr size_t kKeptBlocks = 16;
std::mutex g_pin_mu;
std::vector<uint64_t *> g_pin;

__global__ void k_gather(ReadBack r, uint64_t *out) {
    uint32_t o = 0;
    for (int k = 0; k < ReadBack::kMax; ++k) {
        for (uint32_t i = threadIdx.x; i < r.words[k]; i += blockDim.x) out[o + i] = r.src[k][i];
        o += r.words[k];
    }
}

__global__ void k_clear(Clear c) {
    for (int k = 0; k < Clear::kMax; ++k)
        for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < c.words[k];
             i += (uint64_t)gridDim.x * blockDim.x)
            c.p[k][i] = 0;
}
}  // namespace

void read_back(const ReadBack &r, uint64_t *out, hipStream_t s) {
    JAS_HOST_TIMED("readback_sync");
    uint32_t total = 0;
    for (int k = 0; k < r.n; ++k) total += r.words[k];
    if (total > kReadWords) fail(JAS_EDEVICE, "read back: too many words");
    uint64_t *block = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_pin_mu);
        if (!g_pin.empty()) {
            block = g_pin.back();
            g_pin.pop_back();
        }
    }
    if (!block)
        JAS_HIP(hipHostMalloc(reinterpret_cast<void **>(&block), kReadWords * sizeof(uint64_t), hipHostMallocPortable));
    k_gather<<<1, 128, 0, s>>>(r, block);
    // (on an error the block may still be written: it is not used again)
    check_launch("read back");
    JAS_HIP(hipStreamSynchronize(s));
    std::copy(block, block + total, out);
    std::lock_guard<std::mutex> lk(g_pin_mu);
    if (g_pin.size() < kKeptBlocks) g_pin.push_back(block);
    else (void)hipHostFree(block);
}

void clear_words(const Clear &c, hipStream_t s) {
    uint64_t most = 1;
    for (int k = 0; k < c.n; ++k) most = std::max(most, c.words[k]);
    JAS_TIMED("fill_u64", s);
    k_clear<<<(uint32_t)std::min<uint64_t>(div_up(most, 256), 1024), 256, 0, s>>>(c);
    check_launch("clear");
}

hipStream_t side_stream() {
    static std::mutex mu;
    static std::map<int, hipStream_t> streams;  // one per device, kept for the process
    int dev = 0;
    JAS_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(mu);
    auto it = streams.find(dev);
    if (it != streams.end()) return it->second;
    hipStream_t st = nullptr;
    JAS_HIP(hipStreamCreateWithFlags(&st, hipStreamNonBlocking));  // default priority
    streams[dev] = st;
    return st;
}

void stream_after(hipStream_t waiter, hipStream_t on) {
    hipEvent_t ev = nullptr;
    JAS_HIP(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
    const hipError_t e1 = hipEventRecord(ev, on);
    const hipError_t e2 = e1 == hipSuccess ? hipStreamWaitEvent(waiter, ev, 0) : e1;
    (void)hipEventDestroy(ev);
    if (e2 != hipSuccess) {
        // cannot order the streams by an event: wait for the work itself
        (void)hipGetLastError();
        JAS_HIP(hipStreamSynchronize(on));
    }
}

StreamJoin::~StreamJoin() {
    if (!armed) return;
    // an error is on its way out, and the buffers of both streams are freed
    // next: the host waits too
    (void)hipStreamSynchronize(on);
    try {
        stream_after(waiter, on);
    } catch (...) {
    }
}

void cache_trim() {
    {
        std::lock_guard<std::mutex> lk(g_pin_mu);
        for (uint64_t *b : g_pin) (void)hipHostFree(b);
        g_pin.clear();
    }
    std::lock_guard<std::mutex> lk(g_mu);
    release_all_locked();
}

uint64_t cache_bytes() {
    std::lock_guard<std::mutex> lk(g_mu);
    return g_cached;
}

}  // namespace jas

extern "C" void jas_trim(void) { jas::cache_trim(); }
