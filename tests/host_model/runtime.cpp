// Threads, streams and memory of the host model (see hip/hip_runtime.h).
#include <sys/mman.h>

#include <deque>
#include <map>
#include <memory>
#include <set>
#include <string>
#include <vector>

#include "jas_internal.hpp"
#undef threadIdx
#undef blockIdx
#undef blockDim
#undef gridDim

// ---------------------------------------------------------------------------
// Threads of a block.
namespace model {
Index tid, bid;
dim3 bdim, gdim;
char *dynamic_lds;
long atomic_adds, atomic_swaps, barriers;

namespace {
constexpr uint32_t kMaxThreads = 1024;
constexpr size_t kStackBytes = 256 << 10;
enum State { kRun, kWave, kBlock, kDone };
struct Fiber {
    void *sp;
    char *stack;
    State state;
    uint64_t value;
    void *site;  // where in the code it waits
    int order;
    uint32_t t;
};
Fiber fibers[kMaxThreads], *current;
Group groups[kMaxThreads / 64];
void *scheduler_sp;
const std::function<void()> *thread_body;

extern "C" void model_switch(void **save, void *load);
asm(R"(
.globl model_switch
model_switch:
  pushq %rbp; pushq %rbx; pushq %r12; pushq %r13; pushq %r14; pushq %r15
  movq %rsp, (%rdi)
  movq %rsi, %rsp
  popq %r15; popq %r14; popq %r13; popq %r12; popq %rbx; popq %rbp
  ret
)");

void wait_in(State s) {
    current->state = s;
    model_switch(&current->sp, scheduler_sp);
}
void fiber_main() {
    (*thread_body)();
    wait_in(kDone);
    abort();
}

// Lets the lanes [a, b) of a wave run until each waits for its block or is done.
void run_wave(uint32_t a, uint32_t b) {
    for (;;) {
        for (uint32_t t = a; t < b; ++t) {
            if (fibers[t].state != kRun) continue;
            current = &fibers[t];
            tid = {t % bdim.x, t / bdim.x, 0};
            model_switch(&scheduler_sp, fibers[t].sp);
        }
        const Fiber *first = nullptr;
        for (uint32_t t = a; t < b; ++t) {
            const Fiber &f = fibers[t];
            if (f.state == kWave && (!first || f.order < first->order || (f.order == first->order && f.site < first->site)))
                first = &f;
        }
        if (!first) return;
        Group &g = groups[a / 64];
        void *site = first->site;
        g.mask = 0;
        for (uint32_t t = a; t < b; ++t) {
            Fiber &f = fibers[t];
            if (f.state != kWave || f.site != site) continue;
            g.mask |= 1ull << (t - a);
            g.v[t - a] = f.value;
            f.state = kRun;
        }
    }
}

void run_block() {
    const uint32_t nt = bdim.x * bdim.y;
    for (uint32_t t = 0; t < nt; ++t) {
        Fiber &f = fibers[t];
        if (!f.stack)
            f.stack = (char *)mmap(nullptr, kStackBytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE,
                                   -1, 0);
        uint64_t *sp = (uint64_t *)(f.stack + kStackBytes - 64);
        *--sp = 0;
        *--sp = (uint64_t)&fiber_main;
        for (int i = 0; i < 6; ++i) *--sp = 0;
        f.sp = sp;
        f.state = kRun;
        f.t = t;
    }
    for (bool live = true; live;) {
        for (uint32_t a = 0; a < nt; a += 64) run_wave(a, std::min(nt, a + 64));
        live = false;
        for (uint32_t t = 0; t < nt; ++t) {  // every thread that is left waits at the block's barrier
            if (fibers[t].state != kBlock) continue;
            fibers[t].state = kRun;
            live = true;
        }
        barriers += live;
    }
}
}  // namespace

uint32_t lane() { return current->t % 64; }
void barrier() { wait_in(kBlock); }
__attribute__((noinline)) const Group &exchange(uint64_t v, int order) {
    current->value = v;
    current->order = order;
    current->site = __builtin_return_address(0);
    wait_in(kWave);
    return groups[current->t / 64];
}

void run_grid(dim3 grid, dim3 block, size_t lds, const std::function<void()> &thread) {
    if (block.x * block.y > kMaxThreads) abort();
    gdim = grid;
    bdim = block;
    thread_body = &thread;
    std::unique_ptr<char, decltype(&free)> mem((char *)malloc(lds ? lds : 1), &free);
    memset(mem.get(), 0xA5, lds);
    dynamic_lds = mem.get();
    for (uint32_t y = 0; y < grid.y; ++y)
        for (uint32_t x = 0; x < grid.x; ++x) {
            bid = {x, y, 0};
            run_block();
        }
}
}  // namespace model

// ---------------------------------------------------------------------------
// Streams and events.
struct model_stream {
    std::deque<std::pair<std::string, std::function<void()>>> q;
};
namespace {
struct Marker {
    model_stream *s;
    bool done;
};
}  // namespace
struct model_event {
    std::shared_ptr<Marker> m;
};

namespace model {
namespace {
model_stream null_stream;
std::set<model_stream *> streams{&null_stream};
hipError_t last_error = hipSuccess;
bool lazy = false;
std::map<std::string, long> launches, blocks;

model_stream *stream(hipStream_t s) { return s ? s : &null_stream; }
void step(model_stream *s) {
    auto work = std::move(s->q.front().second);
    s->q.pop_front();
    work();
}
void drain(model_stream *s) {
    while (!s->q.empty()) step(s);
}
}  // namespace

void enqueue(const char *name, hipStream_t s, std::function<void()> f) {
    stream(s)->q.emplace_back(name, std::move(f));
    if (!lazy) drain(stream(s));
}
// The limits of a launch: 2^32 threads along x, 1024 per block, 160 KB of LDS.
bool check_launch(const char *name, dim3 g, dim3 b, size_t lds) {
    const std::string kernel = std::string(name).substr(0, std::string(name).find('<'));
    ++launches[kernel];
    blocks[kernel] += (long)g.x * g.y;
    if (g.x && g.y && b.x && (uint64_t)g.x * b.x < (1ull << 32) && b.x * b.y <= kMaxThreads && lds <= 163840)
        return true;
    fprintf(stderr, "launch of %s refused: grid %u x %u, block %u, %zu bytes of LDS\n", name, g.x, g.y, b.x, lds);
    last_error = hipErrorInvalidConfiguration;
    return false;
}
}  // namespace model
using namespace model;

const char *hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : "error of the host model"; }
hipError_t hipMalloc(void **p, size_t n) {
    *p = malloc(n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) {
    free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
    drain(stream(s));
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
    for (auto *s : streams) drain(s);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *src, size_t n, hipMemcpyKind k, hipStream_t s) {
    if (k == hipMemcpyDeviceToDevice) {
        enqueue("copy", s, [=] { memmove(d, src, n); });
    } else if (k == hipMemcpyHostToDevice) {  // (pageable: the source may change once the call is back)
        std::string copy((const char *)src, n);
        enqueue("copy", s, [d, copy] { memcpy(d, copy.data(), copy.size()); });
    } else {
        drain(stream(s));
        memcpy(d, src, n);
    }
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *src, size_t n, hipMemcpyKind) {
    (void)hipDeviceSynchronize();
    memcpy(d, src, n);
    return hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}
hipError_t hipEventCreate(hipEvent_t *e) {
    *e = new model_event;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
    delete e;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    auto m = std::make_shared<Marker>(Marker{stream(s), false});
    e->m = m;
    enqueue("event", s, [m] { m->done = true; });
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
    if (e->m)
        while (!e->m->done) step(e->m->s);
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = 1.f;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    auto m = e->m;
    if (m)
        enqueue("wait", s, [m] {
            while (!m->done) step(m->s);
        });
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    *s = new model_stream;
    streams.insert(*s);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t *f, size_t *t) {
    *f = *t = (size_t)256 << 30;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, int, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *symbol) {
    *p = const_cast<void *>(symbol);
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// The library's buffers, each an allocation of exactly its size (in place of
// the cache in memory.hip, which rounds sizes up and keeps blocks): one that is
// given back in stream order is freed when its stream gets there, one that is
// given back as idle is freed at once.
namespace jas {
namespace {
std::map<void *, hipStream_t> live;
std::vector<std::string> asked;  // what for, since model_fail_at
long fail_at = -1;
int fill = 0xFF;
}  // namespace

void *cache_alloc(size_t bytes, hipStream_t s, const char *what) {
    if (fail_at >= 0 && (long)asked.size() >= fail_at) fail(JAS_ENOMEM, std::string("refused: ") + what);
    asked.push_back(what);
    void *p = malloc(bytes);
    memset(p, fill, bytes);
    live[p] = s;
    return p;
}
void cache_free(void *p, bool idle) {
    const auto it = live.find(p);
    if (it == live.end()) return;
    const hipStream_t s = it->second;
    live.erase(it);
    if (idle) free(p);
    else model::enqueue("free", s, [p] { free(p); });
}
}  // namespace jas

extern "C" {
void model_lazy(int on) { model::lazy = on != 0; }
void model_drain() { (void)hipDeviceSynchronize(); }
// Kernels and copies enqueued that have not run.
long model_pending() {
    long n = 0;
    for (auto *s : model::streams)
        for (auto &e : s->q) n += e.first != "free" && e.first != "event" && e.first != "wait";
    return n;
}
// The k-th allocation from here on is refused (-1: none).
void model_fail_at(long k) {
    jas::asked.clear();
    jas::fail_at = k;
}
long model_allocations() { return (long)jas::asked.size(); }
long model_atomic_adds() { return model::atomic_adds; }
long model_barriers() { return model::barriers; }  // of blocks
long model_atomic_swaps() { return model::atomic_swaps; }
// Launches of a kernel (of all of a template's) so far, and their blocks.
long model_launches(const char *kernel) { return model::launches[kernel]; }
long model_blocks(const char *kernel) { return model::blocks[kernel]; }
long model_live() { return (long)jas::live.size(); }
}
