// A stand-in for HIP's runtime header that lets the library's sources run on
// the CPU, for tests of its memory accesses and of the order of its work.
// model.py rewrites the few constructs a C++ compiler does not take (launches,
// dynamic LDS, register hints); everything else is compiled as it is.
//
// A kernel's threads run as fibers, 64 to a wave.  A thread runs until it needs
// others: at a block barrier, or at an operation of its wave (ballot, shuffle,
// wave barrier, an LDS atomic whose order within the wave matters).  Of the
// lanes of a wave that wait, those at the same place in the code go on together;
// of several places the earliest goes first, which is how the lanes of a wave
// come together again after a branch or a loop.  Blocks run one after another.
//
// Work on streams runs when it is enqueued, or, to show buffers that are given
// back too early, as late as the host's waits allow (model_lazy).
#pragma once
#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <tuple>
#include <type_traits>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline __attribute__((always_inline))
#define __launch_bounds__(...)
#define __shared__ static
#define __align__(x) __attribute__((aligned(x)))
#define MODEL_INLINE inline __attribute__((always_inline))

struct dim3 {
    uint32_t x, y, z;
    constexpr dim3(uint64_t a = 1, uint64_t b = 1, uint64_t c = 1) : x((uint32_t)a), y((uint32_t)b), z((uint32_t)c) {}
};
struct uint4 {
    uint32_t x, y, z, w;
};
struct alignas(16) ulonglong2 {
    unsigned long long x, y;
};
inline ulonglong2 make_ulonglong2(unsigned long long a, unsigned long long b) { return {a, b}; }

// ---------------------------------------------------------------------------
// The runtime calls the library makes.
typedef int hipError_t;
enum { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorInvalidConfiguration = 9 };
typedef struct model_stream *hipStream_t;
typedef struct model_event *hipEvent_t;
enum hipMemcpyKind { hipMemcpyHostToDevice = 1, hipMemcpyDeviceToHost = 2, hipMemcpyDeviceToDevice = 3 };
enum {
    hipStreamNonBlocking = 1,
    hipEventDisableTiming = 2,
    hipHostMallocPortable = 1,
    hipFuncAttributeMaxDynamicSharedMemorySize = 8
};
const char *hipGetErrorString(hipError_t);
hipError_t hipMalloc(void **, size_t);
hipError_t hipFree(void *);
hipError_t hipHostMalloc(void **, size_t, unsigned);
hipError_t hipHostFree(void *);
hipError_t hipGetDevice(int *);
hipError_t hipSetDevice(int);
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t);
hipError_t hipMemcpy(void *, const void *, size_t, hipMemcpyKind);
hipError_t hipStreamSynchronize(hipStream_t);
hipError_t hipDeviceSynchronize();
hipError_t hipGetLastError();
hipError_t hipEventCreate(hipEvent_t *);
hipError_t hipEventCreateWithFlags(hipEvent_t *, unsigned);
hipError_t hipEventDestroy(hipEvent_t);
hipError_t hipEventRecord(hipEvent_t, hipStream_t = nullptr);
hipError_t hipEventSynchronize(hipEvent_t);
hipError_t hipEventElapsedTime(float *, hipEvent_t, hipEvent_t);
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned);
hipError_t hipStreamCreateWithFlags(hipStream_t *, unsigned);
hipError_t hipMemGetInfo(size_t *, size_t *);
hipError_t hipFuncSetAttribute(const void *, int, int);
hipError_t hipGetSymbolAddress(void **, const void *);
#define HIP_SYMBOL(x) ((const void *)(x))

// ---------------------------------------------------------------------------
// Launches: MODEL_LAUNCH is what `kernel<<<grid, block, lds, stream>>>(args)` becomes.
namespace model {
struct Index {
    uint32_t x, y, z;
};
extern Index tid, bid;
extern dim3 bdim, gdim;
extern char *dynamic_lds;
extern long atomic_adds, atomic_swaps;  // calls of atomicAdd and atomicCAS so far

void enqueue(const char *name, hipStream_t s, std::function<void()> f);
bool check_launch(const char *name, dim3 grid, dim3 block, size_t lds);
void run_grid(dim3 grid, dim3 block, size_t lds, const std::function<void()> &thread);

struct Launch {
    const char *name;
    dim3 grid, block;
    size_t lds;
    hipStream_t s;
    Launch(const char *n, dim3 g, dim3 b, size_t l = 0, hipStream_t st = nullptr) : name(n), grid(g), block(b), lds(l), s(st) {}
    template <class... P, class... A>
    void operator()(void (*kernel)(P...), A &&...args) {
        std::tuple<std::decay_t<P>...> a{static_cast<std::decay_t<P>>(args)...};
        if (check_launch(name, grid, block, lds))
            enqueue(name, s, [kernel, a, g = grid, b = block, l = lds] { run_grid(g, b, l, [&] { std::apply(kernel, a); }); });
    }
};

// The values of the lanes that wait at this place (mask), by lane.
struct Group {
    uint64_t v[64];
    uint64_t mask;
};
__attribute__((noinline)) const Group &exchange(uint64_t v, int order = 1);  // a smaller order goes first
void barrier();
uint32_t lane();
}  // namespace model
#define threadIdx model::tid
#define blockIdx model::bid
#define blockDim model::bdim
#define gridDim model::gdim

// ---------------------------------------------------------------------------
// Device operations.
MODEL_INLINE void __syncthreads() { model::barrier(); }
MODEL_INLINE uint64_t __ballot(bool p) {
    const model::Group &g = model::exchange(p);
    uint64_t m = 0;
    for (int i = 0; i < 64; ++i) m |= (uint64_t)((g.mask >> i & 1) && g.v[i]) << i;
    return m;
}
template <class T>
MODEL_INLINE uint64_t model_bits(T v) {
    uint64_t b = 0;
    memcpy(&b, &v, sizeof(T));
    return b;
}
template <class T>
MODEL_INLINE T model_value(uint64_t b) {
    T v;
    memcpy(&v, &b, sizeof(T));
    return v;
}
template <class T>
MODEL_INLINE T __shfl(T v, int src, int = 64) {
    return model_value<T>(model::exchange(model_bits(v)).v[src & 63]);
}
template <class T>
MODEL_INLINE T __shfl_up(T v, unsigned d, int = 64) {
    const model::Group &g = model::exchange(model_bits(v));
    const uint32_t l = model::lane();
    return l >= d ? model_value<T>(g.v[l - d]) : v;
}
template <class T>
MODEL_INLINE T __shfl_xor(T v, int d, int = 64) {
    return model_value<T>(model::exchange(model_bits(v)).v[(model::lane() ^ d) & 63]);
}
MODEL_INLINE int model_readfirstlane(int v) {
    const model::Group &g = model::exchange((uint32_t)v);
    return (int)(uint32_t)g.v[__builtin_ctzll(g.mask)];
}
MODEL_INLINE int model_readlane(int v, int l) { return (int)(uint32_t)model::exchange((uint32_t)v).v[l & 63]; }
// row_shr:n, row_bcast:15, row_bcast:31 and wave_shr:1
MODEL_INLINE int model_update_dpp(int old, int v, int ctrl, int rows, int, bool) {
    const model::Group &g = model::exchange((uint32_t)v);
    const int l = (int)model::lane(), row = l / 16;
    if (!(rows >> row & 1)) return old;
    int src = -1;
    if (ctrl > 0x110 && ctrl < 0x120) src = l % 16 >= (ctrl & 15) ? l - (ctrl & 15) : -1;
    else if (ctrl == 0x142) src = row > 0 ? row * 16 - 1 : -1;
    else if (ctrl == 0x143) src = row > 1 ? 31 : -1;
    else if (ctrl == 0x138) src = l - 1;
    else abort();
    return src < 0 ? old : (int)(uint32_t)g.v[src];
}
MODEL_INLINE uint32_t model_bitop3(uint32_t a, uint32_t b, uint32_t c, uint32_t table) {
    uint32_t r = 0;
    for (int i = 0; i < 8; ++i)
        if (table >> i & 1) r |= ((i & 4) ? a : ~a) & ((i & 2) ? b : ~b) & ((i & 1) ? c : ~c);
    return r;
}
MODEL_INLINE uint32_t model_mbcnt(uint64_t m, uint32_t base) {
    return base + (uint32_t)__builtin_popcountll(m & ((1ull << model::lane()) - 1));
}
#define __builtin_amdgcn_readfirstlane(x) model_readfirstlane((int)(x))
#define __builtin_amdgcn_readlane(x, l) model_readlane((int)(x), (int)(l))
#define __builtin_amdgcn_update_dpp model_update_dpp
#define __builtin_amdgcn_bitop3_b32 model_bitop3
#define __builtin_amdgcn_mbcnt_lo(m, b) model_mbcnt((uint32_t)(m), b)
#define __builtin_amdgcn_mbcnt_hi(m, b) model_mbcnt((uint64_t)(uint32_t)(m) << 32, b)
#define __builtin_amdgcn_sbfe(v, o, w) ((int32_t)((uint32_t)(v) << (32 - (o) - (w))) >> (32 - (w)))
#define __builtin_amdgcn_ubfe(v, o, w) (((uint32_t)(v) >> (o)) & ((1u << (w)) - 1))
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_wave_barrier() ((void)model::exchange(0))
#define __builtin_amdgcn_s_sleep(x) ((void)0)
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __builtin_amdgcn_sched_group_barrier(...) ((void)0)
// (the matrix kernels are compiled but not run: the tests take the AND + popcount kernel)
#define __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, ...) (c)
#define __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, ...) (c)

// A buffer descriptor: loads past its end read as 0.
struct model_buffer {
    const char *p;
    uint32_t n;
};
MODEL_INLINE model_buffer model_make_buffer(const void *p, int, uint32_t n, uint32_t) { return {(const char *)p, n}; }
template <class T>
MODEL_INLINE T model_buffer_load(model_buffer r, uint32_t off) {
    T v;
    memset(&v, 0, sizeof v);
    for (uint32_t k = 0; k < sizeof(T); k += 4)
        if ((uint64_t)off + k + 4 <= r.n) memcpy((char *)&v + k, r.p + off + k, 4);
    return v;
}
typedef uint32_t model_v2u __attribute__((ext_vector_type(2)));
typedef uint32_t model_v4u __attribute__((ext_vector_type(4)));
#define __builtin_amdgcn_make_buffer_rsrc model_make_buffer
#define __builtin_amdgcn_raw_buffer_load_b32(r, o, s, a) model_buffer_load<uint32_t>(r, o)
#define __builtin_amdgcn_raw_buffer_load_b64(r, o, s, a) model_buffer_load<model_v2u>(r, o)
#define __builtin_amdgcn_raw_buffer_load_b128(r, o, s, a) model_buffer_load<model_v4u>(r, o)

#define __popc __builtin_popcount
#define __popcll __builtin_popcountll
MODEL_INLINE int __clzll(unsigned long long v) { return v ? __builtin_clzll(v) : 64; }
MODEL_INLINE unsigned long long __umul64hi(unsigned long long a, unsigned long long b) {
    return (unsigned long long)((unsigned __int128)a * b >> 64);
}

// LDS atomics of a wave take effect in program order, for all its lanes together.
#define __HIP_MEMORY_SCOPE_WORKGROUP 1
#define __HIP_MEMORY_SCOPE_AGENT 2
#define MODEL_STEP(scope) ((scope) == __HIP_MEMORY_SCOPE_WORKGROUP ? (void)model::exchange(0, 0) : (void)0)
#define __hip_atomic_load(p, o, scope) (MODEL_STEP(scope), *(p))
#define __hip_atomic_store(p, v, o, scope) (MODEL_STEP(scope), (void)(*(p) = (v)), MODEL_STEP(scope))
#define __hip_atomic_fetch_add(p, v, o, scope) (MODEL_STEP(scope), model_fetch_add((p), (v)))
template <class T, class V>
MODEL_INLINE T model_fetch_add(T *p, V v) {
    const T old = *p;
    *p = (T)(old + v);
    return old;
}
template <class T, class V>
MODEL_INLINE T atomicAdd(T *p, V v) {
    ++model::atomic_adds;
    return model_fetch_add(p, v);
}
template <class T, class V>
MODEL_INLINE T atomicOr(T *p, V v) {
    const T old = *p;
    *p = (T)(old | v);
    return old;
}
MODEL_INLINE uint32_t __float_as_uint(float v) {
    uint32_t u;
    memcpy(&u, &v, 4);
    return u;
}
template <class T, class V>
MODEL_INLINE T atomicMin(T *p, V v) {
    const T old = *p;
    if ((T)v < old) *p = (T)v;
    return old;
}
template <class T, class U, class V>
MODEL_INLINE T atomicCAS(T *p, U expected, V v) {
    ++model::atomic_swaps;
    const T old = *p;
    if (old == (T)expected) *p = (T)v;
    return old;
}
template <class A, class B>
constexpr MODEL_INLINE std::common_type_t<A, B> min(A a, B b) {
    typedef std::common_type_t<A, B> C;
    return (C)b < (C)a ? (C)b : (C)a;
}
template <class A, class B>
constexpr MODEL_INLINE std::common_type_t<A, B> max(A a, B b) {
    typedef std::common_type_t<A, B> C;
    return (C)a < (C)b ? (C)b : (C)a;
}
