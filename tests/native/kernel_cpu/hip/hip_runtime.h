/*
 * A stand-in for <hip/hip_runtime.h> that runs HIP kernels on host threads, one thread per
 * GPU thread, one workgroup at a time.  It exists so that the decode and encode kernels' own
 * source can be compiled for the host and run under AddressSanitizer, UBSan and ThreadSanitizer
 * (tests/test_kernel_cpu_build.py, tests/test_encoder_cpu_build.py): "device" memory is host memory, so every access a
 * kernel makes outside a buffer is reported, and LDS is ordinary static memory, so every
 * unsynchronised pair of accesses is.  Only what those kernels and their host code use is
 * here.  Test infrastructure; nothing in the library includes it.
 */
#ifndef L3_KERNEL_CPU_HIP_RUNTIME_H
#define L3_KERNEL_CPU_HIP_RUNTIME_H

#include <pthread.h>
#include <stdint.h>

#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <thread>
#include <tuple>
#include <vector>

/* ---- language ------------------------------------------------------------- */

#define __global__
#define __device__
#define __host__
#define __shared__ static          /* one workgroup runs at a time */
#define __forceinline__ inline __attribute__((always_inline))
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};

namespace l3cpu {

constexpr int kWave = 64;

/* what the threads of the workgroup that is running share */
struct Workgroup {
    unsigned threads = 0;
    pthread_barrier_t all;
    pthread_barrier_t wave[16];
    uint32_t exchange[16][2][kWave];   /* [wave][parity][lane]: values handed between lanes */
};
inline Workgroup*& workgroup() {
    static Workgroup* wg = nullptr;
    return wg;
}
inline dim3& grid_dim() {
    static dim3 d;
    return d;
}
inline dim3& block_dim() {
    static dim3 d;
    return d;
}
inline thread_local dim3 t_thread_idx, t_block_idx;
inline thread_local unsigned t_parity = 0;

inline unsigned lane() { return t_thread_idx.x % kWave; }
inline unsigned wave() { return t_thread_idx.x / kWave; }

inline void wave_barrier() { pthread_barrier_wait(&workgroup()->wave[wave()]); }
inline void workgroup_barrier() { pthread_barrier_wait(&workgroup()->all); }

/* every lane of the wave hands a value in and gets the wave's 64 values to read: the
 * lanes of a wave run in lockstep on the GPU, here they meet at a barrier.  Two sets of
 * slots in turn: a lane that is one exchange ahead writes the other set. */
inline const uint32_t* exchange(uint32_t v) {
    Workgroup* wg = workgroup();
    const unsigned p = t_parity++ & 1u;
    wg->exchange[wave()][p][lane()] = v;
    wave_barrier();
    return wg->exchange[wave()][p];
}

/* LDS whose size the launch gives: a heap block of exactly that size */
inline void*& dynamic_lds() {
    static void* p = nullptr;
    return p;
}

/* Runs `body` once per thread of every workgroup of the grid. */
inline void launch(dim3 grid, dim3 block, const std::function<void()>& body, size_t lds_bytes = 0) {
    const unsigned threads = block.x * block.y * block.z;
    if (threads % kWave != 0 || threads / kWave > 16 || block.y != 1 || block.z != 1) std::abort();
    grid_dim() = grid;
    block_dim() = block;
    for (unsigned bz = 0; bz < grid.z; ++bz)
        for (unsigned by = 0; by < grid.y; ++by)
            for (unsigned bx = 0; bx < grid.x; ++bx) {
                Workgroup wg;
                wg.threads = threads;
                pthread_barrier_init(&wg.all, nullptr, threads);
                for (unsigned w = 0; w < threads / kWave; ++w) pthread_barrier_init(&wg.wave[w], nullptr, kWave);
                workgroup() = &wg;
                dynamic_lds() = lds_bytes ? std::malloc(lds_bytes) : nullptr;
                std::vector<std::thread> pool;
                pool.reserve(threads);
                for (unsigned t = 0; t < threads; ++t)
                    pool.emplace_back([&, t] {
                        t_thread_idx = dim3(t, 0, 0);
                        t_block_idx = dim3(bx, by, bz);
                        t_parity = 0;
                        body();
                    });
                for (auto& th : pool) th.join();
                for (unsigned w = 0; w < threads / kWave; ++w) pthread_barrier_destroy(&wg.wave[w]);
                pthread_barrier_destroy(&wg.all);
                workgroup() = nullptr;
                std::free(dynamic_lds());
            }
}

/* kernels launched through hipLaunchKernel (a function address and an array of argument
 * addresses) are registered with a function that unpacks the arguments */
inline std::map<const void*, std::function<void(void**)>>& registry() {
    static std::map<const void*, std::function<void(void**)>> r;
    return r;
}
/* every block of "device" memory that is alive: address -> bytes (what hipMalloc and
 * hipHostMalloc gave out, device symbols that were asked for, and what the harness adds) */
inline std::map<const void*, size_t>& regions() {
    static std::map<const void*, size_t> r;
    return r;
}
inline const void* symbol(const void* p, size_t n) {
    regions()[p] = n;
    return p;
}
/* called ahead of every hipLaunchKernel, if set (the harness can record the launch) */
inline std::function<void(const void*, dim3, dim3, void**)>& launch_observer() {
    static std::function<void(const void*, dim3, dim3, void**)> f;
    return f;
}

}  // namespace l3cpu

#define threadIdx (l3cpu::t_thread_idx)
#define blockIdx (l3cpu::t_block_idx)
#define blockDim (l3cpu::block_dim())
#define gridDim (l3cpu::grid_dim())

inline void __syncthreads() { l3cpu::workgroup_barrier(); }

inline uint32_t atomicOr(uint32_t* p, uint32_t v) { return __atomic_fetch_or(p, v, __ATOMIC_RELAXED); }
inline float __fdiv_rn(float a, float b) { return a / b; }
inline float __fsub_rn(float a, float b) { return a - b; }
inline uint32_t __float_as_uint(float f) {
    uint32_t u;
    std::memcpy(&u, &f, 4);
    return u;
}
inline uint32_t min(uint32_t a, uint32_t b) { return a < b ? a : b; }
inline uint32_t max(uint32_t a, uint32_t b) { return a > b ? a : b; }
inline int min(int a, int b) { return a < b ? a : b; }
inline int max(int a, int b) { return a > b ? a : b; }
/* a lane outside the wave: the lane's own value */
inline int __shfl(int v, int from) { return (int)l3cpu::exchange((uint32_t)v)[from & 63]; }
inline int __shfl_xor(int v, int mask) { return (int)l3cpu::exchange((uint32_t)v)[l3cpu::lane() ^ (unsigned)mask]; }
inline int __shfl_up(int v, unsigned by) {
    const unsigned l = l3cpu::lane();
    return (int)l3cpu::exchange((uint32_t)v)[l >= by ? l - by : l];
}
inline int __shfl_down(int v, unsigned by) {
    const unsigned l = l3cpu::lane();
    return (int)l3cpu::exchange((uint32_t)v)[l + by < 64 ? l + by : l];
}

/* ---- runtime -------------------------------------------------------------- */

typedef int hipError_t;
constexpr hipError_t hipSuccess = 0;
/* A stream that captures keeps its launches instead of running them; allocations go on as in the
 * relaxed mode.  A replay runs the workgroups of each kept launch, the first `most` of them if that is
 * fewer (a replay that something else on the GPU overtakes). */
struct l3cpu_stream {
    bool capturing = false;
    std::vector<std::function<void(unsigned)>> kept;
    void replay(unsigned most = ~0u) const { for (const auto& launch : kept) launch(most); }
};
typedef l3cpu_stream* hipStream_t;
struct l3cpu_event { bool captured = false; };       /* last recorded by a stream that captured */
typedef l3cpu_event* hipEvent_t;
constexpr unsigned hipEventDisableTiming = 2, hipHostMallocDefault = 0;

inline hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
enum hipDeviceAttribute_t { hipDeviceAttributeMultiprocessorCount = 63 };
/* one CU: launches of more than 8 workgroups have early rounds; with L3CPU_CUS=<n> in the
 * environment n, so that small launches take the kernels that are for launches of few workgroups a CU */
inline hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
    const char* e = std::getenv("L3CPU_CUS");
    *v = e ? std::atoi(e) : 1;
    return hipSuccess;
}
inline hipError_t hipMalloc(void** p, size_t n) {
    *p = std::malloc(n ? n : 1);
    if (*p) l3cpu::regions()[*p] = n;
    return *p ? hipSuccess : 2;
}
inline hipError_t hipFree(void* p) {
    l3cpu::regions().erase(p);
    std::free(p);
    return hipSuccess;
}
inline hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
inline hipError_t hipHostFree(void* p) { return hipFree(p); }
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = new l3cpu_event;
    return hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t e) { delete e; return hipSuccess; }
/* launches are synchronous; an event that a capture recorded stands for nothing outside captures */
constexpr hipError_t hipErrorCapturedEvent = 907;
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { e->captured = s && s->capturing; return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t e) { return e->captured ? hipErrorCapturedEvent : hipSuccess; }
inline hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    return e->captured && !(s && s->capturing) ? hipErrorCapturedEvent : hipSuccess;
}
enum hipMemcpyKind { hipMemcpyHostToDevice = 1 };
inline hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(dst, src, n);
    return hipSuccess;
}
inline hipError_t hipGetLastError() { return hipSuccess; }
#define HIP_SYMBOL(x) l3cpu::symbol(&(x), sizeof(x))
inline hipError_t hipGetSymbolAddress(void** p, const void* symbol) {
    *p = const_cast<void*>(symbol);
    return hipSuccess;
}
inline hipError_t hipLaunchKernel(const void* kernel, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
    auto it = l3cpu::registry().find(kernel);
    if (it == l3cpu::registry().end()) return 98;
    if (l3cpu::launch_observer()) l3cpu::launch_observer()(kernel, grid, block, args);
    void** a = args;
    auto call = it->second;
    l3cpu::launch(grid, block, [call, a] { call(a); });
    return hipSuccess;
}
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone = 0, hipStreamCaptureStatusActive = 1 };
inline hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* status) {
    *status = s && s->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
namespace l3cpu {
template <class... P, class... A>
void launch_on(hipStream_t stream, void (*kernel)(P...), dim3 grid, dim3 block, size_t lds_bytes, const A&... args) {
    if (!stream || !stream->capturing) return launch(grid, block, [&] { kernel(args...); }, lds_bytes);
    const std::tuple<P...> kept(args...);            /* the arguments' values now, as a recorded launch keeps them */
    stream->kept.push_back([=](unsigned most) {
        launch(dim3(grid.x < most ? grid.x : most, grid.y, grid.z), block, [&] { std::apply(kernel, kept); }, lds_bytes);
    });
}
}  // namespace l3cpu
#define hipLaunchKernelGGL(kernel, grid, block, shared_bytes, stream, ...) \
    l3cpu::launch_on((stream), &kernel, (grid), (block), (shared_bytes), __VA_ARGS__)

#endif
