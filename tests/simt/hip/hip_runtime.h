// Host stand-in for the HIP runtime (test infrastructure): runs the library's kernels on the
// CPU, work-item by work-item, so that a test can choose the order in which the wavefronts of a
// launch run.  Every work-item is a fiber; a wavefront's 64 run until each has reached a
// cross-lane operation, a barrier or its end.  As on the hardware, wavefronts that have ended
// drop out of barriers, and LDS keeps what the last workgroup left in it.
// Matrix and buffer instructions are only declared: a kernel that reaches one aborts.
#pragma once

#include <math.h>
#include <setjmp.h>
#include <ucontext.h>

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <thread>
#include <vector>

#define __global__
#define __host__
#define __device__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))
#define amdgpu_waves_per_eu(...) unused
// static storage, one instance per host thread: a workgroup runs in one thread
#define __shared__ thread_local

using std::isfinite;

struct double2 {
    double x, y;
} __attribute__((aligned(16)));
struct float2 {
    float x, y;
} __attribute__((aligned(8)));
struct float4 {
    float x, y, z, w;
} __attribute__((aligned(16)));
struct uint2 {
    unsigned x, y;
};
struct uint4 {
    unsigned x, y, z, w;
} __attribute__((aligned(16)));
inline double2 make_double2(double x, double y) { return {x, y}; }
inline float2 make_float2(float x, float y) { return {x, y}; }
inline float4 make_float4(float x, float y, float z, float w) { return {x, y, z, w}; }
inline uint2 make_uint2(unsigned x, unsigned y) { return {x, y}; }
inline uint4 make_uint4(unsigned x, unsigned y, unsigned z, unsigned w) { return {x, y, z, w}; }

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned x = 1, unsigned y = 1, unsigned z = 1) : x(x), y(y), z(z) {}
};
inline thread_local dim3 threadIdx, blockIdx, blockDim, gridDim;

inline int min(int a, int b) { return a < b ? a : b; }
inline int max(int a, int b) { return a > b ? a : b; }
inline long min(long a, long b) { return a < b ? a : b; }
template <typename To, typename From> To bits_as(From v) {
    static_assert(sizeof(To) == sizeof(From));
    To t;
    memcpy(&t, &v, sizeof(t));
    return t;
}
inline long long __double_as_longlong(double v) { return bits_as<long long>(v); }
inline double __longlong_as_double(long long v) { return bits_as<double>(v); }
inline unsigned __float_as_uint(float v) { return bits_as<unsigned>(v); }
inline float __uint_as_float(unsigned v) { return bits_as<float>(v); }

namespace simt {

constexpr int WAVE = 64;
constexpr size_t STACK = 64 * 1024;
enum State { RUNNING, AT_LANES, AT_BARRIER, DONE };

// Order of the workgroups of a launch.  LATE: the first wavefront of workgroup 1 gets to its
// first barrier, then workgroup 0 runs from start to end, then the rest of workgroup 1.
enum Order { IN_TURN, LATE };
inline Order order = IN_TURN;

// a fiber starts with its context and is resumed with a jump, which takes no system call
struct Item {
    ucontext_t ctx;
    jmp_buf at;
    State state;
    bool started;
    std::vector<char> stack;
};
struct Group {
    std::vector<Item> items;
    std::vector<unsigned long long> lane[2];  // cross-lane values, of even and odd operations
    std::vector<int> nop;                     // operations so far of each work-item
    jmp_buf sched;
    const std::function<void()>* body;
    int cur;
};
inline thread_local Group* group = nullptr;

inline void entry() {
    Group* g = group;
    (*g->body)();
    g->items[g->cur].state = DONE;
    _longjmp(g->sched, 1);
}
inline void wait(State s) {
    Group* g = group;
    Item& it = g->items[g->cur];
    it.state = s;
    if (!_setjmp(it.at)) _longjmp(g->sched, 1);
}
__attribute__((noinline)) inline void resume(Group& g, int i) {
    Item& it = g.items[i];
    g.cur = i;
    threadIdx = dim3(i);
    if (_setjmp(g.sched)) return;
    if (it.started) _longjmp(it.at, 1);
    it.started = true;
    setcontext(&it.ctx);
}

// every work-item of wavefront w to a barrier or its end
inline void run_wave(Group& g, int w) {
    const int n = (int)g.items.size(), i0 = w * WAVE, i1 = i0 + WAVE < n ? i0 + WAVE : n;
    for (;;) {
        for (int i = i0; i < i1; ++i)
            if (g.items[i].state == RUNNING) resume(g, i);
        int lanes = 0, barrier = 0;
        for (int i = i0; i < i1; ++i) {
            lanes += g.items[i].state == AT_LANES;
            barrier += g.items[i].state == AT_BARRIER;
        }
        if (!lanes) return;
        if (barrier) {
            fprintf(stderr, "a wavefront split over a cross-lane operation and a barrier\n");
            abort();
        }
        for (int i = i0; i < i1; ++i)
            if (g.items[i].state == AT_LANES) g.items[i].state = RUNNING;
    }
}

// one workgroup; paused: called when its first wavefront has reached its first barrier
inline void run_group(dim3 grid, dim3 block, unsigned b, const std::function<void()>& body,
                      const std::function<void()>& paused = {}) {
    static thread_local Group g;
    group = &g;
    const int n = (int)(block.x * block.y * block.z), waves = (n + WAVE - 1) / WAVE;
    g.items.resize(n);
    g.lane[0].assign(n, 0);
    g.lane[1].assign(n, 0);
    g.nop.assign(n, 0);
    g.body = &body;
    gridDim = grid;
    blockDim = block;
    blockIdx = dim3(b % grid.x, b / grid.x % grid.y, b / grid.x / grid.y);
    for (Item& it : g.items) {
        it.stack.resize(STACK);
        it.state = RUNNING;
        it.started = false;
        getcontext(&it.ctx);
        it.ctx.uc_stack.ss_sp = it.stack.data();
        it.ctx.uc_stack.ss_size = it.stack.size();
        it.ctx.uc_link = nullptr;
        makecontext(&it.ctx, entry, 0);
    }
    bool first = true;
    for (;;) {
        for (int w = 0; w < waves; ++w) {
            run_wave(g, w);
            if (first && paused) paused();
            first = false;
        }
        bool left = false;
        for (Item& it : g.items)
            if (it.state == AT_BARRIER) {
                it.state = RUNNING;
                left = true;
            }
        if (!left) return;
    }
}

inline void launch(dim3 grid, dim3 block, const std::function<void()>& body) {
    const unsigned nb = grid.x * grid.y * grid.z;
    unsigned b = 0;
    if (order == LATE && nb > 1) {
        // workgroup 0 in a thread of its own: it has its own LDS
        run_group(grid, block, 1, body, [&] { std::thread([&] { run_group(grid, block, 0, body); }).join(); });
        b = 2;
    }
    for (; b < nb; ++b) run_group(grid, block, b, body);
}

// the value that lane from(l) of the wavefront passes
template <typename T, typename F> T exchange(T v, F from) {
    Group* g = group;
    const int i = g->cur, base = i - i % WAVE;
    std::vector<unsigned long long>& slot = g->lane[g->nop[i]++ & 1];
    unsigned long long w = 0;
    memcpy(&w, &v, sizeof(T));
    slot[i] = w;
    wait(AT_LANES);
    const int k = base + (from(i % WAVE) & (WAVE - 1));
    w = slot[k < (int)slot.size() ? k : i];
    memcpy(&v, &w, sizeof(T));
    return v;
}
[[noreturn]] inline void unsupported() {
    fprintf(stderr, "an instruction that the host stand-in does not have\n");
    abort();
}
struct Rsrc {};

}  // namespace simt

inline void __syncthreads() { simt::wait(simt::AT_BARRIER); }
inline void __threadfence() {}
template <typename T> T __shfl_xor(T v, int m) {
    return simt::exchange(v, [m](int l) { return l ^ m; });
}
template <typename T> T __shfl(T v, int lane) {
    return simt::exchange(v, [lane](int) { return lane; });
}
inline int atomicAdd(int* p, int v) {
    const int o = *p;
    *p += v;
    return o;
}
inline int atomicExch(int* p, int v) {
    const int o = *p;
    *p = v;
    return o;
}

#define __builtin_amdgcn_sched_barrier(m) ((void)0)
#define __builtin_amdgcn_s_waitcnt(m) ((void)0)
#define __builtin_amdgcn_update_dpp(old, v, ctrl, rm, bm, bc) simt_dpp(v, ctrl)
inline int simt_dpp(int v, int ctrl) {
    if (ctrl < 0x100)  // quad_perm
        return simt::exchange(v, [ctrl](int l) { return (l & ~3) | ((ctrl >> (2 * (l & 3))) & 3); });
    if (ctrl == 0x140) return simt::exchange(v, [](int l) { return l ^ 15; });  // row_mirror
    if (ctrl == 0x141) return simt::exchange(v, [](int l) { return l ^ 7; });   // row_half_mirror
    simt::unsupported();
}
#define __builtin_amdgcn_readfirstlane(v) (simt::unsupported(), (v))
#define __builtin_amdgcn_alignbit(a, b, n) (simt::unsupported(), (a) + (b))
#define __builtin_amdgcn_global_load_lds(...) simt::unsupported()
#define __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, x, y, z) (simt::unsupported(), (c))
#define __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, x, y, z) (simt::unsupported(), (c))
typedef simt::Rsrc __amdgpu_buffer_rsrc_t;
typedef unsigned simt_u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned simt_u32x4 __attribute__((ext_vector_type(4)));
#define __builtin_amdgcn_make_buffer_rsrc(...) (simt::unsupported(), simt::Rsrc{})
#define __builtin_amdgcn_raw_buffer_load_b128(...) (simt::unsupported(), simt_u32x4{})
#define __builtin_amdgcn_raw_buffer_load_b64(...) (simt::unsupported(), simt_u32x2{})
#define __builtin_amdgcn_raw_buffer_store_b128(...) simt::unsupported()
#define __builtin_amdgcn_raw_buffer_store_b64(...) simt::unsupported()

typedef int hipError_t;
typedef void* hipStream_t;
enum { hipSuccess = 0, hipMemcpyDeviceToHost = 2, hipFuncAttributeMaxDynamicSharedMemorySize = 8 };
inline const char* hipGetErrorString(hipError_t) { return "host"; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
inline hipError_t hipFuncSetAttribute(const void*, int, int) { return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, int, hipStream_t) {
    memcpy(d, s, n);
    return hipSuccess;
}
inline hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
    memset(d, v, n);
    return hipSuccess;
}
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) simt::launch(grid, block, [&] { (kernel)(__VA_ARGS__); })
