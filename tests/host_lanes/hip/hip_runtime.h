// The HIP names that csrc/ uses, for a build of the library on the CPU: every lane of a workgroup
// is a fiber on one thread, device memory is malloc'd to the byte (an address sanitizer then sees
// every access outside it) and filled with NaN.  Wave operations wait for all lanes of the wave
// that are still running, barriers for all of the workgroup; anything else ends the program.
#pragma once
#include <math.h>
#include <sanitizer/asan_interface.h>
#include <sanitizer/common_interface_defs.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

#include <initializer_list>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static
#define __align__(n) __attribute__((aligned(n)))

struct alignas(8) float2 { float x, y; };
struct alignas(16) double2 { double x, y; };
inline float2 make_float2(float a, float b) { return {a, b}; }
inline double2 make_double2(double a, double b) { return {a, b}; }
inline int min(int a, int b) { return a < b ? a : b; }
inline float __uint_as_float(uint32_t u) { return __builtin_bit_cast(float, u); }

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};

namespace lanes {

// Saves the callee-saved registers and the stack pointer in *from, goes on at to (System V x86-64;
// swapcontext's system calls took most of the time).
asm(".pushsection .text\n.weak lanes_switch\n.type lanes_switch,@function\nlanes_switch:\n"
    "push %rbp\npush %rbx\npush %r12\npush %r13\npush %r14\npush %r15\n"
    "mov %rsp, (%rdi)\nmov %rsi, %rsp\n"
    "pop %r15\npop %r14\npop %r13\npop %r12\npop %rbx\npop %rbp\nret\n.popsection\n");
extern "C" void lanes_switch(void** from, void* to);

struct Fiber {
    void* sp = nullptr;
    char* stack = nullptr;
    void* fake = nullptr;
    dim3 tid;
    enum { kRun, kWave, kBlock, kDone } state = kDone;
    unsigned op = 0;  // wave operations so far
};
constexpr size_t kStack = 256 << 10;
constexpr int kMaxLanes = 1024;

inline Fiber pool[kMaxLanes];
inline void* home_sp;
inline void* home_fake;
inline const void* home_bottom;
inline size_t home_size;
inline int cur;             // lane that runs
inline int n_lanes;
inline dim3 block, grid, bid;
inline void (*body)(void*);
inline void* body_arg;
inline uint64_t slot[2][kMaxLanes];  // what each lane brings to its current wave operation
inline unsigned tag[2][kMaxLanes];    // and the number of that operation

[[noreturn]] inline void fail(const char* what) {
    fprintf(stderr, "lanes: %s (workgroup %u %u)\n", what, bid.x, bid.y);
    abort();
}

inline void yield(int state) {
    Fiber& f = pool[cur];
    f.state = (decltype(f.state))state;
    __sanitizer_start_switch_fiber(state == Fiber::kDone ? nullptr : &f.fake, home_bottom, home_size);
    lanes_switch(&f.sp, home_sp);
    __sanitizer_finish_switch_fiber(f.fake, nullptr, nullptr);
}

inline void entry() {
    __sanitizer_finish_switch_fiber(nullptr, &home_bottom, &home_size);
    body(body_arg);
    yield(Fiber::kDone);
}

// Brings v to the lanes of this wave; returns where theirs are (valid until the second next).
inline const uint64_t* exchange(uint64_t v) {
    Fiber& f = pool[cur];
    const int p = ++f.op & 1;
    slot[p][cur] = v;
    tag[p][cur] = f.op;
    yield(Fiber::kWave);
    return slot[p] + cur / 64 * 64;
}
// whether lane l of this wave took part in the operation
inline bool there(int l) { return l >= 0 && l < 64 && tag[pool[cur].op & 1][cur / 64 * 64 + l] == pool[cur].op; }

inline void run_workgroup() {
    for (int i = 0; i < n_lanes; ++i) {
        Fiber& f = pool[i];
        if (!f.stack)
            f.stack = (char*)mmap(nullptr, kStack, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
        // six registers, the entry, and a return address that keeps the stack aligned
        void** top = (void**)(f.stack + kStack) - 1;
        *top = nullptr;
        *--top = (void*)entry;
        f.sp = top - 6;
        f.state = Fiber::kRun;
        f.op = 0;
        f.tid = dim3(i % block.x, i / block.x % block.y, i / (block.x * block.y));
        tag[0][i] = tag[1][i] = 0;
    }
    for (;;) {
        int done = 0, at_block = 0;
        bool moved = false;
        for (int w0 = 0; w0 < n_lanes; w0 += 64) {
            const int w1 = min(w0 + 64, n_lanes);
            int wave = 0, other = 0;
            for (int i = w0; i < w1; ++i) {
                Fiber& f = pool[i];
                if (f.state == Fiber::kRun) {
                    cur = i;
                    __sanitizer_start_switch_fiber(&home_fake, f.stack, kStack);
                    lanes_switch(&home_sp, f.sp);
                    __sanitizer_finish_switch_fiber(home_fake, nullptr, nullptr);
                    moved = true;
                }
                if (f.state == Fiber::kDone) ++done;
                else if (f.state == Fiber::kBlock) ++at_block, ++other;
                else ++wave;
            }
            if (wave && other) fail("lanes of one wave at a wave operation and at a barrier");
            if (wave)
                for (int i = w0; i < w1; ++i)
                    if (pool[i].state == Fiber::kWave) pool[i].state = Fiber::kRun;
            moved = moved || wave;
        }
        if (done == n_lanes) return;
        if (at_block && at_block == n_lanes) {
            for (int i = 0; i < n_lanes; ++i) pool[i].state = Fiber::kRun;
        } else if (!moved) {
            fail("a barrier that part of the workgroup does not reach");
        }
    }
}

struct Launch {
    Launch(dim3 g, dim3 b, size_t = 0, void* = nullptr) {
        grid = g;
        block = b;
        n_lanes = (int)(b.x * b.y * b.z);
        if (n_lanes > kMaxLanes || !n_lanes || !g.x || !g.y || !g.z) fail("launch shape");
    }
    template <class K, class... A>
    void operator()(K kernel, A... args) {
        auto call = [&] { kernel(args...); };
        body = [](void* p) { (*(decltype(call)*)p)(); };
        body_arg = &call;
        for (unsigned y = 0; y < grid.y; ++y)
            for (unsigned x = 0; x < grid.x; ++x) {
                bid = dim3(x, y, 0);
                run_workgroup();
            }
    }
};

template <class T>
uint64_t bits(T v) {
    uint64_t u = 0;
    memcpy(&u, &v, sizeof(T));
    return u;
}
template <class T>
T from(uint64_t u) {
    T v;
    memcpy(&v, &u, sizeof(T));
    return v;
}
template <class T>
T read_lane(T v, int l) {
    const uint64_t* s = exchange(bits(v));
    if (!there(l)) fail("read of a lane that is not there");
    return from<T>(s[l]);
}
template <class T>
T read_first(T v) {
    const uint64_t* s = exchange(bits(v));
    int l = 0;
    while (!there(l)) ++l;
    return from<T>(s[l]);
}
template <class T>
T shfl_xor(T v, int o) {
    const uint64_t* s = exchange(bits(v));
    const int l = (cur & 63) ^ o;
    if (!there(l)) fail("shuffle with a lane that is not there");
    return from<T>(s[l]);
}
inline bool any(bool v) {
    const uint64_t* s = exchange(v);
    bool r = false;
    for (int l = 0; l < 64; ++l) r = r || (there(l) && s[l]);
    return r;
}
typedef double dbl4 __attribute__((ext_vector_type(4)));
// lane l brings A[l % 16][l / 16] and B[l / 16][l % 16]; element v of D is D[l / 16 + 4 v][l % 16]
inline dbl4 mfma_f64(double a, double b, dbl4 d) {
    double A[64], B[64];
    const int l = cur & 63;
    const uint64_t* s = exchange(bits(a));
    for (int i = 0; i < 64; ++i) {
        if (!there(i)) fail("matrix instruction without a lane");
        A[i] = from<double>(s[i]);
    }
    s = exchange(bits(b));
    for (int i = 0; i < 64; ++i) B[i] = from<double>(s[i]);
    for (int v = 0; v < 4; ++v)
        for (int k = 0; k < 4; ++k) d[v] += A[16 * k + l / 16 + 4 * v] * B[16 * k + l % 16];
    return d;
}

}  // namespace lanes

#define threadIdx (lanes::pool[lanes::cur].tid)
#define blockIdx (lanes::bid)
#define blockDim (lanes::block)
#define gridDim (lanes::grid)
#define __syncthreads() lanes::yield(lanes::Fiber::kBlock)
#define __any(p) lanes::any(p)
#define __shfl_xor(v, o, w) lanes::shfl_xor(v, o)
#define __builtin_amdgcn_readfirstlane(v) lanes::read_first(v)
#define __builtin_amdgcn_readlane(v, l) lanes::read_lane(v, l)
#define __builtin_amdgcn_sched_barrier(m) ((void)0)
#define __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, d, x, y, z) lanes::mfma_f64(a, b, d)

typedef int hipError_t;
typedef void* hipStream_t;
enum { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorOutOfMemory = 2 };
enum hipMemcpyKind { hipMemcpyHostToDevice, hipMemcpyDeviceToHost, hipMemcpyDeviceToDevice };
#define HIP_SYMBOL(s) (s)
inline hipError_t hipMalloc(void** p, size_t n) {
    *p = aligned_alloc(256, (n + 255) / 256 * 256);
    if (!*p) return hipErrorOutOfMemory;
    memset(*p, 0xff, n);
    // the rounding up belongs to nobody
    __asan_poison_memory_region((char*)*p + n, (n + 255) / 256 * 256 - n);
    return hipSuccess;
}
inline hipError_t hipFree(void* p) { free(p); return hipSuccess; }
inline hipError_t hipHostMalloc(void** p, size_t n) { *p = malloc(n); return *p ? hipSuccess : hipErrorOutOfMemory; }
inline hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
inline hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    memcpy(d, s, n);
    return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
inline hipError_t hipGetSymbolAddress(void** p, void* s) { *p = s; return hipSuccess; }
