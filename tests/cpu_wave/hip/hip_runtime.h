// The HIP names that the kernels under test use, for a build of their source files for the
// CPU.  A workgroup's lanes are fibers that run one after another, each up to the next point
// where the hardware would make it wait for others: a barrier, a wave barrier or a cross-lane
// operation.  What a lane writes to LDS for another is there only behind such a point, LDS
// holds garbage when a workgroup starts, and memory outside a buffer (Buffer) faults, so a
// missing wait, an entry that nobody wrote and an index out of range show every time.
// Lanes of a wave must reach the same cross-lane operations (no divergence around them).
#pragma once
#include <sys/mman.h>
#include <ucontext.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __constant__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))
#define __shared__ static __attribute__((section("lds")))
#define hipLaunchKernelGGL(...) ((void)0)   // launched by the tests themselves (emu::launch)

#define amdgpu_waves_per_eu(...) unused

using std::isfinite;
using std::max;
using std::min;

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
struct uint2 { uint32_t x, y; };
struct uint4 { uint32_t x, y, z, w; };
struct float4 { float x, y, z, w; };
struct double2 { double x, y; };
inline uint2 make_uint2(uint32_t a, uint32_t b) { return {a, b}; }
inline uint4 make_uint4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) { return {a, b, c, d}; }
inline float4 make_float4(float a, float b, float c, float d) { return {a, b, c, d}; }
inline double2 make_double2(double a, double b) { return {a, b}; }

// host API of the same files: never reached here
typedef void* hipStream_t;
typedef int hipError_t;
constexpr int hipSuccess = 0, hipMemcpyDeviceToDevice = 3;
#define HIP_SYMBOL(x) (x)
#define EMU_HOST_CALL(name)   \
    template <typename... A>  \
    int name(A&&...) {        \
        abort();              \
    }
EMU_HOST_CALL(hipMalloc)
EMU_HOST_CALL(hipFree)
EMU_HOST_CALL(hipDeviceSynchronize)
EMU_HOST_CALL(hipGetDevice)
EMU_HOST_CALL(hipSetDevice)
EMU_HOST_CALL(hipGetSymbolAddress)
EMU_HOST_CALL(hipMemcpyAsync)
inline int hipGetLastError() { return 0; }

extern char __start_lds[], __stop_lds[];

namespace emu {
inline dim3 threadIdx, blockIdx, blockDim, gridDim;

struct Meet {   // a point that `live` lanes have to reach
    int live = 0, here = 0;
    unsigned turn = 0;
    void check() {
        if (live && here == live) {
            here = 0;
            ++turn;
        }
    }
};
struct Wave {
    Meet meet;
    unsigned op[64] = {};
    const void* kind[2][64];
    alignas(16) char val[2][64][64];   // what every lane brought, by the parity of the operation
};
struct Fiber {
    ucontext_t ctx;
    bool done;
};
inline std::vector<Fiber> fibers;
inline std::vector<Wave> waves;
inline Meet block;
inline ucontext_t main_ctx;
inline unsigned cur, progress;
inline std::function<void()> body;
constexpr size_t STACK = 512 << 10;

inline void yield() { swapcontext(&fibers[cur].ctx, &main_ctx); }
inline void wait(Meet& m) {
    const unsigned t = m.turn;
    ++m.here;
    m.check();
    while (m.turn == t) yield();
    ++progress;
}
// every live lane of the wave brings v; their values by lane, and which lanes are live
template <typename T>
const char (*exchange(const void* kind, const T& v))[64] {
    static_assert(sizeof(T) <= 64, "size");
    Wave& w = waves[cur / 64];
    const unsigned l = cur % 64, s = w.op[l]++ & 1;
    memcpy(w.val[s][l], &v, sizeof v);
    w.kind[s][l] = kind;
    wait(w.meet);
    for (unsigned i = 0; i < 64 && i + cur / 64 * 64 < blockDim.x; ++i)
        if (!fibers[cur / 64 * 64 + i].done && w.op[i] >= w.op[l] && w.kind[s][i] != kind) {
            fprintf(stderr, "lanes %u and %u of a wave meet in different operations\n", l, i);
            exit(3);
        }
    return w.val[s];
}
template <typename T>
T from(const char (*v)[64], int lane) {
    T t;
    memcpy(&t, v[lane & 63], sizeof t);
    return t;
}
inline void entry() {
    body();
    fibers[cur].done = true;
    for (Meet* m : {&waves[cur / 64].meet, &block}) {
        --m->live;
        m->check();
    }
    ++progress;
    for (;;) yield();
}

// f(): the kernel called with its arguments
inline void launch(unsigned grid, unsigned threads, const std::function<void()>& f) {
    static char* stacks = nullptr;
    static unsigned have = 0;
    if (threads > have) {
        stacks = (char*)mmap(nullptr, STACK * threads, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
        have = threads;
    }
    body = f;
    gridDim = dim3(grid);
    blockDim = dim3(threads);
    fibers.resize(threads);
    for (unsigned b = 0; b < grid; ++b) {
        blockIdx = dim3(b, 0, 0);
        memset(__start_lds, 0xAB, __stop_lds - __start_lds);
        waves.assign((threads + 63) / 64, Wave());
        for (unsigned w = 0; w < waves.size(); ++w) waves[w].meet.live = (int)min(64u, threads - 64 * w);
        block = Meet();
        block.live = (int)threads;
        for (unsigned t = 0; t < threads; ++t) {
            getcontext(&fibers[t].ctx);
            fibers[t].ctx.uc_stack.ss_sp = stacks + STACK * t;
            fibers[t].ctx.uc_stack.ss_size = STACK;
            fibers[t].ctx.uc_link = nullptr;
            fibers[t].done = false;
            makecontext(&fibers[t].ctx, entry, 0);
        }
        for (bool left = true; left;) {
            const unsigned before = progress;
            left = false;
            for (unsigned t = 0; t < threads; ++t) {
                if (fibers[t].done) continue;
                cur = t;
                threadIdx = dim3(t, 0, 0);
                swapcontext(&main_ctx, &fibers[t].ctx);
                left = left || !fibers[t].done;
            }
            if (left && progress == before) {
                fprintf(stderr, "workgroup %u: every lane waits for another\n", b);
                exit(3);
            }
        }
    }
}

// n elements that end at a page nobody may touch; 16 GiB of such pages on either side, so that
// any 32-bit index out of range faults
template <typename T>
struct Buffer {
    T* p;
    size_t n;
    explicit Buffer(size_t count, int fill = 0xAB) : n(count) {
        const size_t guard = (size_t)16 << 30, bytes = (n * sizeof(T) + 4095) / 4096 * 4096;
        char* base = (char*)mmap(nullptr, 2 * guard + bytes, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
        if (base == MAP_FAILED || mprotect(base + guard, bytes, PROT_READ | PROT_WRITE)) abort();
        p = (T*)(base + guard + bytes) - n;
        memset((void*)p, fill, n * sizeof(T));
    }
    operator T*() { return p; }
};
}  // namespace emu
using emu::blockDim;
using emu::blockIdx;
using emu::gridDim;
using emu::threadIdx;

// ---- barriers -----------------------------------------------------------------------------
inline void __syncthreads() { emu::wait(emu::block); }
inline int __syncthreads_or(int v) {
    static int any;
    __syncthreads();
    any = 0;
    __syncthreads();
    any |= v;
    __syncthreads();
    return any;
}
inline void __builtin_amdgcn_s_barrier() { __syncthreads(); }
inline void __builtin_amdgcn_wave_barrier() { emu::wait(emu::waves[emu::cur / 64].meet); }
template <typename... A>
void __builtin_amdgcn_fence(A...) {}
inline void __builtin_amdgcn_sched_barrier(int) {}

// ---- cross-lane operations ------------------------------------------------------------------
inline unsigned lane_id() { return emu::cur % 64; }
inline uint64_t __ballot(bool v) {
    static const char id = 0;
    const auto* a = emu::exchange(&id, v);
    uint64_t m = 0;
    for (unsigned i = 0; i < 64 && i + emu::cur / 64 * 64 < blockDim.x; ++i)
        if (!emu::fibers[emu::cur / 64 * 64 + i].done && emu::from<bool>(a, i)) m |= 1ull << i;
    return m;
}
inline bool __any(bool v) { return __ballot(v) != 0; }
inline bool __all(bool v) { return __ballot(!v) == 0; }
template <typename T>
T __shfl(T v, int src, int w = 64) {
    static const char id = 0;
    const int base = (int)lane_id() / w * w;
    return emu::from<T>(emu::exchange(&id, v), base + (src & (w - 1)));
}
template <typename T>
T __shfl_xor(T v, int mask, int w = 64) {
    static const char id = 0;
    return emu::from<T>(emu::exchange(&id, v), (int)lane_id() ^ mask);
}
inline int __builtin_amdgcn_readlane(int v, int l) {
    static const char id = 0;
    return emu::from<int>(emu::exchange(&id, v), l);
}
inline int __builtin_amdgcn_readfirstlane(int v) { return __builtin_amdgcn_readlane(v, 0); }
inline int __builtin_amdgcn_update_dpp(int old, int v, int ctrl, int rows, int banks, bool zero) {
    static const char id = 0;
    const auto* a = emu::exchange(&id, v);
    const int l = (int)lane_id(), row = l & 48, i = l & 15;
    int s = -1;   // the lane read
    if (ctrl < 0x100) s = (l & ~3) | (ctrl >> (2 * (l & 3)) & 3);
    else if (ctrl > 0x110 && ctrl < 0x120) s = i >= ctrl - 0x110 ? l - (ctrl - 0x110) : -1;
    else if (ctrl == 0x140) s = row | (15 - i);
    else if (ctrl == 0x141) s = row | (i & 8) | (7 - (i & 7));
    else if (ctrl == 0x142) s = row ? row - 1 : -1;
    else if (ctrl == 0x143) s = l >= 32 ? 31 : -1;
    else abort();
    if (!(rows >> (l >> 4) & 1) || !(banks >> (i >> 2) & 1)) return old;
    return s >= 0 ? emu::from<int>(a, s) : (zero ? 0 : old);
}
inline int __builtin_amdgcn_ds_swizzle(int v, int p) {
    static const char id = 0;
    const int l = (int)lane_id();
    return emu::from<int>(emu::exchange(&id, v), (l & 32) | (((l & p) | (p >> 5 & 31)) ^ (p >> 10 & 31)));
}
// D = A B + C, 32 x 32 x 16: lane l, half h = l / 32, holds A[l % 32][8h + i], B[8h + i][l % 32] and
// D[8(j/4) + 4h + j%4][l % 32]
template <typename AB, typename C>
C __builtin_amdgcn_mfma_f32_32x32x16_bf16(AB a, AB b, C c, int, int, int) {
    static const char id = 0;
    struct { AB a, b; } v = {a, b};
    const auto* x = emu::exchange(&id, v);
    const int l = (int)lane_id(), h = l >> 5;
    decltype(v) B[2] = {emu::from<decltype(v)>(x, l & 31), emu::from<decltype(v)>(x, (l & 31) + 32)};
    for (int j = 0; j < 16; ++j) {
        const int row = 8 * (j >> 2) + 4 * h + (j & 3);
        for (int k = 0; k < 2; ++k) {
            const auto A = emu::from<decltype(v)>(x, row + 32 * k);
            for (int i = 0; i < 8; ++i) c[j] += (float)A.a[i] * (float)B[k].b[i];
        }
    }
    return c;
}

// ---- atomics and arithmetic -------------------------------------------------------------------
#define __HIP_MEMORY_SCOPE_WAVEFRONT 2
template <typename T, typename V>
T atomicAdd(T* p, V v) {
    const T old = *p;
    *p += (T)v;
    return old;
}
inline int __popc(uint32_t v) { return __builtin_popcount(v); }
inline int __popcll(uint64_t v) { return __builtin_popcountll(v); }
inline int __ffsll(uint64_t v) { return __builtin_ffsll((long long)v); }
inline uint32_t __builtin_amdgcn_bitop3_b32(uint32_t a, uint32_t b, uint32_t c, int table) {
    uint32_t r = 0;
    for (int i = 0; i < 32; ++i) r |= (uint32_t)(table >> ((a >> i & 1) * 4 + (b >> i & 1) * 2 + (c >> i & 1)) & 1) << i;
    return r;
}
inline int __double2hiint(double v) { int64_t b; memcpy(&b, &v, 8); return (int)(b >> 32); }
inline int __double2loint(double v) { int64_t b; memcpy(&b, &v, 8); return (int)b; }
inline double __hiloint2double(int hi, int lo) {
    const uint64_t b = (uint64_t)(uint32_t)hi << 32 | (uint32_t)lo;
    double v;
    memcpy(&v, &b, 8);
    return v;
}
inline double __dmul_rn(double a, double b) { return a * b; }
inline double __dsub_rn(double a, double b) { return a - b; }
inline float __expf(float x) { return expf(x); }
inline float __builtin_amdgcn_rcpf(float x) { return 1.0f / x; }
inline float __builtin_amdgcn_sqrtf(float x) { return sqrtf(x); }
inline float __builtin_amdgcn_logf(float x) { return log2f(x); }
inline float __builtin_amdgcn_exp2f(float x) { return exp2f(x); }
inline float __builtin_amdgcn_sinf(float x) { return sinf(6.28318530717958648f * x); }
inline float __builtin_amdgcn_cosf(float x) { return cosf(6.28318530717958648f * x); }
inline float __builtin_amdgcn_div_fixupf(float q, float, float) { return q; }
