// Host-only stand-in for the HIP device language, used to run the library's
// kernels on the CPU (devsim.cpp): work-items are fibers, wavefront operations
// are rendezvous of 64 of them, LDS copies complete as late (or as early) as
// the code's waits allow, LDS starts out as garbage.
#pragma once

#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstring>
#include <functional>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __align__(n) __attribute__((aligned(n)))
#define __launch_bounds__(...)
#define __shared__ static

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
struct alignas(8) float2 { float x, y; };
struct alignas(16) float4 { float x, y, z, w; };
struct alignas(8) uint2 { uint32_t x, y; };
struct alignas(16) uint4 { uint32_t x, y, z, w; };
struct alignas(16) double2 { double x, y; };
struct alignas(8) int2 { int x, y; };
struct alignas(16) int4 { int x, y, z, w; };
struct alignas(4) ushort2 { uint16_t x, y; };
struct alignas(8) ushort4 { uint16_t x, y, z, w; };
inline float2 make_float2(float a, float b) { return {a, b}; }
inline float4 make_float4(float a, float b, float c, float d) { return {a, b, c, d}; }
inline uint2 make_uint2(uint32_t a, uint32_t b) { return {a, b}; }
inline uint4 make_uint4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) { return {a, b, c, d}; }
inline int4 make_int4(int a, int b, int c, int d) { return {a, b, c, d}; }
inline double2 make_double2(double a, double b) { return {a, b}; }

typedef int hipError_t;
enum { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorOutOfMemory = 2, hipErrorNotSupported = 801, hipErrorInvalidSymbol = 13 };
struct ihipStream_t;
struct ihipEvent_t;
struct ihipGraph;
struct hipGraphExec;
typedef ihipStream_t *hipStream_t;
typedef ihipEvent_t *hipEvent_t;
typedef ihipGraph *hipGraph_t;
typedef hipGraphExec *hipGraphExec_t;
typedef void *hipGraphNode_t;
enum hipStreamCaptureMode { hipStreamCaptureModeGlobal = 0, hipStreamCaptureModeThreadLocal = 1,
                            hipStreamCaptureModeRelaxed = 2 };
enum hipDeviceAttribute_t { hipDeviceAttributeMultiprocessorCount = 63 };
constexpr unsigned hipStreamNonBlocking = 1, hipEventDisableTiming = 2;
inline hipError_t hipGetDevice(int *d) { *d = 0; return 0; }
inline hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return 0; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)1; return 0; }
inline hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)1; return 0; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)1; return 0; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return 0; }
inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return 0; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return 0; }
inline hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0; return 0; }
inline hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return 1; }
inline hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return 1; }
inline hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return 1; }
inline hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return 1; }
inline hipError_t hipGraphDestroy(hipGraph_t) { return 0; }
inline hipError_t hipGraphExecDestroy(hipGraphExec_t) { return 0; }
inline hipError_t hipGetLastError() { return 0; }
inline const char *hipGetErrorString(hipError_t) { return "error"; }

namespace sim {

struct Lane {
    void *sp;
    dim3 tid;
    int wave, lane;
    long gen;  // wavefront rendezvous passed
    int state; // 0 runnable, 1 at a rendezvous, 2 at the barrier, 3 done
};
extern Lane *cur;
extern dim3 block, blocks, threads;
extern bool compute;  // false: matrix instructions leave their accumulator alone

void launch(dim3 grid, dim3 blk, size_t lds, const std::function<void()> &f, const char *name);
void lds(void *p, size_t bytes);  // an LDS array of the running work-group
unsigned char *dynamic_lds();
char *meet(const void *v, size_t bytes);  // wavefront rendezvous: the 64 lanes' values
void barrier();
void wait(int vm);  // at most vm LDS copies of this wavefront outstanding
void copy(const void *src, void *dst, int bytes);  // LDS copy of `bytes` per lane

template <typename T> struct All { const T *p; const T &operator[](int i) const { return p[i]; } };
template <typename T> inline All<T> all(const T &v) { return {(const T *)meet(&v, sizeof(T))}; }
inline void wave_sync() { const char c = 0; meet(&c, 1); }
inline int lane() { return cur->lane; }

} // namespace sim

#define threadIdx (sim::cur->tid)
#define blockIdx (sim::block)
#define gridDim (sim::blocks)
#define blockDim (sim::threads)
#define hipLaunchKernelGGL(K, G, B, L, S, ...) \
    ((void)(S), sim::launch(G, B, L, [=]() { K(__VA_ARGS__); }, #K))

inline void __syncthreads() { sim::barrier(); }
template <typename T> inline T __shfl_xor(T v, int m, int = 64) { return sim::all(v)[sim::lane() ^ m]; }
template <typename T> inline T __shfl(T v, int l, int = 64) { return sim::all(v)[l & 63]; }
inline uint64_t __ballot(int p) {
    const auto a = sim::all(p);
    uint64_t m = 0;
    for (int i = 0; i < 64; ++i)
        m |= (uint64_t)(a[i] != 0) << i;
    return m;
}
inline int __popcll(uint64_t v) { return __builtin_popcountll(v); }
inline float __uint_as_float(uint32_t u) { return __builtin_bit_cast(float, u); }
inline uint32_t __float_as_uint(float f) { return __builtin_bit_cast(uint32_t, f); }
inline int __float_as_int(float f) { return __builtin_bit_cast(int, f); }
inline float __int_as_float(int i) { return __builtin_bit_cast(float, i); }
inline long long __double_as_longlong(double d) { return __builtin_bit_cast(long long, d); }
inline double __longlong_as_double(long long d) { return __builtin_bit_cast(double, d); }
inline float __expf(float x) { return std::exp(x); }
template <typename A, typename B> inline auto min(A a, B b) { typedef decltype(a + b) C; return (C)a < (C)b ? (C)a : (C)b; }
template <typename A, typename B> inline auto max(A a, B b) { typedef decltype(a + b) C; return (C)a > (C)b ? (C)a : (C)b; }

// ---- gfx950 builtins -------------------------------------------------------
namespace sim {
typedef float f16 __attribute__((ext_vector_type(16)));
inline int acc_row(int v) { return 8 * (v >> 2) + 4 * (lane() >> 5) + (v & 3); }
inline float bf(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
struct AB { uint16_t a[8], b[8]; };
template <typename V> inline f16 mfma_bf16(V a, V b, f16 c) {
    if (!compute)
        return c;
    AB v;
    memcpy(v.a, &a, 16);
    memcpy(v.b, &b, 16);
    const auto w = all(v);
    for (int r = 0; r < 16; ++r) {
        double s = c[r];
        for (int h = 0; h < 2; ++h)
            for (int k = 0; k < 8; ++k)
                s += (double)bf(w[acc_row(r) + 32 * h].a[k]) * bf(w[(lane() & 31) + 32 * h].b[k]);
        c[r] = (float)s;
    }
    return c;
}
struct ab { float a, b; };
inline f16 mfma_f32(float a, float b, f16 c) {
    if (!compute)
        return c;
    const auto w = all(ab{a, b});
    for (int r = 0; r < 16; ++r) {
        float s = c[r];
        for (int h = 0; h < 2; ++h)
            s = std::fma(w[acc_row(r) + 32 * h].a, w[(lane() & 31) + 32 * h].b, s);
        c[r] = s;
    }
    return c;
}
typedef short s4 __attribute__((ext_vector_type(4)));
template <typename P> inline s4 tr16(P p) {
    s4 mine, out;
    memcpy(&mine, (const void *)p, 8);
    const auto w = all(mine);
    const int g = lane() & ~15, i = lane() & 15;
    for (int j = 0; j < 4; ++j)
        out[j] = w[g + 4 * j + (i >> 2)][i & 3];
    return out;
}
inline int dpp(int v, int ctrl) {  // row_shl:N, lanes past the row's end take 0
    const auto w = all(v);
    const int n = ctrl - 0x100, i = lane();
    return (i & 15) + n < 16 ? w[i + n] : 0;
}
typedef unsigned u2 __attribute__((ext_vector_type(2)));
inline u2 swap_halves(unsigned a, unsigned b, int n) {
    struct P { unsigned a, b; };
    const auto w = all(P{a, b});
    const int l = lane();
    return (l & n) ? u2{w[l - n].b, b} : u2{a, w[l + n].a};
}
inline void copy_rsrc(const int *r, uint32_t voff, uint32_t soff, void *dst, int bytes) {
    const uint64_t base = (uint32_t)r[0] | (uint64_t)(r[1] & 0xffff) << 32;
    copy((const char *)base + (uint64_t)voff + soff, dst, bytes);
}
} // namespace sim
#define __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, x, y, z) sim::mfma_bf16(a, b, c)
#define __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, x, y, z) sim::mfma_f32(a, b, c)
#define __builtin_amdgcn_ds_read_tr16_b64_v4bf16(p) sim::tr16(p)
#define __builtin_amdgcn_readfirstlane(v) (sim::all(v)[0])
#define __builtin_amdgcn_readlane(v, l) (sim::all(v)[l])
#define __builtin_amdgcn_ds_bpermute(a, v) (sim::all(v)[((a) >> 2) & 63])
#define __builtin_amdgcn_update_dpp(old, v, ctrl, rm, bm, bc) sim::dpp(v, ctrl)
#define __builtin_amdgcn_permlane32_swap(a, b, x, y) sim::swap_halves(a, b, 32)
#define __builtin_amdgcn_permlane16_swap(a, b, x, y) sim::swap_halves(a, b, 16)
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_wave_barrier() sim::wave_sync()
#define __builtin_amdgcn_s_waitcnt(imm) sim::wait(((imm) & 15) | (((imm) >> 14) & 3) << 4)
#define __builtin_amdgcn_global_load_lds(s, d, n, o, x) sim::copy((const void *)(s), (void *)(d), n)
