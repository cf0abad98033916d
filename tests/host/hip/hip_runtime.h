// A wave64 machine on the host, so that the kernels' own sources run under the
// address and undefined-behaviour sanitizers: every lane is a fiber, cross-lane
// operations and barriers are rendezvous, and what stands for device and LDS
// memory is checked to the byte.  One workgroup at a time, waves in turn; the
// lanes of a wave run one after another between rendezvous, so a kernel that
// relies on the order of a wave's LDS operations needs one there.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <type_traits>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))

struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
struct uint2 { uint32_t x, y; };
struct int2 { int32_t x, y; };
struct alignas(16) uint4 { uint32_t x, y, z, w; };
struct float2 { float x, y; };
struct alignas(16) float4 { float x, y, z, w; };
static inline uint2 make_uint2(uint32_t a, uint32_t b) { return {a, b}; }
static inline int2 make_int2(int a, int b) { return {a, b}; }
static inline uint4 make_uint4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) { return {a, b, c, d}; }
static inline float2 make_float2(float a, float b) { return {a, b}; }
static inline float4 make_float4(float a, float b, float c, float d) { return {a, b, c, d}; }

// ---- the machine ------------------------------------------------------------
namespace wave {
extern dim3 thread_idx, block_idx, block_dim, grid_dim;
void launch(const char *name, dim3 g, dim3 b, size_t lds, const std::function<void()> &f);
void sync_wave(const char *what, int line);
void sync_block();
uint64_t live();                       // lanes of the wave that have not ended
char *exchange_buffer();               // the wave's buffer of this operation
int lane();
template <typename T>
const T *exchange(T v, const char *what, int line) {
  static_assert(sizeof(T) <= 64, "");
  char *b = exchange_buffer();
  std::memcpy(b + sizeof(T) * lane(), &v, sizeof(T));
  sync_wave(what, line);
  return reinterpret_cast<const T *>(b);
}
}  // namespace wave
#define threadIdx wave::thread_idx
#define blockIdx wave::block_idx
#define blockDim wave::block_dim
#define gridDim wave::grid_dim

// ---- host runtime -----------------------------------------------------------
typedef int hipError_t;
typedef struct w_stream *hipStream_t;
typedef struct w_event *hipEvent_t;
typedef struct w_graph *hipGraph_t;
typedef struct w_gexec *hipGraphExec_t;
enum { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorInvalidDevice = 101, hipErrorInvalidSymbol = 13, hipErrorUnknown = 999 };
enum { hipMemcpyHostToDevice, hipMemcpyDeviceToHost };
enum { hipEventDisableTiming = 2, hipStreamNonBlocking = 1 };
enum hipDeviceAttribute { hipDeviceAttributeMultiprocessorCount };
enum hipFuncAttr { hipFuncAttributeMaxDynamicSharedMemorySize };
enum hipStreamCaptureMode { hipStreamCaptureModeThreadLocal };
struct hipDeviceProp_t { char gcnArchName[64]; size_t sharedMemPerBlock; };
#define HIP_SYMBOL(x) (x)
static inline hipError_t hipGetLastError() { return 0; }
static inline const char *hipGetErrorName(hipError_t) { return "x"; }
static inline hipError_t hipGetDeviceCount(int *n) { *n = 1; return 0; }
static inline hipError_t hipGetDevice(int *n) { *n = 0; return 0; }
static inline hipError_t hipSetDevice(int) { return 0; }
static inline hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) {
  std::strcpy(p->gcnArchName, "gfx950");
  p->sharedMemPerBlock = 163840;
  return 0;
}
static inline hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute, int) { *v = 4; return 0; }
static inline hipError_t hipFuncSetAttribute(const void *, hipFuncAttr, int) { return 0; }
template <typename F> static inline hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, F, int, size_t) { *n = 2; return 0; }
template <typename T> static inline hipError_t hipMalloc(T **p, size_t n) { *p = (T *)std::malloc(n); return 0; }
static inline hipError_t hipFree(void *p) { std::free(p); return 0; }
static inline hipError_t hipMemcpy(void *d, const void *s, size_t n, int) { std::memcpy(d, s, n); return 0; }
static inline hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, int, hipStream_t) { std::memcpy(d, s, n); return 0; }
template <typename T> static inline hipError_t hipGetSymbolAddress(void **p, T &s) { *p = (void *)&s; return 0; }
static inline hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)std::malloc(1); return 0; }
static inline hipError_t hipStreamDestroy(hipStream_t s) { std::free((void *)s); return 0; }
static inline hipError_t hipStreamSynchronize(hipStream_t) { return 0; }
static inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return 0; }
static inline hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)std::malloc(1); return 0; }
static inline hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
static inline hipError_t hipEventDestroy(hipEvent_t e) { std::free((void *)e); return 0; }
static inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return 0; }
static inline hipError_t hipEventSynchronize(hipEvent_t) { return 0; }
static inline hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t) { *t = 1.0f; return 0; }
static inline hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return 0; }
static inline hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { *g = nullptr; return 0; }
static inline hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, void *, void *, size_t) { return 0; }
static inline hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return 0; }
static inline hipError_t hipGraphDestroy(hipGraph_t) { return 0; }
static inline hipError_t hipGraphExecDestroy(hipGraphExec_t) { return 0; }
#define hipLaunchKernelGGL(k, g, b, l, s, ...) wave::launch(#k, g, b, l, [=] { (k)(__VA_ARGS__); })


// ---- device functions ---------------------------------------------------------
template <typename A, typename B> static inline std::common_type_t<A, B> min(A a, B b) { typedef std::common_type_t<A, B> T; return (T)a < (T)b ? (T)a : (T)b; }
template <typename A, typename B> static inline std::common_type_t<A, B> max(A a, B b) { typedef std::common_type_t<A, B> T; return (T)a > (T)b ? (T)a : (T)b; }
static inline int __popc(uint32_t x) { return __builtin_popcount(x); }
static inline int __popcll(uint64_t x) { return __builtin_popcountll(x); }
static inline float __uint_as_float(uint32_t x) { float f; std::memcpy(&f, &x, 4); return f; }
static inline uint32_t __float_as_uint(float x) { uint32_t f; std::memcpy(&f, &x, 4); return f; }
static inline float __int_as_float(int x) { return __uint_as_float((uint32_t)x); }
static inline int __float_as_int(float x) { return (int)__float_as_uint(x); }
static inline uint32_t __umul24(uint32_t a, uint32_t b) { return (a & 0xFFFFFFu) * (b & 0xFFFFFFu); }
template <typename T> static inline T atomicAdd(T *p, std::common_type_t<T> v) { T o = *p; *p = o + v; return o; }
static inline uint32_t atomicOr(uint32_t *p, uint32_t v) { uint32_t o = *p; *p = o | v; return o; }
static inline uint32_t atomicCAS(uint32_t *p, uint32_t c, uint32_t v) { uint32_t o = *p; if (o == c) *p = v; return o; }
#define __syncthreads() wave::sync_block()
#define __threadfence() ((void)0)
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_wave_barrier() wave::sync_wave("barrier", __LINE__)
#define __builtin_amdgcn_s_waitcnt(...) ((void)0)
#define __builtin_amdgcn_sched_barrier(...) ((void)0)
#define __builtin_amdgcn_sched_group_barrier(...) ((void)0)
template <typename T> static inline T w_readlane(T x, int k, int line) { return wave::exchange(x, "readlane", line)[k & 63]; }
#define __builtin_amdgcn_readlane(x, k) w_readlane((int)(x), (int)(k), __LINE__)
static inline int w_first(int x, int line) { return wave::exchange(x, "readfirstlane", line)[__builtin_ctzll(wave::live())]; }
#define __builtin_amdgcn_readfirstlane(x) w_first((int)(x), __LINE__)
static inline uint64_t w_ballot(bool p, int line) {
  const uint8_t *v = wave::exchange((uint8_t)p, "ballot", line);
  uint64_t m = 0, a = wave::live();
  for (int l = 0; l < 64; ++l) if ((a >> l & 1) && v[l]) m |= 1ull << l;
  return m;
}
#define __ballot(p) w_ballot((p) != 0, __LINE__)
template <typename T> static inline T w_shfl(T x, int src, int line) { const T *v = wave::exchange(x, "shfl", line); return src < 0 || src > 63 ? x : v[src]; }
#define __shfl(x, s, w) w_shfl(x, (s) & 63, __LINE__)
#define __shfl_up(x, d, w) w_shfl(x, wave::lane() - (int)(d), __LINE__)
#define __shfl_xor(x, d, w) w_shfl(x, wave::lane() ^ (int)(d), __LINE__)
#define __shfl_down(x, d, w) w_shfl(x, wave::lane() + (int)(d), __LINE__)
static inline int w_dpp(int old, int src, int ctrl, bool bound, int line) {
  const int *v = wave::exchange(src, "dpp", line);
  const int l = wave::lane();
  int s = -1;
  if (ctrl < 0x100) s = (l & ~3) | (ctrl >> 2 * (l & 3) & 3);
  else if (ctrl == 0x140) s = l ^ 15;
  else if (ctrl == 0x141) s = l ^ 7;
  else if (ctrl > 0x120 && ctrl < 0x130) s = (l & ~15) | ((l - (ctrl & 15)) & 15);
  else if (ctrl == 0x138) s = l - 1;
  else if (ctrl == 0x130) s = l == 63 ? -1 : l + 1;
  else { std::fprintf(stderr, "lane shift %x\n", ctrl); std::abort(); }
  if (s < 0) return bound ? 0 : old;
  return v[s];
}
#define __builtin_amdgcn_update_dpp(o, s, c, rm, bm, b) w_dpp(o, s, c, b, __LINE__)
struct w_u2 { uint32_t v[2]; uint32_t operator[](int i) const { return v[i]; } };
static inline w_u2 w_swap(uint32_t a, uint32_t b, int d, int line) {
  const w_u2 *v = wave::exchange(w_u2{{a, b}}, "swap", line);
  const int l = wave::lane();
  // odd groups of d lanes of a <-> even groups of b
  return w_u2{{(l & d) ? v[l ^ d].v[1] : a, (l & d) ? b : v[l ^ d].v[0]}};
}
#define __builtin_amdgcn_permlane16_swap(a, b, f, c) w_swap(a, b, 16, __LINE__)
#define __builtin_amdgcn_permlane32_swap(a, b, f, c) w_swap(a, b, 32, __LINE__)
static inline uint32_t __builtin_amdgcn_mbcnt_lo(uint32_t m, uint32_t x) { const int l = wave::lane(); return x + __builtin_popcount(l >= 32 ? m : m & ((1u << l) - 1u)); }
static inline uint32_t __builtin_amdgcn_mbcnt_hi(uint32_t m, uint32_t x) { const int l = wave::lane(); return x + (l <= 32 ? 0 : __builtin_popcount(m & ((1u << (l - 32)) - 1u))); }
static inline uint32_t __builtin_amdgcn_ubfe(uint32_t x, uint32_t o, uint32_t w) { return (x >> (o & 31)) & ((1u << w) - 1u); }
static inline int __builtin_amdgcn_sbfe(int x, uint32_t o, uint32_t) { return ((uint32_t)x >> (o & 31) & 1u) ? -1 : 0; }
static inline float __builtin_amdgcn_rcpf(float x) { return 1.0f / x; }
static inline float __builtin_amdgcn_exp2f(float x) { return std::exp2(x); }

// ---- buffers: loads past the range give 0, stores past it are dropped -------------
struct __amdgpu_buffer_rsrc_t { char *base; uint32_t range; };
static inline __amdgpu_buffer_rsrc_t __builtin_amdgcn_make_buffer_rsrc(void *p, short, int n, int) { return {(char *)p, (uint32_t)n}; }
typedef unsigned int w_u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int w_u32x4 __attribute__((ext_vector_type(4)));
template <int N> static inline void w_load(uint32_t *d, __amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s) {
  for (int k = 0; k < N; ++k) {
    const uint64_t o = (uint64_t)v + 4 * k;
    d[k] = 0;
    if (o + 4 <= r.range) std::memcpy(&d[k], r.base + o + s, 4);
  }
}
template <int N> static inline void w_store(const uint32_t *d, __amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s) {
  for (int k = 0; k < N; ++k) {
    const uint64_t o = (uint64_t)v + 4 * k;
    if (o + 4 <= r.range) std::memcpy(r.base + o + s, &d[k], 4);
  }
}
static inline uint32_t __builtin_amdgcn_raw_buffer_load_b32(__amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s, int) { uint32_t d; w_load<1>(&d, r, v, s); return d; }
static inline w_u32x2 __builtin_amdgcn_raw_buffer_load_b64(__amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s, int) { uint32_t d[2]; w_load<2>(d, r, v, s); return w_u32x2{d[0], d[1]}; }
static inline w_u32x4 __builtin_amdgcn_raw_buffer_load_b128(__amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s, int) { uint32_t d[4]; w_load<4>(d, r, v, s); return w_u32x4{d[0], d[1], d[2], d[3]}; }
static inline void __builtin_amdgcn_raw_buffer_store_b32(uint32_t x, __amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s, int) { w_store<1>(&x, r, v, s); }
static inline void __builtin_amdgcn_raw_buffer_store_b64(w_u32x2 x, __amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s, int) { uint32_t d[2] = {x.x, x.y}; w_store<2>(d, r, v, s); }
static inline void __builtin_amdgcn_raw_buffer_store_b128(w_u32x4 x, __amdgpu_buffer_rsrc_t r, uint32_t v, uint32_t s, int) { uint32_t d[4] = {x.x, x.y, x.z, x.w}; w_store<4>(d, r, v, s); }

// ---- matrix cores -------------------------------------------------------------
typedef __bf16 w_bf8 __attribute__((ext_vector_type(8)));
typedef float w_f4 __attribute__((ext_vector_type(4)));
static inline float w_bf(__bf16 x) { uint16_t u; std::memcpy(&u, &x, 2); return __uint_as_float((uint32_t)u << 16); }
static inline w_f4 w_mfma_bf16(w_bf8 a, w_bf8 b, w_f4 c, int line) {
  struct AB { __bf16 a[8], b[8]; } x;
  for (int i = 0; i < 8; ++i) x.a[i] = a[i], x.b[i] = b[i];
  const AB *v = wave::exchange(x, "mfma", line);
  const int l = wave::lane();
  for (int r = 0; r < 4; ++r) {
    float s = c[r];
    for (int k = 0; k < 32; ++k) s += w_bf(v[16 * (k >> 3) + 4 * (l >> 4) + r].a[k & 7]) * w_bf(v[16 * (k >> 3) + (l & 15)].b[k & 7]);
    c[r] = s;
  }
  return c;
}
static inline w_f4 w_mfma_f32(float a, float b, w_f4 c, int line) {
  const float2 *v = wave::exchange(float2{a, b}, "mfma", line);
  const int l = wave::lane();
  for (int r = 0; r < 4; ++r) {
    float s = c[r];
    for (int k = 0; k < 4; ++k) s = std::fma(v[16 * k + 4 * (l >> 4) + r].x, v[16 * k + (l & 15)].y, s);
    c[r] = s;
  }
  return c;
}
#define __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, x, y, z) w_mfma_bf16(a, b, c, __LINE__)
#define __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, x, y, z) w_mfma_f32(a, b, c, __LINE__)
