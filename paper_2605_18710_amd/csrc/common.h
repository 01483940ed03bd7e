// Shared host/device helpers for the gfx950 kernels and the C-ABI layer.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <stdarg.h>
#include "../../include/mosaic.h"

typedef __bf16 bf16;

// ---------------------------------------------------------------------------- errors
void mosaic_set_error(const char* fmt, ...);

#define MOSAIC_FAIL(code, ...)            \
  do {                                    \
    mosaic_set_error(__VA_ARGS__);        \
    return (code);                        \
  } while (0)

#define MOSAIC_HIP(expr)                                                          \
  do {                                                                            \
    hipError_t e__ = (expr);                                                      \
    if (e__ != hipSuccess) {                                                      \
      mosaic_set_error("%s failed: %s", #expr, hipGetErrorString(e__));           \
      return MOSAIC_EHIP;                                                         \
    }                                                                             \
  } while (0)

#define MOSAIC_TRY(expr)                  \
  do {                                    \
    mosaic_status s__ = (expr);           \
    if (s__ != MOSAIC_OK) return s__;     \
  } while (0)

// Launch check: kernel launches report configuration errors through hipGetLastError.
#define MOSAIC_LAUNCH_CHECK()                                                     \
  do {                                                                            \
    hipError_t e__ = hipGetLastError();                                           \
    if (e__ != hipSuccess) {                                                      \
      mosaic_set_error("kernel launch failed: %s", hipGetErrorString(e__));       \
      return MOSAIC_EHIP;                                                         \
    }                                                                             \
  } while (0)

static inline size_t dtype_size(int32_t dtype) { return dtype == MOSAIC_BF16 ? 2 : 4; }
static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Device properties cached per process.
struct DeviceInfo {
  int cu_count;
  int xcd_count;
  bool ok;
};
mosaic_status mosaic_device_info(DeviceInfo* out);

// Persistent-grid sizing: `quota` CUs times the number of workgroups that fit on a CU,
// capped by the number of work items.  The grid only decides WHICH workgroup computes a
// work item, never how, so results do not depend on it.
static inline int grid_for(int quota, int wg_per_cu, int64_t items) {
  int64_t g = (int64_t)quota * wg_per_cu;
  if (g > items) g = items;
  if (g < 1) g = 1;
  return (int)g;
}

// Grid of a pass over `items` blocks that moves `bytes` in all.  Up to `from` bytes, a persistent grid; above, a
// workgroup per block, started in order: the accesses in flight then lie side by side, where workgroups that stride drift apart over the
// whole tensors.  A plain copy of 1 GiB: 4.5 TB/s by 2048 striding workgroups, 6.1 by one per block.  Such a launch is held to its
// quota by the stream's CU mask alone, so it is made only where there is one (stream_within) or the quota is the device.
constexpr int64_t kSweepBytes = (int64_t)64 << 20;
bool stream_within(hipStream_t s, int quota);      // launcher.hip: whether work on `s` runs on at most `quota` CUs
struct Sweep { int grid; bool in_order; };
static inline Sweep sweep_grid(hipStream_t s, int quota, int64_t items, int64_t bytes, int64_t from = kSweepBytes) {
  if (bytes <= from || !stream_within(s, quota)) return {grid_for(quota, 8, items), false};
  return {(int)(items < (1 << 22) ? items : (1 << 22)), true};        // a launch holds fewer than 2^32 threads; kernels stride past that
}
// Tensors larger than the last-level cache (256 MB) together are read and written past it, by workgroups in order.
constexpr int64_t kPastCacheBytes = (int64_t)256 << 20;

// --------------------------------------------------------------- device-side helpers
#ifdef __HIPCC__
__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16 x) { return (float)x; }
template <typename T> __device__ __forceinline__ T from_f32(float x);
template <> __device__ __forceinline__ float from_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ bf16 from_f32<bf16>(float x) { return (bf16)x; }

// plain accesses, or (PAST) ones that do not stay in the caches
template <bool PAST, typename V> __device__ __forceinline__ V load_from(const V* p) {
  if constexpr (PAST) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool PAST, typename V> __device__ __forceinline__ void store_to(V* p, V v) {
  if constexpr (PAST) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// 16-byte vector of T: 4 floats or 8 bf16.
template <typename T> struct Vec16;
template <> struct Vec16<float> {
  static constexpr int N = 4;
  float4 v;
  typedef __attribute__((ext_vector_type(4))) float v4;
  template <bool PAST = false> __device__ __forceinline__ void load(const float* p) { v = __builtin_bit_cast(float4, load_from<PAST>(reinterpret_cast<const v4*>(p))); }
  template <bool PAST = false> __device__ __forceinline__ void store(float* p) const { store_to<PAST>(reinterpret_cast<v4*>(p), __builtin_bit_cast(v4, v)); }
  __device__ __forceinline__ float get(int i) const { return (&v.x)[i]; }
  __device__ __forceinline__ void set(int i, float f) { (&v.x)[i] = f; }
};
template <> struct Vec16<bf16> {
  static constexpr int N = 8;
  typedef __attribute__((ext_vector_type(8))) __bf16 v8;
  v8 v;
  template <bool PAST = false> __device__ __forceinline__ void load(const bf16* p) { v = load_from<PAST>(reinterpret_cast<const v8*>(p)); }
  template <bool PAST = false> __device__ __forceinline__ void store(bf16* p) const { store_to<PAST>(reinterpret_cast<v8*>(p), v); }
  __device__ __forceinline__ float get(int i) const { return (float)v[i]; }
  __device__ __forceinline__ void set(int i, float f) { v[i] = (bf16)f; }
};

// V consecutive elements as one access: 16 bytes, or a single element for rows that do not start
// on 16-byte boundaries (a caller's tensor may be a slice of a larger buffer).
template <typename T, int V> struct Pack { typedef T type __attribute__((ext_vector_type(V))); };
template <typename T> struct Pack<T, 1> { typedef T type; };
template <typename T, int V> __device__ __forceinline__ float pack_get(const typename Pack<T, V>::type& v, int i) {
  if constexpr (V == 1) return to_f32(v);
  else return (float)v[i];
}
template <typename T, int V> __device__ __forceinline__ void pack_set(typename Pack<T, V>::type& v, int i, float f) {
  if constexpr (V == 1) v = from_f32<T>(f);
  else v[i] = (T)f;
}

__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}
__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, 64));
  return x;
}
#endif
