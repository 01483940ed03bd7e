// Bandwidth-bound kernels of the module step: LayerNorm / RMSNorm forward and backward
// (with fused residual add and fixed-order column reductions), GELU / SwiGLU forward and
// backward, MSE loss and gradient, column sums for bias gradients, and the stem kernels
// (patch unfold, position table).
//
// All reductions run in an order fixed by the problem shape alone: persistent grids only
// decide which workgroup handles a work item, so results are bit-identical for any quota.
#include "activations.h"
#include <algorithm>
#include <type_traits>
#include "kernels.h"

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

// ------------------------------------------------------------------------ norm forward
// One wave per row; the row lives in registers (NV 16-byte vectors per lane), so x is
// read from HBM once.  LayerNorm: biased variance around the mean; RMSNorm: mean square.
template <typename T, int NORM, int NV>
__global__ __launch_bounds__(kThreads) void norm_fwd_kernel(
    const T* __restrict__ x, const T* __restrict__ gamma, const T* __restrict__ beta,
    T* __restrict__ y, float* __restrict__ stats, int64_t rows, int h, float eps) {
  constexpr int VN = Vec16<T>::N;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float inv_h = 1.0f / (float)h;
  for (int64_t row = (int64_t)blockIdx.x * kWaves + wave; row < rows;
       row += (int64_t)gridDim.x * kWaves) {
    Vec16<T> v[NV];
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int c = (j * 64 + lane) * VN;
      if (c < h) {
        v[j].load(x + row * h + c);
#pragma unroll
        for (int i = 0; i < VN; ++i) s += (NORM == MOSAIC_LAYERNORM) ? v[j].get(i) : v[j].get(i) * v[j].get(i);
      }
    }
    s = wave_sum(s);
    float mean = 0.f, rstd;
    if (NORM == MOSAIC_LAYERNORM) {
      mean = s * inv_h;
      float q = 0.f;
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        const int c = (j * 64 + lane) * VN;
        if (c < h) {
#pragma unroll
          for (int i = 0; i < VN; ++i) { const float dlt = v[j].get(i) - mean; q += dlt * dlt; }
        }
      }
      q = wave_sum(q);
      rstd = 1.0f / sqrtf(q * inv_h + eps);
    } else {
      rstd = 1.0f / sqrtf(s * inv_h + eps);
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int c = (j * 64 + lane) * VN;
      if (c < h) {
        Vec16<T> g, b, o;
        g.load(gamma + c);
        if (NORM == MOSAIC_LAYERNORM) b.load(beta + c);
#pragma unroll
        for (int i = 0; i < VN; ++i) {
          float r = (v[j].get(i) - mean) * rstd * g.get(i);
          if (NORM == MOSAIC_LAYERNORM) r += b.get(i);
          o.set(i, r);
        }
        o.store(y + row * h + c);
      }
    }
    if (lane == 0) { stats[row * 2] = mean; stats[row * 2 + 1] = rstd; }
  }
}

// ------------------------------------------------------------------------ column sums
// Partial column sums of a row partition: a lane owns V columns and adds the rows in ascending order, ONCE of them requested
// together (request(row, column)) and then used (use(what was requested, row, column, sums)).  A wave takes 64 * V columns
// of a partition; with QUARTERS (colsum_quarters says where) the four waves of a workgroup take a quarter of its rows each, and
// the four sums are added in the order of the rows.
// block, blocks: this workgroup's number among those that share the pass.
template <int V, int ONCE, bool QUARTERS, typename Request, typename Use>
__device__ __forceinline__ void column_sums(int block, int blocks, int64_t rows, int64_t n, int rp, int np, int ctiles, float* __restrict__ partial,
                                            const Request& request, const Use& use) {
  static_assert(!QUARTERS || V % 4 == 0, "the quarters' sums pass through LDS in pieces of four");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t items = (int64_t)np * ctiles, step = QUARTERS ? blocks : (int64_t)blocks * kWaves;
  for (int64_t it = QUARTERS ? block : (int64_t)block * kWaves + wave; it < items; it += step) {
    const int p = (int)(it / ctiles), ct = (int)(it - (int64_t)p * ctiles);
    const int64_t c = ((int64_t)ct * 64 + lane) * V;
    int64_t r = (int64_t)p * rp, r1 = r + rp < rows ? r + rp : rows;
    if constexpr (QUARTERS) {
      const int64_t per = (r1 - r + 3) >> 2;
      r += wave * per;
      r1 = r + per < r1 ? r + per : r1;
    }
    float acc[V] = {};
    if (c < n) {
      decltype(request(r, c)) q[ONCE];
      for (; r + ONCE <= r1; r += ONCE) {
#pragma unroll
        for (int u = 0; u < ONCE; ++u) q[u] = request(r + u, c);
#pragma unroll
        for (int u = 0; u < ONCE; ++u) use(q[u], r + u, c, acc);
      }
      if (r < r1) {
#pragma unroll
        for (int u = 0; u < ONCE - 1; ++u) if (r + u < r1) q[u] = request(r + u, c);
#pragma unroll
        for (int u = 0; u < ONCE - 1; ++u) if (r + u < r1) use(q[u], r + u, c, acc);
      }
    }
    if constexpr (QUARTERS) {
      __shared__ float4 red[3][V / 4][64];
      if (wave > 0) {
#pragma unroll
        for (int j = 0; j < V / 4; ++j) red[wave - 1][j][lane] = make_float4(acc[4 * j], acc[4 * j + 1], acc[4 * j + 2], acc[4 * j + 3]);
      }
      __syncthreads();
      if (wave == 0) {
#pragma unroll
        for (int j = 0; j < V / 4; ++j)
#pragma unroll
          for (int w = 0; w < 3; ++w) { const float4 o = red[w][j][lane]; acc[4 * j] += o.x; acc[4 * j + 1] += o.y; acc[4 * j + 2] += o.z; acc[4 * j + 3] += o.w; }
      }
      __syncthreads();
    }
    if (c < n && (!QUARTERS || wave == 0)) {
#pragma unroll
      for (int k = 0; k < V; ++k) partial[(int64_t)p * n + c + k] = acc[k];
    }
  }
}

template <typename T, bool QUARTERS>
__device__ __forceinline__ void plain_column_sums(int block, int blocks, const T* __restrict__ X, float* __restrict__ partial, int64_t rows, int64_t n, int rp,
                                                  int np, int ctiles) {
  constexpr int V = Vec16<T>::N;
  typedef typename Pack<T, V>::type vec;
  column_sums<V, QUARTERS ? 4 : 8, QUARTERS>(block, blocks, rows, n, rp, np, ctiles, partial, [&](int64_t r, int64_t c) { return *reinterpret_cast<const vec*>(X + r * n + c); },
                           [&](const vec& x, int64_t, int64_t, float (&acc)[V]) {
#pragma unroll
                             for (int k = 0; k < V; ++k) acc[k] += pack_get<T, V>(x, k);
                           });
}
// The first `blocks` workgroups of a launch that takes a ColSumJob along form its sums; true in those.  A pass of its own costs a launch: layers of
// 1568 rows, width 768 (two; three such passes) 480.0 -> 473.4 us, projector 768 -> 2048 117.1 -> 114.5, 9216 rows, width 1024, 1071 -> 1063.
struct Along { ColSumJob job; int blocks; };
template <typename T>
__device__ __forceinline__ bool sums_along(const Along& a) {
  if ((int)blockIdx.x >= a.blocks) return false;
  plain_column_sums<T, false>(blockIdx.x, a.blocks, (const T*)a.job.X, a.job.partial, a.job.rows, a.job.n, a.job.rp, a.job.np, a.job.ctiles);
  return true;
}

// ----------------------------------------------------------------------- norm backward
// dx: one wave per row, the row of x and dy held in registers (read once), optional
// residual added on the way out.
template <typename T, int NORM, int NV>
__global__ __launch_bounds__(kThreads) void norm_bwd_dx_kernel(
    const T* __restrict__ x, const T* __restrict__ gamma, const float* __restrict__ stats,
    const T* __restrict__ dy, const T* __restrict__ R, T* __restrict__ dx, int64_t rows, int h) {
  constexpr int VN = Vec16<T>::N;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float inv_h = 1.0f / (float)h;
  Vec16<T> g[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int c = (j * 64 + lane) * VN;
    if (c < h) g[j].load(gamma + c);
  }
  for (int64_t row = (int64_t)blockIdx.x * kWaves + wave; row < rows; row += (int64_t)gridDim.x * kWaves) {
    const float mean = stats[row * 2], rstd = stats[row * 2 + 1];
    Vec16<T> xv[NV], dv[NV];
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int c = (j * 64 + lane) * VN;
      if (c < h) {
        xv[j].load(x + row * h + c);
        dv[j].load(dy + row * h + c);
#pragma unroll
        for (int i = 0; i < VN; ++i) {
          const float t = dv[j].get(i) * g[j].get(i);
          if (NORM == MOSAIC_LAYERNORM) {
            const float xh = (xv[j].get(i) - mean) * rstd;
            s1 += t; s2 += t * xh;
          } else {
            s2 += t * xv[j].get(i);
          }
        }
      }
    }
    if (NORM == MOSAIC_LAYERNORM) s1 = wave_sum(s1) * inv_h;
    s2 = wave_sum(s2) * inv_h;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int c = (j * 64 + lane) * VN;
      if (c < h) {
        Vec16<T> o, rv;
        if (R) rv.load(R + row * h + c);
#pragma unroll
        for (int i = 0; i < VN; ++i) {
          const float xr = xv[j].get(i);
          const float t = dv[j].get(i) * g[j].get(i);
          float r;
          if (NORM == MOSAIC_LAYERNORM) r = (t - s1 - (xr - mean) * rstd * s2) * rstd;
          else r = rstd * t - rstd * rstd * rstd * xr * s2;
          if (R) r += rv.get(i);
          o.set(i, r);
        }
        o.store(dx + row * h + c);
      }
    }
  }
}

// dx and the dgamma / dbeta partial sums in one pass over x and dy.  Work item = row
// partition p (rp rows; rp depends on the row count alone).  Wave w of the workgroup takes
// rows r0+w, r0+w+4, ... in ascending order, holds the row of x and dy in registers, writes
// dx and adds dy*xhat (and dy) into per-lane column accumulators.  The four waves'
// accumulators are added in wave order through LDS, one 64-lane column slab at a time, and
// land in scratch[p][2][h]; col_reduce_kernel adds the partitions in a fixed order.
// A row's x, dy and residual are requested together: with the residual behind the row's sums its latency stood alone, two waves to a SIMD.
// 32768 x 4096 RMSNorm 296 -> 226 us (4.75 TB/s), LayerNorm 321 -> 243, 8192 x 2048 30.7 -> 30.0 and 41.7 -> 38.4; on 64 CUs 956 -> 567, 1060 -> 672,
// 61.3 -> 48.2, 126.8 -> 96.5.  The next row requested under the current one gains nothing more and costs small calls up to 3 us.
// CS: the column sums of the values written to dx (as stored, after rounding) are formed the
// same way in a third slab, scratch[p][3][h]: dx is the output gradient of the linear layer in
// front of the residual branch, so this is that layer's bias gradient, without another pass.
// EARLY: the residual with the row.  norm_bwd_tight names the kernels whose waves per SIMD its registers halve (or take from four to three).
template <typename T, int NORM, int NV>
constexpr bool norm_bwd_tight() {
  constexpr bool ln = NORM == MOSAIC_LAYERNORM;
  return std::is_same<T, float>::value ? (ln ? NV == 3 || NV == 8 : NV == 10) : !ln && (NV == 3 || NV == 5);
}
template <typename T, int NORM, int NV, bool CS = false, bool EARLY = true>
__global__ __launch_bounds__(kThreads) void norm_bwd_fused_kernel(
    const T* __restrict__ x, const T* __restrict__ gamma, const float* __restrict__ stats,
    const T* __restrict__ dy, const T* __restrict__ R, T* __restrict__ dx, float* __restrict__ scratch,
    int64_t rows, int h, int rp, int np, Along along) {
  if (sums_along<T>(along)) return;
  constexpr int VN = Vec16<T>::N;
  constexpr int NSUM = (NORM == MOSAIC_LAYERNORM) ? 2 : 1;
  constexpr int NSLAB = CS ? 3 : 2;                    // slabs per partition in scratch
  __shared__ float red[kWaves - 1][NSUM + (CS ? 1 : 0)][64 * VN];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float inv_h = 1.0f / (float)h;
  Vec16<T> g[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int c = (j * 64 + lane) * VN;
    if (c < h) g[j].load(gamma + c);
  }
  for (int p = (int)blockIdx.x - along.blocks; p < np; p += (int)gridDim.x - along.blocks) {
    float ag[NV][VN], ab[NSUM == 2 ? NV : 1][VN], ax[CS ? NV : 1][VN];
#pragma unroll
    for (int j = 0; j < NV; ++j)
#pragma unroll
      for (int i = 0; i < VN; ++i) { ag[j][i] = 0.f; if (NSUM == 2) ab[j][i] = 0.f; if (CS) ax[j][i] = 0.f; }
    const int64_t r0 = (int64_t)p * rp;
    const int64_t r1 = (r0 + rp < rows) ? r0 + rp : rows;
    for (int64_t row = r0 + wave; row < r1; row += kWaves) {
      const float mean = stats[row * 2], rstd = stats[row * 2 + 1];
      Vec16<T> xv[NV], dv[NV], rv[EARLY ? NV : 1];
      float s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        const int c = (j * 64 + lane) * VN;
        if (c < h) {
          xv[j].load(x + row * h + c);
          dv[j].load(dy + row * h + c);
          if (EARLY && R) rv[EARLY ? j : 0].load(R + row * h + c);
        }
      }
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        const int c = (j * 64 + lane) * VN;
        if (c < h) {
#pragma unroll
          for (int i = 0; i < VN; ++i) {
            const float d = dv[j].get(i);
            const float t = d * g[j].get(i);
            if (NORM == MOSAIC_LAYERNORM) {
              const float xh = (xv[j].get(i) - mean) * rstd;
              s1 += t; s2 += t * xh;
              ag[j][i] += d * xh; ab[NSUM == 2 ? j : 0][i] += d;
            } else {
              s2 += t * xv[j].get(i);
              ag[j][i] += d * xv[j].get(i) * rstd;
            }
          }
        }
      }
      if (NORM == MOSAIC_LAYERNORM) s1 = wave_sum(s1) * inv_h;
      s2 = wave_sum(s2) * inv_h;
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        const int c = (j * 64 + lane) * VN;
        if (c < h) {
          Vec16<T> o;
          if (!EARLY && R) rv[0].load(R + row * h + c);
#pragma unroll
          for (int i = 0; i < VN; ++i) {
            const float xr = xv[j].get(i);
            const float t = dv[j].get(i) * g[j].get(i);
            float r;
            if (NORM == MOSAIC_LAYERNORM) r = (t - s1 - (xr - mean) * rstd * s2) * rstd;
            else r = rstd * t - rstd * rstd * rstd * xr * s2;
            if (R) r += rv[EARLY ? j : 0].get(i);
            o.set(i, r);
            if (CS) ax[CS ? j : 0][i] += o.get(i);
          }
          o.store(dx + row * h + c);
        }
      }
    }
    // waves 1..3 hand their sums to wave 0, slab by slab; every wave passes every barrier
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      if (wave > 0) {
#pragma unroll
        for (int i = 0; i < VN; ++i) {
          red[wave - 1][0][i * 64 + lane] = ag[j][i];
          if (NSUM == 2) red[wave - 1][NSUM - 1][i * 64 + lane] = ab[NSUM == 2 ? j : 0][i];
          if (CS) red[wave - 1][NSUM][i * 64 + lane] = ax[CS ? j : 0][i];
        }
      }
      __syncthreads();
      if (wave == 0) {
        const int c = (j * 64 + lane) * VN;
        if (c < h) {
#pragma unroll
          for (int i = 0; i < VN; ++i) {
            float a = ag[j][i], b = (NSUM == 2) ? ab[NSUM == 2 ? j : 0][i] : 0.f, xs = CS ? ax[CS ? j : 0][i] : 0.f;
#pragma unroll
            for (int w = 0; w < kWaves - 1; ++w) {
              a += red[w][0][i * 64 + lane];
              if (NSUM == 2) b += red[w][NSUM - 1][i * 64 + lane];
              if (CS) xs += red[w][NSUM][i * 64 + lane];
            }
            scratch[((int64_t)p * NSLAB + 0) * h + c + i] = a;
            if (NSUM == 2) scratch[((int64_t)p * NSLAB + 1) * h + c + i] = b;
            if (CS) scratch[((int64_t)p * NSLAB + 2) * h + c + i] = xs;
          }
        }
      }
      __syncthreads();
    }
  }
}

// dgamma / dbeta partial column sums: work item = (row partition p, tile of 256 column
// vectors); a thread owns VN columns and walks the partition's rows in ascending order.
// scratch[p][2][h]; the partitions are added in a fixed order by col_reduce_kernel.
template <typename T, int NORM>
__global__ __launch_bounds__(kThreads) void norm_colgrad_partial_kernel(
    const T* __restrict__ x, const float* __restrict__ stats, const T* __restrict__ dy,
    float* __restrict__ scratch, int64_t rows, int h, int rp, int np, int ctiles) {
  constexpr int VN = Vec16<T>::N;
  const int64_t items = (int64_t)np * ctiles;
  for (int64_t it = blockIdx.x; it < items; it += gridDim.x) {
    const int p = (int)(it / ctiles), ct = (int)(it - (int64_t)p * ctiles);
    const int c = (ct * kThreads + threadIdx.x) * VN;
    if (c >= h) continue;
    float ag[VN], ab[VN];
#pragma unroll
    for (int i = 0; i < VN; ++i) { ag[i] = 0.f; ab[i] = 0.f; }
    const int64_t r0 = (int64_t)p * rp;
    const int64_t r1 = (r0 + rp < rows) ? r0 + rp : rows;
    auto add_row = [&](const Vec16<T>& xv, const Vec16<T>& dv, float mean, float rstd) {
#pragma unroll
      for (int i = 0; i < VN; ++i) {
        const float d = dv.get(i);
        if (NORM == MOSAIC_LAYERNORM) { ag[i] += d * ((xv.get(i) - mean) * rstd); ab[i] += d; }
        else ag[i] += d * xv.get(i) * rstd;
      }
    };
    int64_t row = r0;
    // four rows requested together, added in ascending row order
    for (; row + 4 <= r1; row += 4) {
      Vec16<T> xv[4], dv[4];
      float mean[4], rstd[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        xv[u].load(x + (row + u) * h + c);
        dv[u].load(dy + (row + u) * h + c);
        mean[u] = stats[(row + u) * 2]; rstd[u] = stats[(row + u) * 2 + 1];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) add_row(xv[u], dv[u], mean[u], rstd[u]);
    }
    for (; row < r1; ++row) {
      Vec16<T> xv, dv;
      xv.load(x + row * h + c);
      dv.load(dy + row * h + c);
      add_row(xv, dv, stats[row * 2], stats[row * 2 + 1]);
    }
#pragma unroll
    for (int i = 0; i < VN; ++i) {
      scratch[((int64_t)p * 2 + 0) * h + c + i] = ag[i];
      scratch[((int64_t)p * 2 + 1) * h + c + i] = ab[i];
    }
  }
}

__device__ __forceinline__ float block_sum_fixed(float v, float* red) {
  // fixed-shape reduction: butterfly inside each wave, then waves added in index order
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) red[wave] = v;
  __syncthreads();
  float t = 0.f;
  for (int w = 0; w < kWaves; ++w) t += red[w];
  __syncthreads();
  return t;
}

// loss = scale * (the partial sums in a fixed order)
__device__ __forceinline__ void loss_sum(const float* __restrict__ partial, int np, float* __restrict__ loss, float scale, float* red) {
  float acc = 0.f;
  for (int p = threadIdx.x; p < np; p += kThreads) acc += partial[p];
  const float t = block_sum_fixed(acc, red);
  if (threadIdx.x == 0) *loss = t * scale;
}

// The final pass of column reductions (ColReduce): partitions taken in 8 contiguous slices that are added in slice
// order, a fixed tree that depends on np only.  A workgroup takes 32 columns of one of the list's reductions.  Bound by
// launch and latency: one alone takes 4.5 to 8 us for a few hundred KB to 10 MB of partial sums, so a layer's go in one launch
// (two encoder layers of 1568 rows: 9 launches, 41 us -> 2, 12 us; one of 12000 rows: 5, 38 us -> 1).
template <typename T>
__global__ __launch_bounds__(kThreads) void col_reduce_kernel(ColReduceList list, int64_t total) {
  __shared__ float red[8][32];
  const int cl = threadIdx.x & 31, sl = threadIdx.x >> 5;
  if (list.loss && blockIdx.x == gridDim.x - 1) loss_sum(list.loss_partial, list.loss_np, list.loss, list.loss_scale, &red[0][0]);
  for (int64_t at = blockIdx.x; at < total; at += gridDim.x) {
    int64_t gidx = at;
    int which = 0;
    while (gidx >= (list.job[which].ncols + 31) / 32) { gidx -= (list.job[which].ncols + 31) / 32; ++which; }
    const ColReduce& r = list.job[which];
    const int np = r.np, per = (np + 7) / 8;
    const int64_t col = gidx * 32 + cl, ld = r.ld;
    const float* partial = r.partial;
    float acc = 0.f;
    T* dst = nullptr;
    if (col < r.ncols)
      dst = col < r.split ? (T*)r.out0 + col : col < r.split2 ? (r.out1 ? (T*)r.out1 + (col - r.split) : nullptr) : (r.out2 ? (T*)r.out2 + (col - r.split2) : nullptr);
    if (dst) {
      const int p1 = (sl + 1) * per < np ? (sl + 1) * per : np;
      int p = sl * per;
      // sixteen independent requests in flight, added in ascending p; past the slice's end the last partition is asked for again and not
      // added (one by one, the up to seven partitions behind whole batches of eight took most of the time: 12000 x 1280, 500 partitions, partial
      // sums included 11.9 -> 9.4 us, 12000 x 5120 26.8 -> 24.2; this kernel alone 256 x 128, 32 partitions, 3.0 -> 2.4, 64 x 64, 8 partitions,
      // 1.8 -> 2.2; batches of 32 8.7 and 23.5; of four where a slice has no more 2.4 and 2.2)
      constexpr int ONCE = 16;
      for (; p < p1; p += ONCE) {
        float v[ONCE];
#pragma unroll
        for (int u = 0; u < ONCE; ++u) v[u] = partial[(int64_t)min(p + u, p1 - 1) * ld + col];
#pragma unroll
        for (int u = 0; u < ONCE; ++u) acc = p + u < p1 ? acc + v[u] : acc;
      }
    }
    red[sl][cl] = acc;
    __syncthreads();
    if (sl == 0 && dst) {
      float t = 0.f;
#pragma unroll
      for (int q = 0; q < 8; ++q) t += red[q][cl];
      *dst = from_f32<T>(t);
    }
    __syncthreads();
  }
}

// -------------------------------------------------------------------------- activations
// gelu_f, gelu_grad_f, sigmoid_f, swiglu_f: activations.h

template <typename T>
__global__ __launch_bounds__(kThreads) void gelu_fwd_kernel(const T* __restrict__ z, T* __restrict__ a, int64_t nvec) {
  constexpr int VN = Vec16<T>::N;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < nvec; i += (int64_t)gridDim.x * kThreads) {
    Vec16<T> v, o;
    v.load(z + i * VN);
#pragma unroll
    for (int k = 0; k < VN; ++k) o.set(k, gelu_f(v.get(k)));
    o.store(a + i * VN);
  }
}

// GELU backward: HBM-bound at 6 bytes per bf16 element once erf comes from a table that the workgroup fills
// first (ErfTable; the same bits): with an erff per element the pass was bound by instructions.  12000 x 5120
// 90 -> 73 us, 9216 x 4096 48 -> 39 (5.8 TB/s), on 64 CUs 12000 x 5120 285 -> 189; at eight elements a thread, the fewest
// that there are, 7.6 -> 7.2.
template <typename T>
__global__ __launch_bounds__(kThreads) void gelu_bwd_kernel(const T* __restrict__ z, const T* __restrict__ da,
                                                            T* __restrict__ dz, int64_t nvec) {
  constexpr int VN = Vec16<T>::N;
  constexpr bool TAB = std::is_same<T, bf16>::value;
  __shared__ float table[TAB ? ErfTable::kEntries : 1];
  if constexpr (TAB) { ErfTable::fill(table, threadIdx.x, kThreads); __syncthreads(); }
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < nvec; i += (int64_t)gridDim.x * kThreads) {
    Vec16<T> v, d, o;
    v.load(z + i * VN);
    d.load(da + i * VN);
#pragma unroll
    for (int k = 0; k < VN; ++k) o.set(k, d.get(k) * (TAB ? ErfTable::gelu_grad(table, v.get(k)) : gelu_grad_f(v.get(k))));
    o.store(dz + i * VN);
  }
}

// dz = da * gelu'(z) and, in the same pass, the partial column sums of dz as stored (the bias
// gradient of the linear layer that produced z), in the order of launch_colsum over the stored dz, so the sums have the same bits.
// Bound by memory where waves are many, by the chain of one wave where they are few: 8 bytes a lane and four rows at once in the first
// case, 4 bytes and eight rows, so twice the waves, in the second (the rule is at the launch; both add in the same order).
// Microseconds, final reduction included, on 256 CUs (on 64), bf16: partitions walked by one thread per 16 bytes of a row / by
// four waves, a quarter each / this: 1568 x 3072 16.5 (30.7) / 13.6 (24.6) / 13.2 (23.4), 4608 x 4096 27.6 (67.1) / 30.0 (77.5) / 27.5 (66.6),
// 9216 x 4096 44.7 (121.8) / 46.8 (127.1) / 45.0 (119.6), 12000 x 5120 90.9 (212) / 83.6 (201) / 83.6 (196), 24000 x 1280 55.8 (139) / 41.6 (117) / 39.3 (98).
// TAPS: da is the gradient [B * lo, 3n] of the gathered input of a three-tap convolution of stride 2 over B x 2 lo rows, and a row's
// gradient the sum of its taps (ascending) in fp32: row 2t is tap 1 of output t, row 2t + 1 tap 0 of output t + 1 and tap 2 of output t.
// A pass of its own for that wrote and read 61 MB each for 24000 rows of 1280: 32 + 42 us -> 58, and with one multiplication for the
// address of a row's taps 46 (on 64 CUs 143 -> 114).
template <typename T, int V, int ONCE, bool QUARTERS, bool TAPS>
__global__ __launch_bounds__(kThreads) void gelu_bwd_colsum_kernel(const T* __restrict__ z, const T* __restrict__ da,
                                                                   T* __restrict__ dz, float* __restrict__ partial,
                                                                   int64_t rows, int64_t n, int rp, int np, int ctiles, int lo, uint64_t m_lo, Along along) {
  if (sums_along<T>(along)) return;
  typedef typename Pack<T, V>::type vec;
  constexpr bool TAB = std::is_same<T, bf16>::value;
  __shared__ float table[TAB ? ErfTable::kEntries : 1];
  if constexpr (TAB) { ErfTable::fill(table, threadIdx.x, kThreads); __syncthreads(); }
  struct Req { vec z, d, d2; bool two; };
  column_sums<V, ONCE, QUARTERS>((int)blockIdx.x - along.blocks, (int)gridDim.x - along.blocks, rows, n, rp, np, ctiles, partial, [&](int64_t r, int64_t c) {
    Req q;
    q.z = *reinterpret_cast<const vec*>(z + r * n + c);
    if constexpr (TAPS) {
      const int64_t t = r >> 1, odd = r & 1;                        // t: output row, over all samples
      // the sample's last row has no output after it; m_lo = 2^64 / lo, rounded up: exact for 32-bit numbers (lo 1: every row)
      q.two = odd && lo > 1 && (uint32_t)(t + 1) != (uint32_t)__umul64hi((uint64_t)(t + 1), m_lo) * (uint32_t)lo;
      const T* at = da + (3 * t + 1 + odd) * n;
      q.d2 = *reinterpret_cast<const vec*>(at + c);
      q.d = *reinterpret_cast<const vec*>((q.two ? at + n : at) + c);
    } else {
      q.d = *reinterpret_cast<const vec*>(da + r * n + c);
    }
    return q;
  }, [&](const Req& q, int64_t r, int64_t c, float (&acc)[V]) {
#pragma clang fp contract(off)          // what is stored is added: a product rounded to T, not one fused with the addition
    vec o;
#pragma unroll
    for (int k = 0; k < V; ++k) {
      const float zk = pack_get<T, V>(q.z, k);
      float d = pack_get<T, V>(q.d, k);
      if constexpr (TAPS) d = q.two ? d + pack_get<T, V>(q.d2, k) : pack_get<T, V>(q.d2, k);
      pack_set<T, V>(o, k, d * (TAB ? ErfTable::gelu_grad(table, zk) : gelu_grad_f(zk)));
      acc[k] += pack_get<T, V>(o, k);
    }
    *reinterpret_cast<vec*>(dz + r * n + c) = o;
  });
}

template <typename T>
__global__ __launch_bounds__(kThreads) void swiglu_fwd_kernel(const T* __restrict__ gu, T* __restrict__ a,
                                                              int64_t rows, int fv) {
  constexpr int VN = Vec16<T>::N;
  const int64_t nvec = rows * fv;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < nvec; i += (int64_t)gridDim.x * kThreads) {
    const int64_t r = i / fv;
    const int64_t c = (i - r * fv) * VN;
    const int64_t f = (int64_t)fv * VN;
    Vec16<T> g, u, o;
    g.load(gu + r * 2 * f + c);
    u.load(gu + r * 2 * f + f + c);
#pragma unroll
    for (int k = 0; k < VN; ++k) o.set(k, swiglu_f(g.get(k), u.get(k)));
    o.store(a + r * f + c);
  }
}

// Bound by memory, 10 bytes per bf16 pair: workgroups in order above 64 MB, accesses past the caches above 256 MB.  8192 x 5632 88.2 -> 70.8 us (208 ->
// 190 on 64 CUs; in order alone 80.6), 32768 x 11008 757 -> 596 (1591 -> 1476; 668).
template <typename T, bool PAST>
__global__ __launch_bounds__(kThreads) void swiglu_bwd_kernel(const T* __restrict__ gu, const T* __restrict__ da,
                                                              T* __restrict__ dgu, int64_t rows, int fv) {
  constexpr int VN = Vec16<T>::N;
  const int64_t nvec = rows * fv;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < nvec; i += (int64_t)gridDim.x * kThreads) {
    const int64_t r = i / fv;
    const int64_t c = (i - r * fv) * VN;
    const int64_t f = (int64_t)fv * VN;
    Vec16<T> g, u, d, og, ou;
    g.template load<PAST>(gu + r * 2 * f + c);
    u.template load<PAST>(gu + r * 2 * f + f + c);
    d.template load<PAST>(da + r * f + c);
#pragma unroll
    for (int k = 0; k < VN; ++k) {
      float dg, du;
      swiglu_grad_f(g.get(k), u.get(k), d.get(k), &dg, &du);
      og.set(k, dg);
      ou.set(k, du);
    }
    og.template store<PAST>(dgu + r * 2 * f + c);
    ou.template store<PAST>(dgu + r * 2 * f + f + c);
  }
}

// ---------------------------------------------------------------------------------- MSE
constexpr int kMsePartials = 1024;

template <typename T>
__global__ __launch_bounds__(kThreads) void mse_kernel(const T* __restrict__ y, const T* __restrict__ tg,
                                                       T* __restrict__ dy, float* __restrict__ partial,
                                                       int64_t nvec, int np, float scale) {
  constexpr int VN = Vec16<T>::N;
  __shared__ float red[kWaves];
  for (int p = blockIdx.x; p < np; p += gridDim.x) {
    float acc = 0.f;
    for (int64_t i = (int64_t)p * kThreads + threadIdx.x; i < nvec; i += (int64_t)np * kThreads) {
      Vec16<T> a, b, o;
      a.load(y + i * VN);
      b.load(tg + i * VN);
#pragma unroll
      for (int k = 0; k < VN; ++k) {
        const float dlt = a.get(k) - b.get(k);
        acc += dlt * dlt;
        o.set(k, dlt * scale);
      }
      o.store(dy + i * VN);
    }
    const float t = block_sum_fixed(acc, red);
    if (threadIdx.x == 0) partial[p] = t;
  }
}

__global__ __launch_bounds__(kThreads) void mse_final_kernel(const float* __restrict__ partial, int np, float* __restrict__ loss, float inv_n) {
  __shared__ float red[kWaves];
  loss_sum(partial, np, loss, inv_n, red);
}

// ------------------------------------------------------------------------------ colsum
// row partitions of a column reduction (a function of the row count alone).  512: two
// workgroups per CU for the one-pass norm backward (5.1 TB/s at the decoder shape against 4.8
// with 256; 1024 partitions make the partial sums too much traffic: 4.1)
constexpr int kColsumMaxParts = 512;
// widest row (in 16-byte vectors per lane) whose column accumulators the fused norm backward keeps in registers
constexpr int kNormFusedMaxNV = 8;   // LayerNorm; RMSNorm (one sum per column) also fits at 10

template <typename T, bool QUARTERS>
__global__ __launch_bounds__(kThreads) void colsum_partial_kernel(const T* __restrict__ X, float* __restrict__ partial,
                                                                  int64_t rows, int64_t n, int rp, int np, int ctiles) {
  plain_column_sums<T, QUARTERS>(blockIdx.x, gridDim.x, X, partial, rows, n, rp, np, ctiles);
}

// The sums of column_sums with QUARTERS, by one wave: two rows of each quarter are requested together.  32768 x 2048 on 256, 128,
// 64 CUs: four waves 28.1 36.4 34.1 us, this 27.5 26.6 31.2; 24000 x 4096 38.1 38.1 50.3 -> 37.5 37.4 46.6; 65536 x 4096 100 122 187 -> 101 117 179.
template <typename T>
__global__ __launch_bounds__(kThreads) void colsum_quarters_kernel(const T* __restrict__ X, float* __restrict__ partial,
                                                                   int64_t rows, int64_t n, int rp, int np, int ctiles) {
  constexpr int V = Vec16<T>::N;
  const int64_t items = (int64_t)np * ctiles;
  for (int64_t it = (int64_t)blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); it < items; it += (int64_t)gridDim.x * kWaves) {
    const int p = (int)(it / ctiles), ct = (int)(it - (int64_t)p * ctiles);
    const unsigned c = (unsigned)(ct * 64 + (threadIdx.x & 63)) * V;
    const int64_t r0 = (int64_t)p * rp;
    if (c >= n) continue;
    const int count = (int)(r0 + rp < rows ? rp : rows - r0), per = (count + 3) >> 2, whole = max(count - 3 * per, 0) & ~1;
    const T* x = X + r0 * n;
    float acc[4][V] = {};
    Vec16<T> v[4][2];
    for (int i = 0; i < whole; i += 2, x += 2 * n) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int u = 0; u < 2; ++u) v[k][u].load(x + (k * per + u) * n + c);
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int e = 0; e < V; ++e) acc[k][e] += v[k][u].get(e);
    }
    for (int i = whole; i < per; ++i, x += n) {
#pragma unroll
      for (int k = 0; k < 4; ++k) if (k * per + i < count) v[k][0].load(x + k * per * n + c);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (k * per + i < count) {
#pragma unroll
          for (int e = 0; e < V; ++e) acc[k][e] += v[k][0].get(e);
        }
    }
#pragma unroll
    for (int e = 0; e < V; ++e) partial[(int64_t)p * n + c + e] = acc[0][e] + acc[1][e] + acc[2][e] + acc[3][e];
  }
}

// ------------------------------------------------------------------------------- stems
// Patch vector index = (c*p + i)*p + j; patches row-major over the image.  Rows are `ld` >= 3*p*p
// elements apart; what lies between is filled with zeros, so that rows of 588 elements (14 x 14
// patches) start on 16-byte boundaries and the matrix-core product takes them.  A thread writes one
// 16-byte piece of a row; its pixels are neighbours, so the 2-byte reads hit the cache.  I: index
// type (32 bits where they hold every piece: a 64-bit division per element took the 26 us that
// this pass spent on 16 images of 336 x 336; with it in 32 bits, once per piece, it takes 11).
template <typename T, typename I>
__global__ __launch_bounds__(kThreads) void unfold_kernel(const T* __restrict__ img, T* __restrict__ out,
                                                          int B, int side, int patch, int ld) {
  constexpr int VN = Vec16<T>::N;
  const int g = side / patch, pd = 3 * patch * patch, pieces = ld / VN;
  const I total = (I)B * g * g * pieces;
  for (I v = (I)blockIdx.x * kThreads + threadIdx.x; v < total; v += (I)gridDim.x * kThreads) {
    const I tok = v / pieces;
    int e = (int)(v - tok * pieces) * VN;
    const I prow = tok / g;
    const int px = (int)(tok - prow * g), py = (int)(prow % g), b = (int)(prow / g);
    int c = e / (patch * patch), ij = e - c * patch * patch, i = ij / patch, j = ij - i * patch;
    Vec16<T> o;
#pragma unroll
    for (int k = 0; k < VN; ++k, ++e) {
      o.set(k, e < pd ? to_f32(img[(((int64_t)b * 3 + c) * side + (py * patch + i)) * side + (px * patch + j)]) : 0.f);
      if (++j == patch) { j = 0; if (++i == patch) { i = 0; ++c; } }
    }
    o.store(out + (int64_t)tok * ld + (int64_t)(v - tok * pieces) * VN);
  }
}

// The same for bf16 and an even patch: work item = one channel of a row of patches, `patch` whole rows of the image, which lie
// one after the other and pass through LDS, read and written 8 bytes at a time.  Bound by memory: with a projection to 64 columns
// behind it, 16 images of 512 x 512 in 16 x 16 patches 36.6 -> 24.2 us, 16 of 336 x 336 in 14 x 14 20.8 -> 20.1 (rows that end in
// mid line), one of 112 x 112 13.6 -> 13.3.  P2 = patch * patch (a multiple of 4); rows of out are ld elements apart, a multiple of 8.
constexpr int kStripBytes = 32 << 10;        // of an image's rows that a workgroup takes; wider images go to unfold_kernel
__global__ __launch_bounds__(kThreads) void unfold_strip_kernel(const bf16* __restrict__ img, bf16* __restrict__ out, int64_t strips, int side, int patch,
                                                                int ld, uint32_t m_quads, uint32_t m_patch) {
  // m_quads, m_patch: 2^32 / divisor + 1, exact for the numbers below 2^16 that they divide
  extern __shared__ __align__(16) uint32_t strip[];        // [patch][side / 2]
  const int g = side / patch, p2 = patch * patch, quads = p2 >> 2, n8 = patch * side >> 2, half = side >> 1;
  for (int64_t it = blockIdx.x; it < strips; it += gridDim.x) {
    const int64_t by = it / 3;                             // row of patches, over all images
    const int c = (int)(it - by * 3), py = (int)(by % g);
    const uint2* src = reinterpret_cast<const uint2*>(img + ((by / g * 3 + c) * side + py * patch) * side);
    for (int i = threadIdx.x; i < n8; i += 4 * kThreads) {
      uint2 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) if (i + u * kThreads < n8) v[u] = src[i + u * kThreads];
#pragma unroll
      for (int u = 0; u < 4; ++u) if (i + u * kThreads < n8) reinterpret_cast<uint2*>(strip)[i + u * kThreads] = v[u];
    }
    __syncthreads();
    bf16* const row0 = out + by * g * ld;
    for (int w = threadIdx.x; w < g * quads; w += kThreads) {
      const int px = (int)__umulhi(w, m_quads), e = (w - px * quads) << 2, i = (int)__umulhi(e, m_patch), j = e - i * patch;
      const int at = (i * side + px * patch + j) >> 1;
      uint2 v;
      v.x = strip[at];
      v.y = strip[j + 2 < patch ? at + 1 : at + 1 + half - (patch >> 1)];
      *reinterpret_cast<uint2*>(row0 + (int64_t)px * ld + c * p2 + e) = v;
    }
    if (c == 2) {                                          // zeros between a patch's values and the next row
      const int pad = (ld - 3 * p2) >> 2;
      for (int w = threadIdx.x; w < g * pad; w += kThreads) {
        const int px = w / pad;
        *reinterpret_cast<uint2*>(row0 + (int64_t)px * ld + 3 * p2 + ((w - px * pad) << 2)) = make_uint2(0u, 0u);
      }
    }
    __syncthreads();
  }
}

// y[b, t, :] += pos[t, :].  Work item = (sample, block of kThreads pieces of the N x h table): one
// division per item.  V elements per access: 16 bytes, or one for tensors that are not 16-byte aligned.
// Bound by memory: 16 x 576 x 1024 in bf16 12 us one element at a time -> 7.5, 8 x 1500 x 1280 20 -> 14.
template <typename T, int V>
__global__ __launch_bounds__(kThreads) void add_pos_kernel(const T* __restrict__ pos, T* __restrict__ y, int B, int64_t per, int blocks) {
  typedef typename Pack<T, V>::type vec;
  for (int64_t it = blockIdx.x; it < (int64_t)B * blocks; it += gridDim.x) {
    const int64_t b = it / blocks, i = ((it - b * blocks) * kThreads + threadIdx.x) * V;
    if (i >= per) continue;
    const vec p = *reinterpret_cast<const vec*>(pos + i);
    vec v = *reinterpret_cast<const vec*>(y + b * per + i);
#pragma unroll
    for (int k = 0; k < V; ++k) pack_set<T, V>(v, k, pack_get<T, V>(v, k) + pack_get<T, V>(p, k));
    *reinterpret_cast<vec*>(y + b * per + i) = v;
  }
}

// dpos[t, :] = sum over samples in ascending order; four samples' pieces are requested together.
// Bound by memory: 16 x 576 x 1024 in bf16 9.6 us one element at a time -> 4.3, 8 x 1500 x 1280 19 -> 10.
template <typename T, int V>
__global__ __launch_bounds__(kThreads) void pos_grad_kernel(const T* __restrict__ dy, T* __restrict__ dpos, int B, int64_t per) {
  typedef typename Pack<T, V>::type vec;
  for (int64_t i = ((int64_t)blockIdx.x * kThreads + threadIdx.x) * V; i < per; i += (int64_t)gridDim.x * kThreads * V) {
    float acc[V];
#pragma unroll
    for (int k = 0; k < V; ++k) acc[k] = 0.f;
    int b = 0;
    for (; b + 4 <= B; b += 4) {
      vec v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const vec*>(dy + (int64_t)(b + u) * per + i);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int k = 0; k < V; ++k) acc[k] += pack_get<T, V>(v[u], k);
    }
    for (; b < B; ++b) {
      const vec v = *reinterpret_cast<const vec*>(dy + (int64_t)b * per + i);
#pragma unroll
      for (int k = 0; k < V; ++k) acc[k] += pack_get<T, V>(v, k);
    }
    vec o = {};
#pragma unroll
    for (int k = 0; k < V; ++k) pack_set<T, V>(o, k, acc[k]);
    *reinterpret_cast<vec*>(dpos + i) = o;
  }
}

// What the gradient of a patch stem's output gives besides the product: dpos[t, :] = sum over samples (ascending) of dy, and the partial
// column sums of the bias gradient.  A wave takes 64 * V columns of `rp` positions and goes through the samples of a position, eight of them
// requested together; the bias sums run over its positions and samples in that order.  Bound by memory and, as the waves are few, by the
// latency of their requests: four bytes a lane, up to four samples 16 (bits do not follow it: a lane owns its columns).  One pass over dy where there
// were two, and a launch less: the backward pass of 16 x 576 x 1024 31.0 -> 25.1 us (eight bytes a lane 25.9), of 4 x 196 x 768 19.9 -> 16.2.  Four / 16
// bytes a lane at 2 x 4096 x 1024, us: 27.2 / 26.6, on 32 CUs 55 / 38 (two passes 43); at 8 x 1024 x 1024 24.6 / 26.1.
template <typename T, int V>
__global__ __launch_bounds__(kThreads) void stem_grad_kernel(const T* __restrict__ dy, T* __restrict__ dpos, float* __restrict__ partial, int B, int N, int h,
                                                             int rp, int np, int ctiles) {
  typedef typename Pack<T, V>::type vec;
  constexpr int ONCE = 8;
  const int lane = threadIdx.x & 63;
  const int64_t items = (int64_t)np * ctiles, per = (int64_t)N * h;
  for (int64_t it = (int64_t)blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); it < items; it += (int64_t)gridDim.x * kWaves) {
    const int p = (int)(it / ctiles), c = ((int)(it - (int64_t)p * ctiles) * 64 + lane) * V;
    if (c >= h) continue;
    float col[V] = {};
    for (int t = p * rp; t < min(N, (p + 1) * rp); ++t) {
      const int64_t at = (int64_t)t * h + c;
      float pos[V] = {};
      for (int b0 = 0; b0 < B; b0 += ONCE) {
        vec d[ONCE];
#pragma unroll
        for (int u = 0; u < ONCE; ++u) if (b0 + u < B) d[u] = *reinterpret_cast<const vec*>(dy + (b0 + u) * per + at);
#pragma unroll
        for (int u = 0; u < ONCE; ++u)
          if (b0 + u < B) {
#pragma unroll
            for (int k = 0; k < V; ++k) { pos[k] += pack_get<T, V>(d[u], k); col[k] += pack_get<T, V>(d[u], k); }
          }
      }
      vec o;
#pragma unroll
      for (int k = 0; k < V; ++k) pack_set<T, V>(o, k, pos[k]);
      *reinterpret_cast<vec*>(dpos + at) = o;
    }
#pragma unroll
    for (int k = 0; k < V; ++k) partial[(int64_t)p * h + c + k] = col[k];
  }
}

int pick_nv(int need) {
  const int opts[] = {1, 2, 3, 4, 5, 6, 8, 10};
  for (int o : opts) if (o >= need) return o;
  return -1;
}

}  // namespace

// =================================================================== host launchers
#define DISPATCH_NV(NVV, MACRO) \
  switch (NVV) {                \
    case 1: MACRO(1); break;    \
    case 2: MACRO(2); break;    \
    case 3: MACRO(3); break;    \
    case 4: MACRO(4); break;    \
    case 5: MACRO(5); break;    \
    case 6: MACRO(6); break;    \
    case 8: MACRO(8); break;    \
    default: MACRO(10); break;  \
  }

// workgroups of kThreads that a CU holds at once, by the kernel's registers
template <auto kernel>
static int resident_workgroups() {
  static const int n = [] {
    int r = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&r, reinterpret_cast<const void*>(kernel), kThreads, 0) != hipSuccess) { (void)hipGetLastError(); r = 0; }
    return r > 0 ? r : 8;
  }();
  return n;
}

template <typename T>
static mosaic_status norm_fwd_t(hipStream_t s, int quota, int norm, int64_t rows, int64_t h, float eps,
                                const T* x, const T* gamma, const T* beta, T* y, float* stats) {
  constexpr int VN = Vec16<T>::N;
  if (h % VN) MOSAIC_FAIL(MOSAIC_EUNSUPPORTED, "norm width %lld is not a multiple of %d", (long long)h, VN);
  const int nv = pick_nv((int)ceil_div(h, 64 * VN));
  if (nv < 0) MOSAIC_FAIL(MOSAIC_EUNSUPPORTED, "norm width %lld too large", (long long)h);
  if (rows == 0) return MOSAIC_OK;
  // Workgroups that a CU holds at once, not eight where registers allow three to seven: those behind the first would start when the first have
  // walked their whole share.  Eight to a CU / resident, us on 256 and 64 CUs: LayerNorm 24576 x 1536 (seven) 27.5 / 24.0 and 65.6 / 47.7, 35840 x 2048
  // (five) 66.5 / 59.4 and 189 / 165; RMSNorm 35840 x 4096 (seven) 134 / 119 and 370 / 272.  One workgroup per four rows, started in order, reads the
  // gains again for every row: rows of 64 to 1024 values up to a quarter slower (1048576 x 64 225 / 262, on 64 CUs 858 / 1044).
  auto launch = [&](auto nvc, auto kind) {
    constexpr auto kern = norm_fwd_kernel<T, decltype(kind)::value, decltype(nvc)::value>;
    kern<<<grid_for(quota, std::min(8, resident_workgroups<kern>()), ceil_div(rows, kWaves)), kThreads, 0, s>>>(x, gamma, beta, y, stats, rows, (int)h, eps);
  };
#define L(NVC)                                                                                                                          \
  if (norm == MOSAIC_LAYERNORM) launch(std::integral_constant<int, NVC>{}, std::integral_constant<int, MOSAIC_LAYERNORM>{});           \
  else launch(std::integral_constant<int, NVC>{}, std::integral_constant<int, MOSAIC_RMSNORM>{})
  DISPATCH_NV(nv, L);
#undef L
  MOSAIC_LAUNCH_CHECK();
  return MOSAIC_OK;
}

mosaic_status launch_norm_fwd(hipStream_t s, int quota, int dtype, int norm, int64_t T, int64_t h, float eps,
                              const void* x, const void* gamma, const void* beta, void* y, float* stats) {
  if (norm != MOSAIC_LAYERNORM && norm != MOSAIC_RMSNORM) MOSAIC_FAIL(MOSAIC_EINVAL, "bad norm kind %d", norm);
  if (dtype == MOSAIC_BF16)
    return norm_fwd_t<bf16>(s, quota, norm, T, h, eps, (const bf16*)x, (const bf16*)gamma, (const bf16*)beta, (bf16*)y, stats);
  return norm_fwd_t<float>(s, quota, norm, T, h, eps, (const float*)x, (const float*)gamma, (const float*)beta, (float*)y, stats);
}

static mosaic_status launch_pending(hipStream_t s, int quota, int dtype, const ColSumJob& j) {
  if (j.np == 0) return MOSAIC_OK;
  const int grid = grid_for(quota, 8, ceil_div((int64_t)j.np * j.ctiles, kWaves));
  if (dtype == MOSAIC_BF16) colsum_partial_kernel<bf16, false><<<grid, kThreads, 0, s>>>((const bf16*)j.X, j.partial, j.rows, j.n, j.rp, j.np, j.ctiles);
  else colsum_partial_kernel<float, false><<<grid, kThreads, 0, s>>>((const float*)j.X, j.partial, j.rows, j.n, j.rp, j.np, j.ctiles);
  MOSAIC_LAUNCH_CHECK();
  return MOSAIC_OK;
}
mosaic_status launch_col_reduce(hipStream_t s, int quota, int dtype, const ColReduceList& list) {
  MOSAIC_TRY(launch_pending(s, quota, dtype, list.pending));
  int64_t total = 0;
  for (int i = 0; i < list.n; ++i) total += ceil_div(list.job[i].ncols, 32);
  if (total == 0 && !list.loss) return MOSAIC_OK;
  const int grid = grid_for(quota, 8, total);
  if (dtype == MOSAIC_BF16) col_reduce_kernel<bf16><<<grid, kThreads, 0, s>>>(list, total);
  else col_reduce_kernel<float><<<grid, kThreads, 0, s>>>(list, total);
  MOSAIC_LAUNCH_CHECK();
  return MOSAIC_OK;
}
// the pending sums of a layer, to go with the launch at hand
static Along take_along(int quota, ColReduceList* later) {
  Along a = {};
  if (!later || later->pending.np == 0) return a;
  a.job = later->pending;
  a.blocks = grid_for(quota, 8, ceil_div((int64_t)a.job.np * a.job.ctiles, kWaves));
  later->pending = ColSumJob();
  return a;
}
// now, or with the rest of `later`
static mosaic_status col_reduce(hipStream_t s, int quota, int dtype, const ColReduce& r, ColReduceList* later) {
  if (later && later->n < ColReduceList::kMax) { later->job[later->n++] = r; return MOSAIC_OK; }
  ColReduceList one;
  one.job[one.n++] = r;
  return launch_col_reduce(s, quota, dtype, one);
}

int64_t colsum_partition_rows(int64_t T) { return std::max<int64_t>(8, ceil_div(T, kColsumMaxParts)); }
static inline void col_partition(int64_t T, int* rp, int* np) {
  const int64_t r = colsum_partition_rows(T);
  *rp = (int)r;
  *np = (int)ceil_div(T, r);
}

size_t norm_bwd_scratch_bytes(int64_t h, bool with_dxsum) { return (size_t)kColsumMaxParts * (with_dxsum ? 3 : 2) * (size_t)h * sizeof(float); }
// widest row (16-byte vectors per lane) for which the one-pass kernel also keeps the column sums of dx
constexpr int kNormDxSumMaxNV = 4;

template <typename T>
static mosaic_status norm_bwd_t(hipStream_t s, int quota, int norm, int64_t rows, int64_t h, const T* x,
                                const T* gamma, const float* stats, const T* dy, const T* R, T* dx,
                                T* dgamma, T* dbeta, float* scratch, T* dxsum, int dtype, ColReduceList* later) {
  constexpr int VN = Vec16<T>::N;
  if (h % VN) MOSAIC_FAIL(MOSAIC_EUNSUPPORTED, "norm width %lld is not a multiple of %d", (long long)h, VN);
  const int nv = pick_nv((int)ceil_div(h, 64 * VN));
  if (nv < 0) MOSAIC_FAIL(MOSAIC_EUNSUPPORTED, "norm width %lld too large", (long long)h);
  if (rows == 0) return MOSAIC_OK;
  int rp, np;
  col_partition(rows, &rp, &np);
  if (dxsum && norm == MOSAIC_LAYERNORM && nv <= kNormDxSumMaxNV) {
    // one pass that also sums the columns of dx
    const int gf = grid_for(quota, 8, np);
    const Along along = take_along(quota, later);
#define LC(NVC) norm_bwd_fused_kernel<T, MOSAIC_LAYERNORM, NVC, true><<<along.blocks + gf, kThreads, 0, s>>>(x, gamma, stats, dy, R, dx, scratch, rows, (int)h, rp, np, along)
    switch (nv) {
      case 1: LC(1); break;
      case 2: LC(2); break;
      case 3: LC(3); break;
      default: LC(4); break;
    }
#undef LC
    MOSAIC_LAUNCH_CHECK();
    return col_reduce(s, quota, dtype, {scratch, np, 3 * h, 3 * h, h, 2 * h, dgamma, dbeta, dxsum}, later);
  }
  const ColReduce sums = {scratch, np, 2 * h, 2 * h, h, INT64_MAX, dgamma, norm == MOSAIC_LAYERNORM ? dbeta : nullptr, nullptr};
  const bool fused = nv <= kNormFusedMaxNV || norm == MOSAIC_RMSNORM;
  if (later && (dxsum || !fused)) {      // no kernel below takes them along, and dx may lie on what they are formed of
    MOSAIC_TRY(launch_pending(s, quota, dtype, later->pending));
    later->pending = ColSumJob();
  }
  if (dxsum) later = nullptr;            // the pass over dx below writes its partial sums into the same scratch
  // no kernel that sums dx on the way for this norm or width: the sums take a pass of their own, afterwards
  auto sum_dx = [&]() -> mosaic_status { return dxsum ? launch_colsum(s, quota, dtype, rows, h, dx, dxsum, scratch) : MOSAIC_OK; };
  if (fused) {
    // one pass: x and dy are read once for dx and for the column sums
    const int gf = grid_for(quota, 8, np);
    const Along along = take_along(quota, later);
    // A kernel that the residual's registers cost a wave per SIMD requests it with the row where a CU has one workgroup at most, and (three vectors a
    // lane) where there is one: late / early, fp32 RMSNorm 500 x 2560 15.2 / 12.3 us, 4096 x 2560 33.9 / 37.7, on 64 CUs without a residual 49.0 / 62.4;
    // bf16 RMSNorm 4096 x 2560 on 64 CUs 45.7 / 56.9, 4096 x 1536 on 256 16.7 / 15.5, on 64 without 23.3 / 24.6.
    auto launch = [&](auto kind, auto nvc) {
      constexpr int KIND = decltype(kind)::value, NVC = decltype(nvc)::value;
      auto go = [&](auto early) {
        norm_bwd_fused_kernel<T, KIND, NVC, false, decltype(early)::value><<<along.blocks + gf, kThreads, 0, s>>>(x, gamma, stats, dy, R, dx, scratch, rows, (int)h, rp, np, along);
      };
      if constexpr (norm_bwd_tight<T, KIND, NVC>()) {
        if (!(NVC == 3 ? R != nullptr : np <= quota)) return go(std::false_type{});
      }
      go(std::true_type{});
    };
#define LF(NVC)                                                                                                                \
    if (norm == MOSAIC_LAYERNORM) launch(std::integral_constant<int, MOSAIC_LAYERNORM>{}, std::integral_constant<int, NVC>{}); \
    else launch(std::integral_constant<int, MOSAIC_RMSNORM>{}, std::integral_constant<int, NVC>{})
    switch (nv) {
      case 1: LF(1); break;
      case 2: LF(2); break;
      case 3: LF(3); break;
      case 4: LF(4); break;
      case 5: LF(5); break;
      case 6: LF(6); break;
      case 8: LF(8); break;
      default:
        launch(std::integral_constant<int, MOSAIC_RMSNORM>{}, std::integral_constant<int, 10>{});
        break;
    }
#undef LF
    MOSAIC_LAUNCH_CHECK();
    MOSAIC_TRY(col_reduce(s, quota, dtype, sums, later));
    return sum_dx();
  }
  const int grid = grid_for(quota, 8, ceil_div(rows, kWaves));
#define L(NVC)                                                                                        \
  if (norm == MOSAIC_LAYERNORM)                                                                       \
    norm_bwd_dx_kernel<T, MOSAIC_LAYERNORM, NVC><<<grid, kThreads, 0, s>>>(x, gamma, stats, dy, R, dx, rows, (int)h); \
  else                                                                                                \
    norm_bwd_dx_kernel<T, MOSAIC_RMSNORM, NVC><<<grid, kThreads, 0, s>>>(x, gamma, stats, dy, R, dx, rows, (int)h)
  DISPATCH_NV(nv, L);
#undef L
  MOSAIC_LAUNCH_CHECK();
  const int ctiles = (int)ceil_div(h, (int64_t)kThreads * VN);
  const int g1 = grid_for(quota, 8, (int64_t)np * ctiles);
  if (norm == MOSAIC_LAYERNORM)
    norm_colgrad_partial_kernel<T, MOSAIC_LAYERNORM><<<g1, kThreads, 0, s>>>(x, stats, dy, scratch, rows, (int)h, rp, np, ctiles);
  else
    norm_colgrad_partial_kernel<T, MOSAIC_RMSNORM><<<g1, kThreads, 0, s>>>(x, stats, dy, scratch, rows, (int)h, rp, np, ctiles);
  MOSAIC_LAUNCH_CHECK();
  MOSAIC_TRY(col_reduce(s, quota, dtype, sums, later));
  return sum_dx();
}

mosaic_status launch_norm_bwd(hipStream_t s, int quota, int dtype, int norm, int64_t T, int64_t h, const void* x,
                              const void* gamma, const float* stats, const void* dy, const void* R, void* dx,
                              void* dgamma, void* dbeta, void* scratch, void* dxsum, ColReduceList* later) {
  if (norm != MOSAIC_LAYERNORM && norm != MOSAIC_RMSNORM) MOSAIC_FAIL(MOSAIC_EINVAL, "bad norm kind %d", norm);
  if (dtype == MOSAIC_BF16)
    return norm_bwd_t<bf16>(s, quota, norm, T, h, (const bf16*)x, (const bf16*)gamma, stats, (const bf16*)dy,
                            (const bf16*)R, (bf16*)dx, (bf16*)dgamma, (bf16*)dbeta, (float*)scratch, (bf16*)dxsum, dtype, later);
  return norm_bwd_t<float>(s, quota, norm, T, h, (const float*)x, (const float*)gamma, stats, (const float*)dy,
                           (const float*)R, (float*)dx, (float*)dgamma, (float*)dbeta, (float*)scratch, (float*)dxsum, dtype, later);
}

#define EW_CHECK_VEC(n, dtype)                                                               \
  const int vn__ = (dtype == MOSAIC_BF16) ? 8 : 4;                                           \
  if ((n) % vn__) MOSAIC_FAIL(MOSAIC_EUNSUPPORTED, "element count %lld is not a multiple of %d", (long long)(n), vn__)

mosaic_status launch_gelu_fwd(hipStream_t s, int quota, int dtype, int64_t n, const void* z, void* a) {
  EW_CHECK_VEC(n, dtype);
  if (n == 0) return MOSAIC_OK;
  const int64_t nvec = n / vn__;
  // bf16, striding / in order on 256 and 64 CUs: 68 MB 17.7 / 16.2 us and 51.8 / 44.5, 560 MB 130 / 123 and 423 / 362.  fp32: 160 MB 25.9 / 25.0 and 62.7 /
  // 56.9, but 72 MB 12.5 / 12.7 on 256, and above the last-level cache only on most of the device: 272 MB 45.5 / 46.5 and 116 / 129, 512 MB
  // 97 / 88 and 222 / 230.
  const int64_t bytes = 2 * n * (int64_t)dtype_size(dtype), blocks = ceil_div(nvec, kThreads), mb = (int64_t)1 << 20;
  const bool stride = dtype == MOSAIC_F32 && (quota > 128 ? bytes <= 100 * mb || (bytes > 256 * mb && bytes <= 320 * mb) : bytes > 256 * mb);
  const int grid = stride ? grid_for(quota, 8, blocks) : sweep_grid(s, quota, blocks, bytes).grid;
  if (dtype == MOSAIC_BF16) gelu_fwd_kernel<bf16><<<grid, kThreads, 0, s>>>((const bf16*)z, (bf16*)a, nvec);
  else gelu_fwd_kernel<float><<<grid, kThreads, 0, s>>>((const float*)z, (float*)a, nvec);
  MOSAIC_LAUNCH_CHECK();
  return MOSAIC_OK;
}

mosaic_status launch_gelu_bwd(hipStream_t s, int quota, int dtype, int64_t n, const void* z, const void* da, void* dz) {
  EW_CHECK_VEC(n, dtype);
  if (n == 0) return MOSAIC_OK;
  const int64_t nvec = n / vn__;
  const int grid = grid_for(quota, 8, ceil_div(nvec, kThreads));
  if (dtype == MOSAIC_BF16) gelu_bwd_kernel<bf16><<<grid, kThreads, 0, s>>>((const bf16*)z, (const bf16*)da, (bf16*)dz, nvec);
  else gelu_bwd_kernel<float><<<grid, kThreads, 0, s>>>((const float*)z, (const float*)da, (float*)dz, nvec);
  MOSAIC_LAUNCH_CHECK();
  return MOSAIC_OK;
}

mosaic_status launch_swiglu_fwd(hipStream_t s, int quota, int dtype, int64_t T, int64_t f, const void* gu, void* a) {
  EW_CHECK_VEC(f, dtype);
  if (T * f == 0) return MOSAIC_OK;
  const int fv = (int)(f / vn__);
  // bf16, striding / in order on 256 and 64 CUs: 67 MB 13.9 / 13.4 us and 41.5 / 36.1, 193 MB 35.2 / 33.5 and 114 / 98; fp32 528 MB 105 / 94 and 207 / 192
  const int grid = sweep_grid(s, quota, ceil_div(T * fv, kThreads), 3 * T * f * (int64_t)dtype_size(dtype)).grid;
  if (dtype == MOSAIC_BF16) swiglu_fwd_kernel<bf16><<<grid, kThreads, 0, s>>>((const bf16*)gu, (bf16*)a, T, fv);
  else swiglu_fwd_kernel<float><<<grid, kThreads, 0, s>>>((const float*)gu, (float*)a, T, fv);
  MOSAIC_LAUNCH_CHECK();
  return MOSAIC_OK;
}

mosaic_status launch_swiglu_bwd(hipStream_t s, int quota, int dtype, int64_t T, int64_t f, const void* gu,
                                const void* da, void* dgu) {
  EW_CHECK_VEC(f, dtype);
  if (T * f == 0) return MOSAIC_OK;
  const int fv = (int)(f / vn__);
  const int64_t bytes = 5 * T * f * (int64_t)dtype_size(dtype);
  // bf16 on all CUs only above the last-level cache: striding / in order 112 MB 18.8 / 20.4 us, 177 MB 28.8 / 29.9; on 192 CUs 31.5 / 30.1, on 64 82 / 72
  const Sweep sw = sweep_grid(s, quota, ceil_div(T * fv, kThreads), bytes, dtype == MOSAIC_BF16 && quota > 192 ? kPastCacheBytes : kSweepBytes);
  auto launch = [&](auto type, auto past) {
    typedef decltype(type) E;
    swiglu_bwd_kernel<E, decltype(past)::value><<<sw.grid, kThreads, 0, s>>>((const E*)gu, (const E*)da, (E*)dgu, T, fv);
  };
  auto of_type = [&](auto type) { if (sw.in_order && bytes > kPastCacheBytes) launch(type, std::true_type{}); else launch(type, std::false_type{}); };
  if (dtype == MOSAIC_BF16) of_type(bf16{}); else of_type(float{});
  MOSAIC_LAUNCH_CHECK();
  return MOSAIC_OK;
}

size_t mse_scratch_bytes() { return kMsePartials * sizeof(float); }

mosaic_status launch_mse(hipStream_t s, int quota, int dtype, int64_t n, const void* y, const void* target,
                         void* dy, float* loss, void* scratch, ColReduceList* later) {
  EW_CHECK_VEC(n, dtype);
  if (n == 0) MOSAIC_FAIL(MOSAIC_EINVAL, "mse over zero elements");
  const int64_t nvec = n / vn__;
  const int np = (int)std::min<int64_t>(kMsePartials, ceil_div(nvec, kThreads));      // a function of the size alone
  const int grid = grid_for(quota, 8, np);
  const float scale = (float)(2.0 / (double)n);
  if (dtype == MOSAIC_BF16)
    mse_kernel<bf16><<<grid, kThreads, 0, s>>>((const bf16*)y, (const bf16*)target, (bf16*)dy, (float*)scratch, nvec, np, scale);
  else
    mse_kernel<float><<<grid, kThreads, 0, s>>>((const float*)y, (const float*)target, (float*)dy, (float*)scratch, nvec, np, scale);
  MOSAIC_LAUNCH_CHECK();
  if (later) {
    later->loss_partial = (const float*)scratch; later->loss = loss; later->loss_np = np; later->loss_scale = (float)(1.0 / (double)n);
    return MOSAIC_OK;
  }
  mse_final_kernel<<<1, kThreads, 0, s>>>((const float*)scratch, np, loss, (float)(1.0 / (double)n));
  MOSAIC_LAUNCH_CHECK();
  return MOSAIC_OK;
}

size_t colsum_scratch_bytes(int64_t n) { return (size_t)kColsumMaxParts * (size_t)n * sizeof(float); }

// Long partitions of wide rows are summed in quarters.  A function of the shape: the bits follow it.  Partitions then start so far
// apart, often by a power of two, that waves which walk them in step meet in the same parts of memory; four waves in four places of a
// partition do not.  GELU's pass in us on 256 CUs (on 64), ascending / in quarters: 16384 x 4096 94.2 (208) / 84.1 (209), 32768 x 4096
// 179 (405) / 168 (400), 24000 x 4096 131 (303) / 126 (305), 16384 x 3072 61.0 (158) / 60.2 (160); not so where rows are short or
// partitions are: 32768 x 1024 44.8 (106) / 45.2 (105), 24000 x 1280 39.3 (98) / 41.6 (117), 12000 x 3840 (24 rows) 55 (148) / 59.5 (162).
static bool colsum_quarters(int rp, int64_t n) { return rp >= 28 && n >= 2048; }

mosaic_status launch_colsum(hipStream_t s, int quota, int dtype, int64_t T, int64_t n, const void* X, void* out,
                            void* scratch, ColReduceList* later, bool in_passing) {
  EW_CHECK_VEC(n, dtype);
  if (n == 0) return MOSAIC_OK;
  int rp, np;
  col_partition(T, &rp, &np);
  if (in_passing && later && later->n < ColReduceList::kMax && later->pending.np == 0 && np > 0 && !colsum_quarters(rp, n)) {
    later->pending.X = X; later->pending.partial = (float*)scratch; later->pending.rows = T; later->pending.n = n;
    later->pending.rp = rp; later->pending.np = np; later->pending.ctiles = (int)ceil_div(n, (int64_t)64 * vn__);
    np = -np;
  }
  if (np > 0) {
    const int ctiles = (int)ceil_div(n, (int64_t)64 * vn__);
    // One wave's requests go to four rows a quarter of a partition apart.  Where that is a multiple of 128 KB and the CUs are many, the four
    // waves of a workgroup, which drift apart, are faster: one wave / four, us on 256 (192) CUs, 32768 x 4096 54 (49) / 46 (44),
    // 65536 x 2048 49.3 (47.6) / 46.0 (45.5), 131072 x 2048 103 (105) / 98.5 (99); on 64 CUs 78 / 79, 69.5 / 71.5, 174 / 181.
    const bool quarters = colsum_quarters(rp, n), apart = quota > 128 && (int64_t)rp / 4 * n * (int64_t)dtype_size(dtype) % (128 << 10) == 0;
    const int grid = grid_for(quota, 8, ceil_div((int64_t)np * ctiles, quarters && apart ? 1 : kWaves));
    auto launch = [&](auto type) {
      typedef decltype(type) E;
      if (quarters && apart) colsum_partial_kernel<E, true><<<grid, kThreads, 0, s>>>((const E*)X, (float*)scratch, T, n, rp, np, ctiles);
      else if (quarters) colsum_quarters_kernel<E><<<grid, kThreads, 0, s>>>((const E*)X, (float*)scratch, T, n, rp, np, ctiles);
      else colsum_partial_kernel<E, false><<<grid, kThreads, 0, s>>>((const E*)X, (float*)scratch, T, n, rp, np, ctiles);
    };
    if (dtype == MOSAIC_BF16) launch(bf16{}); else launch(float{});
    MOSAIC_LAUNCH_CHECK();
  }
  return col_reduce(s, quota, dtype, {(const float*)scratch, np < 0 ? -np : np, n, n, n, INT64_MAX, out, nullptr, nullptr}, later);
}

mosaic_status launch_gelu_bwd_colsum(hipStream_t s, int quota, int dtype, int64_t T, int64_t n, const void* z,
                                     const void* da, void* dz, void* colsum, void* scratch, ColReduceList* later, int taps_lo) {
  EW_CHECK_VEC(n, dtype);
  if (n == 0) return MOSAIC_OK;
  if (taps_lo < 0 || (taps_lo > 0 && (T % (2 * (int64_t)taps_lo) || T / 2 >= UINT32_MAX))) MOSAIC_FAIL(MOSAIC_EINVAL, "%lld rows are no whole samples", (long long)T);
  int rp, np;
  col_partition(T, &rp, &np);
  if (np > 0) {
    const uint64_t m_lo = taps_lo > 1 ? ~(uint64_t)0 / (uint64_t)taps_lo + 1 : 0;
    auto launch = [&](auto type, auto bytes, auto once, auto quarters, auto taps) {
      typedef decltype(type) E;
      constexpr int V = decltype(bytes)::value / sizeof(E);
      constexpr bool Q = decltype(quarters)::value;
      const int ctiles = (int)ceil_div(n, (int64_t)64 * V), grid = grid_for(quota, 8, ceil_div((int64_t)np * ctiles, Q ? 1 : kWaves));
      const Along along = take_along(quota, later);
      gelu_bwd_colsum_kernel<E, V, decltype(once)::value, Q, decltype(taps)::value><<<along.blocks + grid, kThreads, 0, s>>>((const E*)z, (const E*)da, (E*)dz, (float*)scratch, T, n, rp, np, ctiles, taps_lo, m_lo, along);
    };
    // Waves on a CU with 8 bytes a lane.  Measured with 8 bytes / 4 bytes a lane, us, waves in brackets: partitions of a whole number of
    // eights 1568 x 3072 14.3 / 13.2 (9), 17.1 / 16.5 (18), 24.1 / 23.4 (37); 12000 x 3840 58.1 / 54 (30), 80.6 / 84 (60); others
    // 4608 x 3072 22.3 / 22.8 (24), 31.0 / 33.1 (48), 4608 x 4096 27.5 / 28.1 (32), 24000 x 1280 44 / 39 (10), 58.2 / 55.9 (20), 98.1 / 99.6 (40);
    // taps 24000 x 1280 57 / 46 (10), 73 / 80 (20), 6748 x 768 24.9 / 24.8 (11), 33.2 / 37.6 (23).
    const double waves = (double)np * (double)ceil_div(n, (int64_t)512 / (int64_t)dtype_size(dtype)) / quota;
    const bool many = waves >= (taps_lo ? 16 : rp % 8 ? 24 : 48), quarters = colsum_quarters(rp, n);
    typedef std::integral_constant<int, 4> Four;
    typedef std::integral_constant<int, 8> Eight;
    typedef std::integral_constant<int, 16> Sixteen;
    auto of_type = [&](auto type, auto taps) {
      if (quarters) launch(type, Sixteen{}, Four{}, std::true_type{}, taps);
      else if (many) launch(type, Eight{}, Four{}, std::false_type{}, taps);
      else launch(type, Four{}, std::conditional_t<decltype(taps)::value, Four, Eight>{}, std::false_type{}, taps);
    };
    auto of_taps = [&](auto type) { if (taps_lo) of_type(type, std::true_type{}); else of_type(type, std::false_type{}); };
    if (dtype == MOSAIC_BF16) of_taps(bf16{}); else of_taps(float{});
    MOSAIC_LAUNCH_CHECK();
  }
  return col_reduce(s, quota, dtype, {(const float*)scratch, np, n, n, n, INT64_MAX, colsum, nullptr, nullptr}, later);
}

// 16-byte accesses where every row of both tensors starts on a 16-byte boundary
static inline bool wide_access(int64_t n, int dtype, const void* a, const void* b) {
  return n % (dtype == MOSAIC_BF16 ? 8 : 4) == 0 && (((uintptr_t)a | (uintptr_t)b) & 15) == 0;
}

mosaic_status launch_unfold(hipStream_t s, int quota, int dtype, int B, int side, int patch, const void* img, void* out, int ld) {
  if (patch <= 0 || side % patch) MOSAIC_FAIL(MOSAIC_EINVAL, "image side %d is not a multiple of patch %d", side, patch);
  const int vn = dtype == MOSAIC_BF16 ? 8 : 4;
  if (ld < 3 * patch * patch || ld % vn || ((uintptr_t)out & 15)) MOSAIC_FAIL(MOSAIC_EINVAL, "patch rows must start on 16-byte boundaries");
  const int64_t g = side / patch, pieces = (int64_t)B * g * g * (ld / vn);
  if (pieces == 0) return MOSAIC_OK;
  const int64_t strip_bytes = (int64_t)patch * side * 2;
  if (dtype == MOSAIC_BF16 && patch % 2 == 0 && patch >= 4 && strip_bytes <= kStripBytes && (uintptr_t)img % 8 == 0) {
    const int64_t strips = 3 * (int64_t)B * g;
    auto magic = [](int d) { return (uint32_t)(((uint64_t)1 << 32) / (uint64_t)d + 1); };
    unfold_strip_kernel<<<grid_for(quota, 4, strips), kThreads, (size_t)strip_bytes, s>>>((const bf16*)img, (bf16*)out, strips, side, patch, ld, magic(patch * patch / 4), magic(patch));
    MOSAIC_LAUNCH_CHECK();
    return MOSAIC_OK;
  }
  const int grid = grid_for(quota, 8, ceil_div(pieces, kThreads));
  const bool small = pieces + (int64_t)grid * kThreads < INT32_MAX;
#define UNFOLD(TT, II) unfold_kernel<TT, II><<<grid, kThreads, 0, s>>>((const TT*)img, (TT*)out, B, side, patch, ld)
  if (dtype == MOSAIC_BF16) { if (small) UNFOLD(bf16, int32_t); else UNFOLD(bf16, int64_t); }
  else { if (small) UNFOLD(float, int32_t); else UNFOLD(float, int64_t); }
#undef UNFOLD
  MOSAIC_LAUNCH_CHECK();
  return MOSAIC_OK;
}

template <typename T, int V>
static void add_pos_t(hipStream_t s, int quota, int B, int64_t per, const void* pos, void* y) {
  const int blocks = (int)ceil_div(per, (int64_t)kThreads * V);
  add_pos_kernel<T, V><<<grid_for(quota, 8, (int64_t)B * blocks), kThreads, 0, s>>>((const T*)pos, (T*)y, B, per, blocks);
}

mosaic_status launch_add_pos(hipStream_t s, int quota, int dtype, int B, int N, int h, const void* pos, void* y) {
  const int64_t per = (int64_t)N * h;
  if (per == 0 || B == 0) return MOSAIC_OK;
  const bool wide = wide_access(per, dtype, pos, y);
  if (dtype == MOSAIC_BF16) { if (wide) add_pos_t<bf16, 8>(s, quota, B, per, pos, y); else add_pos_t<bf16, 1>(s, quota, B, per, pos, y); }
  else { if (wide) add_pos_t<float, 4>(s, quota, B, per, pos, y); else add_pos_t<float, 1>(s, quota, B, per, pos, y); }
  MOSAIC_LAUNCH_CHECK();
  return MOSAIC_OK;
}

template <typename T, int V>
static void pos_grad_t(hipStream_t s, int quota, int B, int64_t per, const void* dy, void* dpos) {
  pos_grad_kernel<T, V><<<grid_for(quota, 8, ceil_div(per, (int64_t)kThreads * V)), kThreads, 0, s>>>((const T*)dy, (T*)dpos, B, per);
}

mosaic_status launch_pos_grad(hipStream_t s, int quota, int dtype, int B, int N, int h, const void* dy, void* dpos) {
  const int64_t per = (int64_t)N * h;
  if (per == 0) return MOSAIC_OK;
  const bool wide = wide_access(per, dtype, dy, dpos);
  if (dtype == MOSAIC_BF16) { if (wide) pos_grad_t<bf16, 8>(s, quota, B, per, dy, dpos); else pos_grad_t<bf16, 1>(s, quota, B, per, dy, dpos); }
  else { if (wide) pos_grad_t<float, 4>(s, quota, B, per, dy, dpos); else pos_grad_t<float, 1>(s, quota, B, per, dy, dpos); }
  MOSAIC_LAUNCH_CHECK();
  return MOSAIC_OK;
}

mosaic_status launch_stem_grad(hipStream_t s, int quota, int dtype, int B, int N, int h, const void* dy, void* dpos, void* colsum, void* scratch) {
  // Rows that start off a 16-byte boundary.  More than 32 samples would be faster here too (48 x 576 x 1024 50.9 -> 42.1 us), but a position's
  // samples are one chain of additions in the bias sums, where the column sums' partitions start at eight rows: it is kept short.
  if (B <= 0 || N <= 0 || h <= 0 || B > 32 || !wide_access(h, dtype, dy, dpos)) {
    MOSAIC_TRY(launch_pos_grad(s, quota, dtype, B, N, h, dy, dpos));
    return launch_colsum(s, quota, dtype, (int64_t)B * N, h, dy, colsum, scratch);
  }
  const int rp = (int)ceil_div(N, kColsumMaxParts), np = (int)ceil_div(N, rp);
  auto launch = [&](auto type) {
    typedef decltype(type) E;
    auto wide = [&](auto bytes) {
      constexpr int V = decltype(bytes)::value / sizeof(E);
      const int ctiles = (int)ceil_div(h, 64 * V), grid = grid_for(quota, 8, ceil_div((int64_t)np * ctiles, kWaves));
      stem_grad_kernel<E, V><<<grid, kThreads, 0, s>>>((const E*)dy, (E*)dpos, (float*)scratch, B, N, h, rp, np, ctiles);
    };
    if (B <= 4) wide(std::integral_constant<int, 16>{});
    else wide(std::integral_constant<int, 4>{});
  };
  if (dtype == MOSAIC_BF16) launch(bf16{}); else launch(float{});
  MOSAIC_LAUNCH_CHECK();
  return col_reduce(s, quota, dtype, {(const float*)scratch, np, h, h, h, INT64_MAX, colsum, nullptr, nullptr}, nullptr);
}
