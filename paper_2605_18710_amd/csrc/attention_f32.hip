// Attention with fp32 arithmetic, any head size up to 128: the fp32 path, and bf16 head sizes and
// tensors that the bf16 matrix-core kernels do not cover.
//
// v_mfma_f32_16x16x4_f32, 16 owned rows (an item) per wave, or per four waves, no LDS and no
// barriers in the loops: scores are formed so that a lane owns one column (lane%16) and four rows (4*(lane/16)+e),
// which is exactly the layout in which the next product wants them as its second operand
// (contraction index e-th instruction: row 4*(lane/16)+e), so probabilities go from one product to
// the next in registers, and row maxima and sums are four values plus two exchanges.
// Forward and dQ own 16 queries and stream keys; dK/dV owns 16 keys and streams queries, for every
// query head of its group in turn.  Every sum has one owner and a fixed order, without atomics.
// P is recomputed from the saved row log-sum-exp; D_i = sum_c dO_ic O_ic is formed by the dQ
// kernel, which runs first, and read by the dK/dV kernel.
//
// What bounds it: the fp32 workloads have few rows (2 x 128 tokens x 4 heads = 64 items), so a
// kernel is one chain of load latency, products and softmax per streamed block.  The streamed
// rows of the next block are requested before the current block's products, and the second
// reading of the block's rows (in the other orientation) is in flight under them.  Where items are few, four waves share
// one, each with every fourth step over the streamed rows, and add their sums in wave order: B2 N128 H4 d32 forward
// 9.1 -> 5.3 us, backward 14.6 -> 7.0.  At that size, one wave to an item: forward 29 -> 10.1 us, dQ 25 -> 10.7,
// dK/dV 41 -> 13.7 against workgroups of 16 rows that formed each score by scalar FMA over LDS (launches of 4.5 us included).  Longer rows and the bf16 head sizes
// that come here, forward and backward in us, against those workgroups: fp32 B4 N1500 H8 d80 3944 -> 529 and
// 19622 -> 1868, fp32 B1 N2048 H8/2 d128 causal 2442 -> 308 and 13313 -> 2253; bf16 B8 N1500 H16 d80 15614 -> 3484 and
// 74581 -> 14185, B2 N576 H16 d72 733 -> 206 and 2852 -> 870.
#include <algorithm>
#include <type_traits>
#include "kernels.h"

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ f32x4 mfma4(f32x4 a, f32x4 b, f32x4 c) {
#pragma unroll
  for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], c, 0, 0, 0);
  return c;
}

// columns c .. c+3 of a row of d; zero past the end and for rows that do not exist
template <typename T, bool VEC>
__device__ __forceinline__ f32x4 cols4(const T* row, int c, int d, bool live) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (!live) return v;
  if constexpr (VEC) {
    typedef T vec __attribute__((ext_vector_type(4)));
    if (c < d) {
      const vec x = *reinterpret_cast<const vec*>(row + c);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = (float)x[e];
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) if (c + e < d) v[e] = to_f32(row[c + e]);
  }
  return v;
}
template <typename T, bool VEC>
__device__ __forceinline__ void put4(T* row, int c, int d, f32x4 v) {
  if constexpr (VEC) {
    typedef T vec __attribute__((ext_vector_type(4)));
    if (c < d) {
      vec o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (T)v[e];
      *reinterpret_cast<vec*>(row + c) = o;
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) if (c + e < d) row[c + e] = from_f32<T>(v[e]);
  }
}
// DB blocks of 16 columns of one row: lane group g holds columns 16s + 4g .. +3
template <typename T, int DB, bool VEC>
__device__ __forceinline__ void row_frag(f32x4 (&f)[DB], const T* row, int g, int d, bool live) {
#pragma unroll
  for (int s = 0; s < DB; ++s) f[s] = cols4<T, VEC>(row, 16 * s + 4 * g, d, live);
}
// the other orientation: column 16s + lane%16 of rows r0 + 4g + e
template <typename T, int DB>
__device__ __forceinline__ void col_frag(f32x4 (&f)[DB], const T* base, int64_t rs, int r0, int N, int lr, int g, int d) {
#pragma unroll
  for (int s = 0; s < DB; ++s)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = r0 + 4 * g + e, c = 16 * s + lr;
      f[s][e] = (r < N && c < d) ? to_f32(base[(int64_t)r * rs + c]) : 0.f;
    }
}
__device__ __forceinline__ float groups_max(float v) { v = fmaxf(v, __shfl_xor(v, 16, 64)); return fmaxf(v, __shfl_xor(v, 32, 64)); }
__device__ __forceinline__ float groups_sum(float v) { v += __shfl_xor(v, 16, 64); return v + __shfl_xor(v, 32, 64); }

// streamed blocks of 16 rows per step: two at small head sizes, where their fragments leave room
template <int DB> constexpr int kBlocks = DB <= 2 ? 2 : 1;

struct AttnArgs {
  int B, N, H, Hkv, d, causal;
  float scale;
  int tiles;                 // tiles of 16 rows
};

// An item's steps over the streamed rows go to SPLIT sums, every SPLIT-th to each, which are added in order: with WAVES = SPLIT each wave
// forms one and they meet in LDS; with WAVES = 1 one wave forms them in turn, with the same additions.
// sums[w][b][lane]: block b of 16 x 16 values of wave w.
template <int SPLIT, int NB>
__device__ __forceinline__ void add_waves(f32x4 (&v)[NB], f32x4* sums, int wave, int lane) {
#pragma unroll
  for (int b = 0; b < NB; ++b) sums[(wave * NB + b) * 64 + lane] = v[b];
  __syncthreads();
  // wave w finishes blocks w, w + SPLIT, ...; the others' values are not used
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    if (b % SPLIT != wave) continue;
    v[b] = sums[b * 64 + lane];
#pragma unroll
    for (int w = 1; w < SPLIT; ++w) v[b] += sums[(w * NB + b) * 64 + lane];
  }
  __syncthreads();
}
template <int WAVES> __device__ __forceinline__ bool mine(int block, int wave) { return WAVES == 1 || block % WAVES == wave; }
template <int WAVES, int DB> constexpr int kSums = WAVES == 1 ? 1 : WAVES * DB * 64;
template <int N>
__device__ __forceinline__ float top_of(const float (&m)[N]) {
  float top = m[0];
#pragma unroll
  for (int w = 1; w < N; ++w) top = fmaxf(top, m[w]);
  return top;
}
template <int N>
__device__ __forceinline__ float total_of(const float (&m)[N], const float (&l)[N], float top) {
#pragma clang fp contract(off)
  float total = 0.f;
#pragma unroll
  for (int w = 0; w < N; ++w) total += l[w] == 0.f ? 0.f : l[w] * expf(m[w] - top);
  return total;
}
__device__ __forceinline__ float weight_of(float m, float top) { return m == -INFINITY ? 0.f : expf(m - top); }

template <typename T, int DB, bool VEC, int SPLIT, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void attn_fwd_f32(const T* __restrict__ qkv, T* __restrict__ O, float* __restrict__ lse, AttnArgs p) {
  constexpr int KB = kBlocks<DB>, SUMS = SPLIT / WAVES;
  const int lane = threadIdx.x & 63, lr = lane & 15, g = lane >> 4, wave = WAVES == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  __shared__ f32x4 sums[kSums<WAVES, DB>];
  __shared__ float rows_m[WAVES][16], rows_l[WAVES][16];
  // rows are [q (H heads) | k (Hkv heads) | v (Hkv heads)]; query head t uses key/value head t / (H/Hkv)
  const int N = p.N, d = p.d, GQ = p.H / p.Hkv;
  const int64_t rs = (int64_t)(p.H + 2 * p.Hkv) * d;
  const int64_t items = (int64_t)p.B * p.H * p.tiles;
  for (int64_t item = blockIdx.x; item < items; item += gridDim.x) {
    const int64_t hb = item / p.tiles;
    // the last tile of a causal row is the longest: it starts first
    const int qt = p.causal ? p.tiles - 1 - (int)(item - hb * p.tiles) : (int)(item - hb * p.tiles);
    const int hd = (int)(hb % p.H);
    const int64_t b = hb / p.H;
    const T* rowb = qkv + b * N * rs;
    const T* kb_ = rowb + (int64_t)p.H * d + (hd / GQ) * d;
    const T* vb_ = kb_ + (int64_t)p.Hkv * d;
    const int i = qt * 16 + lr;
    f32x4 qf[DB], kf[KB][DB], o_[SUMS][DB];
    row_frag<T, DB, VEC>(qf, rowb + (int64_t)i * rs + hd * d, g, d, i < N);
    float m_[SUMS], l_[SUMS];
    const int kv_end = p.causal ? min(N, qt * 16 + 16) : N;
    auto k_rows = [&](int j0) {
#pragma unroll
      for (int u = 0; u < KB; ++u) {
        const int j = j0 + 16 * u + lr;
        row_frag<T, DB, VEC>(kf[u], kb_ + (int64_t)j * rs, g, d, j < kv_end);
      }
    };
#pragma unroll
    for (int x = 0; x < SUMS; ++x) {
      f32x4 (&o)[DB] = o_[x];
      float m = -INFINITY, l = 0.f;
#pragma unroll
      for (int s = 0; s < DB; ++s) o[s] = f32x4{0.f, 0.f, 0.f, 0.f};
      const int first = (SUMS == 1 ? wave : x) * 16 * KB;
      if (x == 0 && (SPLIT == 1 || first < kv_end)) k_rows(first);       // a later sum's were requested under the last step of the one before
      for (int j0 = first; j0 < kv_end; j0 += 16 * KB * SPLIT) {
        f32x4 vt[KB][DB], sc[KB];
#pragma unroll
        for (int u = 0; u < KB; ++u) col_frag<T, DB>(vt[u], vb_, rs, j0 + 16 * u, kv_end, lr, g, d);
#pragma unroll
        for (int u = 0; u < KB; ++u) {
          sc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int s = 0; s < DB; ++s) sc[u] = mfma4(kf[u][s], qf[s], sc[u]);
        }
        if (j0 + 16 * KB * SPLIT < kv_end) k_rows(j0 + 16 * KB * SPLIT);
        else if (x + 1 < SUMS && first + 16 * KB < kv_end) k_rows(first + 16 * KB);
        float mx = -INFINITY;
#pragma unroll
        for (int u = 0; u < KB; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int j = j0 + 16 * u + 4 * g + e;
            sc[u][e] = (j >= N || (p.causal && j > i)) ? -INFINITY : sc[u][e] * p.scale;
            mx = fmaxf(mx, sc[u][e]);
          }
        const float mn = fmaxf(m, groups_max(mx));
        // a row that has seen no unmasked key yet keeps m = -inf; exp(-inf - -inf) is avoided
        const float corr = (m == -INFINITY) ? 0.f : expf(m - mn);
        float ps = 0.f;
#pragma unroll
        for (int u = 0; u < KB; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            sc[u][e] = (sc[u][e] == -INFINITY) ? 0.f : expf(sc[u][e] - mn);
            ps += sc[u][e];
          }
        l = l * corr + ps;
        m = mn;
#pragma unroll
        for (int s = 0; s < DB; ++s) {
          o[s] *= corr;
#pragma unroll
          for (int u = 0; u < KB; ++u) o[s] = mfma4(vt[u][s], sc[u], o[s]);
        }
      }
      m_[x] = m;
      l_[x] = groups_sum(l);                 // every lane group has summed its own keys
    }
    f32x4 (&o)[DB] = o_[0];
    float m = m_[0], l = l_[0];
    // the sums brought to one reference; one without keys has l = 0 (a NaN among its scores: l = NaN, m = -inf)
    if constexpr (WAVES > 1) {
      if (g == 0) { rows_m[wave][lr] = m; rows_l[wave][lr] = l; }
      __syncthreads();
      float ms[SPLIT], ls[SPLIT];
#pragma unroll
      for (int w = 0; w < SPLIT; ++w) { ms[w] = rows_m[w][lr]; ls[w] = rows_l[w][lr]; }
      const float top = top_of(ms);
      l = total_of(ms, ls, top);
#pragma unroll
      for (int s = 0; s < DB; ++s) o[s] *= weight_of(m, top);
      m = top;
      add_waves<SPLIT, DB>(o, sums, wave, lane);       // its barriers also keep the rows' values until all have read them
    } else if constexpr (SPLIT > 1) {
#pragma clang fp contract(off)
      const float top = top_of(m_);
      l = total_of(m_, l_, top);
      m = top;
#pragma unroll
      for (int x = 0; x < SPLIT; ++x) {
        const float w = weight_of(m_[x], top);
#pragma unroll
        for (int s = 0; s < DB; ++s) {
          const f32x4 v = o_[x][s] * w;
          o[s] = x == 0 ? v : o[s] + v;
        }
      }
    }
    if (i < N) {
      const float inv = 1.0f / l;
      T* row = O + (b * N + i) * (int64_t)p.H * d + hd * d;
#pragma unroll
      for (int s = 0; s < DB; ++s) if (mine<WAVES>(s, wave)) put4<T, VEC>(row, 16 * s + 4 * g, d, o[s] * inv);
      if (g == 0 && wave == 0) lse[hb * N + i] = m + logf(l);
    }
  }
}

// workgroups first .. first + count - 1 of the launch
struct Share { int first, count; };

template <typename T, int DB, bool VEC, int SPLIT, int WAVES>
__device__ __forceinline__ void dq_items(const T* __restrict__ qkv, const T* __restrict__ O, const T* __restrict__ dO,
                                         const float* __restrict__ lse, float* __restrict__ delta, T* __restrict__ dqkv, const AttnArgs& p, Share sh, f32x4* sums) {
  constexpr int KB = kBlocks<DB>, SUMS = SPLIT / WAVES;
  const int lane = threadIdx.x & 63, lr = lane & 15, g = lane >> 4, wave = WAVES == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int N = p.N, d = p.d, GQ = p.H / p.Hkv;
  const int64_t rs = (int64_t)(p.H + 2 * p.Hkv) * d, h = (int64_t)p.H * d;
  const int64_t items = (int64_t)p.B * p.H * p.tiles;
  for (int64_t item = (int)blockIdx.x - sh.first; item < items; item += sh.count) {
    const int64_t hb = item / p.tiles;
    const int qt = p.causal ? p.tiles - 1 - (int)(item - hb * p.tiles) : (int)(item - hb * p.tiles);
    const int hd = (int)(hb % p.H);
    const int64_t b = hb / p.H;
    const T* rowb = qkv + b * N * rs;
    const T* kb_ = rowb + h + (hd / GQ) * d;
    const T* vb_ = kb_ + (int64_t)p.Hkv * d;
    const int i = qt * 16 + lr;
    f32x4 qf[DB], dof[DB], kf[KB][DB], vf[KB][DB], dq[DB];
    row_frag<T, DB, VEC>(qf, rowb + (int64_t)i * rs + hd * d, g, d, i < N);
    row_frag<T, DB, VEC>(dof, dO + (b * N + i) * h + hd * d, g, d, i < N);
    float dl = 0.f;
    {
      f32x4 of[DB];
      row_frag<T, DB, VEC>(of, O + (b * N + i) * h + hd * d, g, d, i < N);
#pragma unroll
      for (int s = 0; s < DB; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e) dl = fmaf(dof[s][e], of[s][e], dl);
    }
    dl = groups_sum(dl);
    if (delta && i < N && g == 0 && wave == 0) delta[hb * N + i] = dl;
    const float li = i < N ? lse[hb * N + i] : 0.f;
    const int kv_end = p.causal ? min(N, qt * 16 + 16) : N;
    auto kv_rows = [&](int j0) {
#pragma unroll
      for (int u = 0; u < KB; ++u) {
        const int j = j0 + 16 * u + lr;
        row_frag<T, DB, VEC>(kf[u], kb_ + (int64_t)j * rs, g, d, j < kv_end);
        row_frag<T, DB, VEC>(vf[u], vb_ + (int64_t)j * rs, g, d, j < kv_end);
      }
    };
#pragma unroll 1        // unrolled, the addresses of all sums' rows take the registers of a wave per SIMD
    for (int x = 0; x < SUMS; ++x) {
      const int first = (SUMS == 1 ? wave : x) * 16 * KB;
      f32x4 sum[DB];
#pragma unroll
      for (int s = 0; s < DB; ++s) sum[s] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (x == 0 && (SPLIT == 1 || first < kv_end)) kv_rows(first);
      for (int j0 = first; j0 < kv_end; j0 += 16 * KB * SPLIT) {
        f32x4 kt[KB][DB], sc[KB], dp[KB];
#pragma unroll
        for (int u = 0; u < KB; ++u) col_frag<T, DB>(kt[u], kb_, rs, j0 + 16 * u, kv_end, lr, g, d);
#pragma unroll
        for (int u = 0; u < KB; ++u) {
          sc[u] = f32x4{0.f, 0.f, 0.f, 0.f}; dp[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int s = 0; s < DB; ++s) { sc[u] = mfma4(kf[u][s], qf[s], sc[u]); dp[u] = mfma4(vf[u][s], dof[s], dp[u]); }
        }
        if (j0 + 16 * KB * SPLIT < kv_end) kv_rows(j0 + 16 * KB * SPLIT);
        else if (x + 1 < SUMS && first + 16 * KB < kv_end) kv_rows(first + 16 * KB);
#pragma unroll
        for (int u = 0; u < KB; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int j = j0 + 16 * u + 4 * g + e;
            const bool masked = i >= N || j >= N || (p.causal && j > i);
            sc[u][e] = masked ? 0.f : expf(sc[u][e] * p.scale - li) * (dp[u][e] - dl);
          }
#pragma unroll
        for (int s = 0; s < DB; ++s)
#pragma unroll
          for (int u = 0; u < KB; ++u) sum[s] = mfma4(kt[u][s], sc[u], sum[s]);
      }
#pragma unroll
      for (int s = 0; s < DB; ++s) dq[s] = x == 0 ? sum[s] : dq[s] + sum[s];
    }
    if constexpr (WAVES > 1) add_waves<SPLIT, DB>(dq, sums, wave, lane);
    if (i < N) {
      T* row = dqkv + (b * N + i) * rs + hd * d;
#pragma unroll
      for (int s = 0; s < DB; ++s) if (mine<WAVES>(s, wave)) put4<T, VEC>(row, 16 * s + 4 * g, d, dq[s] * p.scale);
    }
  }
}

// OWN_DELTA: the row sums D_i are formed here from dO and O, with the additions of dq_items, and not read
template <typename T, int DB, bool VEC, bool OWN_DELTA, int SPLIT, int WAVES>
__device__ __forceinline__ void dkv_items(const T* __restrict__ qkv, const T* __restrict__ O, const T* __restrict__ dO, const float* __restrict__ lse,
                                          const float* __restrict__ delta, T* __restrict__ dqkv, const AttnArgs& p, Share sh, f32x4* sums) {
  constexpr int QB = kBlocks<DB>, SUMS = SPLIT / WAVES;
  const int lane = threadIdx.x & 63, lr = lane & 15, g = lane >> 4, wave = WAVES == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int N = p.N, d = p.d, GQ = p.H / p.Hkv;
  const int64_t rs = (int64_t)(p.H + 2 * p.Hkv) * d, h = (int64_t)p.H * d;
  const int64_t items = (int64_t)p.B * p.Hkv * p.tiles;
  for (int64_t item = (int)blockIdx.x - sh.first; item < items; item += sh.count) {
    const int64_t hb = item / p.tiles;
    const int kt = (int)(item - hb * p.tiles);             // the first tile of a causal row has the most queries
    const int kvh = (int)(hb % p.Hkv);
    const int64_t b = hb / p.Hkv;
    const T* rowb = qkv + b * N * rs;
    const int j = kt * 16 + lr;
    f32x4 kf[DB], vf[DB], dk[DB], dv[DB], qf[QB][DB], of[QB][DB], out[OWN_DELTA ? QB : 1][DB];
    row_frag<T, DB, VEC>(kf, rowb + (int64_t)j * rs + h + kvh * d, g, d, j < N);
    row_frag<T, DB, VEC>(vf, rowb + (int64_t)j * rs + h + (int64_t)(p.Hkv + kvh) * d, g, d, j < N);
#pragma unroll 1
    for (int x = 0; x < SUMS; ++x) {
      f32x4 sk[DB], sv[DB];
#pragma unroll
      for (int s = 0; s < DB; ++s) { sk[s] = f32x4{0.f, 0.f, 0.f, 0.f}; sv[s] = f32x4{0.f, 0.f, 0.f, 0.f}; }
      const int i_begin = (p.causal ? kt * 16 : 0) + (SUMS == 1 ? wave : x) * 16 * QB;
      // every query head of the group in turn, query blocks ascending inside a head
      for (int hd = kvh * GQ; hd < (kvh + 1) * GQ; ++hd) {
        const T* qb_ = rowb + hd * d;
        const T* db_ = dO + b * N * h + hd * d;
        const float* lse_ = lse + (b * p.H + hd) * N;
        const float* del_ = OWN_DELTA ? nullptr : delta + (b * p.H + hd) * N;
        const T* ob_ = O + b * N * h + hd * d;
        auto q_rows = [&](int i0) {
#pragma unroll
          for (int u = 0; u < QB; ++u) {
            const int i = i0 + 16 * u + lr;
            row_frag<T, DB, VEC>(qf[u], qb_ + (int64_t)i * rs, g, d, i < N);
            row_frag<T, DB, VEC>(of[u], db_ + (int64_t)i * h, g, d, i < N);
            if constexpr (OWN_DELTA) row_frag<T, DB, VEC>(out[u], ob_ + (int64_t)i * h, g, d, i < N);
          }
        };
        if ((x == 0 || GQ > 1) && (SPLIT == 1 || i_begin < N)) q_rows(i_begin);
        for (int i0 = i_begin; i0 < N; i0 += 16 * QB * SPLIT) {
          f32x4 qt[QB][DB], ot[QB][DB], sc[QB], dp[QB], li[QB], dl[QB];
#pragma unroll
          for (int u = 0; u < QB; ++u) {
            col_frag<T, DB>(ot[u], db_, h, i0 + 16 * u, N, lr, g, d);
            col_frag<T, DB>(qt[u], qb_, rs, i0 + 16 * u, N, lr, g, d);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int i = i0 + 16 * u + 4 * g + e;
              li[u][e] = i < N ? lse_[i] : 0.f;
              if constexpr (!OWN_DELTA) dl[u][e] = i < N ? del_[i] : 0.f;
            }
            if constexpr (OWN_DELTA) {                     // of row lr of the block in every lane group, then of this lane's rows
              float t = 0.f;
#pragma unroll
              for (int s = 0; s < DB; ++s)
#pragma unroll
                for (int e = 0; e < 4; ++e) t = fmaf(of[u][s][e], out[u][s][e], t);
              t = groups_sum(t);
#pragma unroll
              for (int e = 0; e < 4; ++e) dl[u][e] = __shfl(t, 4 * g + e, 64);
            }
          }
#pragma unroll
          for (int u = 0; u < QB; ++u) {
            sc[u] = f32x4{0.f, 0.f, 0.f, 0.f}; dp[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < DB; ++s) { sc[u] = mfma4(qf[u][s], kf[s], sc[u]); dp[u] = mfma4(of[u][s], vf[s], dp[u]); }
          }
          if (i0 + 16 * QB * SPLIT < N) q_rows(i0 + 16 * QB * SPLIT);
          else if (x + 1 < SUMS && GQ == 1 && i_begin + 16 * QB < N) q_rows(i_begin + 16 * QB);
#pragma unroll
          for (int u = 0; u < QB; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int i = i0 + 16 * u + 4 * g + e;
              const bool masked = i >= N || j >= N || (p.causal && j > i);
              sc[u][e] = masked ? 0.f : expf(sc[u][e] * p.scale - li[u][e]);
              dp[u][e] = sc[u][e] * (dp[u][e] - dl[u][e]);
            }
#pragma unroll
          for (int s = 0; s < DB; ++s)
#pragma unroll
            for (int u = 0; u < QB; ++u) { sv[s] = mfma4(ot[u][s], sc[u], sv[s]); sk[s] = mfma4(qt[u][s], dp[u], sk[s]); }
        }
      }
#pragma unroll
      for (int s = 0; s < DB; ++s) { dk[s] = x == 0 ? sk[s] : dk[s] + sk[s]; dv[s] = x == 0 ? sv[s] : dv[s] + sv[s]; }
    }
    if constexpr (WAVES > 1) { add_waves<SPLIT, DB>(dk, sums, wave, lane); add_waves<SPLIT, DB>(dv, sums, wave, lane); }
    if (j < N) {
      T* row = dqkv + (b * N + j) * rs + h + kvh * d;
#pragma unroll
      for (int s = 0; s < DB; ++s) {
        if (!mine<WAVES>(s, wave)) continue;
        put4<T, VEC>(row, 16 * s + 4 * g, d, dk[s] * p.scale);
        put4<T, VEC>(row + (int64_t)p.Hkv * d, 16 * s + 4 * g, d, dv[s]);
      }
    }
  }
}

template <typename T, int DB, bool VEC, int SPLIT, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void attn_bwd_dq_f32(const T* __restrict__ qkv, const T* __restrict__ O, const T* __restrict__ dO,
                                                              const float* __restrict__ lse, float* __restrict__ delta, T* __restrict__ dqkv, AttnArgs p) {
  __shared__ f32x4 sums[kSums<WAVES, DB>];
  dq_items<T, DB, VEC, SPLIT, WAVES>(qkv, O, dO, lse, delta, dqkv, p, {0, (int)gridDim.x}, sums);
}
template <typename T, int DB, bool VEC, int SPLIT, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void attn_bwd_dkv_f32(const T* __restrict__ qkv, const T* __restrict__ dO, const float* __restrict__ lse,
                                                               const float* __restrict__ delta, T* __restrict__ dqkv, AttnArgs p) {
  __shared__ f32x4 sums[kSums<WAVES, DB>];
  dkv_items<T, DB, VEC, false, SPLIT, WAVES>(qkv, nullptr, dO, lse, delta, dqkv, p, {0, (int)gridDim.x}, sums);
}
// Both in one launch where every item has wave slots of its own: the two chains, each a launch's latency and a few blocks
// long, then run side by side, at the price of reading O for dK/dV as well.  B2 N128 H4 d32, one wave to an item: 10.3 + 13.7 us -> 15.0; four 7.0.
template <int DB, int SPLIT, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void attn_bwd_f32(const float* __restrict__ qkv, const float* __restrict__ O, const float* __restrict__ dO,
                                                           const float* __restrict__ lse, float* __restrict__ delta, float* __restrict__ dqkv, AttnArgs p, int ndkv) {
  __shared__ f32x4 sums[kSums<WAVES, DB>];
  if ((int)blockIdx.x < ndkv) dkv_items<float, DB, true, true, SPLIT, WAVES>(qkv, O, dO, lse, nullptr, dqkv, p, {0, ndkv}, sums);
  else dq_items<float, DB, true, SPLIT, WAVES>(qkv, O, dO, lse, delta, dqkv, p, {ndkv, (int)gridDim.x - ndkv}, sums);
}

// four columns per access where every head of every row starts on such a boundary
template <typename T>
bool four_columns(int d, const void* a, const void* b, const void* c, const void* e) {
  return d % 4 == 0 && (((uintptr_t)a | (uintptr_t)b | (uintptr_t)c | (uintptr_t)e) & (4 * sizeof(T) - 1)) == 0;
}

// Four sums to an item where the items are few (with 1024 waves every SIMD of the device has one): a function of the shape, because the
// order of the additions follows it.  How many waves form them follows the share of the CUs as well.  Forward: four while four to a SIMD hold
// all items, and beyond where the rows are long (B2 N192 H6 d32 causal on 16 CUs 20.2 / 17.4 / 22.9 us).  Backward: four where both gradients then fit side by side, or the rows are long.  Otherwise one wave to an item: waves that
// wait for each other at few steps a wave cost more than they hide.  One sum / four waves / four sums by one wave, us: B8 N48 H8 d64
// causal on 16 CUs 11.8 / 22.3 / 14.1, backward 38.5 / 69.8 / 42.2; B1 N64 H64 d16 on 64 backward 14.7 / 17.0 / 16.5, on 128 6.4 / 10.9 / 8.0; B4 N256 H4
// d64 causal on 64 32.5 / 23.3 / -, backward 97 / 71 / -, on 16 65.6 / 81.5 / 72.2 and 230 / 263 / 235;
// B1 N200 H4 d32 on 32 backward 25.0 / 23.9 / 25.8, B2 N128 H4 d64 22.6 / 26.0 / 24.1.
bool split_items(const AttnArgs& p) { return p.N > 32 && p.d <= 64 && (int64_t)p.B * p.H * p.tiles <= 256; }

template <typename T, int DB, bool VEC>
mosaic_status fwd_t(hipStream_t s, int quota, const AttnArgs& p, const void* qkv, void* O, float* lse) {
  const int64_t items = (int64_t)p.B * p.H * p.tiles;
  bool split = false;
  if constexpr (std::is_same<T, float>::value && DB <= 4) {
    split = split_items(p);
    const int64_t fit = (p.N < 192 ? 4 : DB <= 2 ? 16 : 6) * (int64_t)quota;
    if (split && items <= fit) attn_fwd_f32<T, DB, VEC, 4, 4><<<grid_for(quota, 4, items), 256, 0, s>>>((const T*)qkv, (T*)O, lse, p);
    else if (split) attn_fwd_f32<T, DB, VEC, 4, 1><<<grid_for(quota, 8, items), 64, 0, s>>>((const T*)qkv, (T*)O, lse, p);
  }
  if (!split) attn_fwd_f32<T, DB, VEC, 1, 1><<<grid_for(quota, 8, items), 64, 0, s>>>((const T*)qkv, (T*)O, lse, p);
  MOSAIC_LAUNCH_CHECK();
  return MOSAIC_OK;
}

template <typename T, int DB, bool VEC, int SPLIT, int WAVES>
mosaic_status bwd_split_t(hipStream_t s, int quota, const AttnArgs& p, const void* qkv, const void* O, const float* lse, const void* dO,
                          void* dqkv, float* delta) {
  const int64_t ndq = (int64_t)p.B * p.H * p.tiles, ndkv = (int64_t)p.B * p.Hkv * p.tiles;
  if constexpr (std::is_same<T, float>::value && VEC && DB <= 4) {
    // one wave per SIMD at most; two where four waves share an item
    if ((ndq + ndkv) * WAVES <= (int64_t)quota * (WAVES > 1 ? 8 : 4)) {
      attn_bwd_f32<DB, SPLIT, WAVES><<<(int)(ndq + ndkv), 64 * WAVES, 0, s>>>((const float*)qkv, (const float*)O, (const float*)dO, lse, delta, (float*)dqkv, p, (int)ndkv);
      MOSAIC_LAUNCH_CHECK();
      return MOSAIC_OK;
    }
  }
  constexpr int PER_CU = WAVES > 1 ? 2 : 8;
  attn_bwd_dq_f32<T, DB, VEC, SPLIT, WAVES><<<grid_for(quota, PER_CU, ndq), 64 * WAVES, 0, s>>>((const T*)qkv, (const T*)O, (const T*)dO, lse, delta, (T*)dqkv, p);
  MOSAIC_LAUNCH_CHECK();
  attn_bwd_dkv_f32<T, DB, VEC, SPLIT, WAVES><<<grid_for(quota, PER_CU, ndkv), 64 * WAVES, 0, s>>>((const T*)qkv, (const T*)dO, lse, delta, (T*)dqkv, p);
  MOSAIC_LAUNCH_CHECK();
  return MOSAIC_OK;
}

template <typename T, int DB, bool VEC>
mosaic_status bwd_t(hipStream_t s, int quota, const AttnArgs& p, const void* qkv, const void* O, const float* lse, const void* dO,
                    void* dqkv, float* delta) {
  if constexpr (std::is_same<T, float>::value && DB <= 4) {
    const int64_t ndq = (int64_t)p.B * p.H * p.tiles, ndkv = (int64_t)p.B * p.Hkv * p.tiles;
    const bool four = 4 * (ndq + ndkv) <= 8 * (int64_t)quota || (p.N >= 192 && ndq <= 4 * (int64_t)quota);
    if (split_items(p) && four) return bwd_split_t<T, DB, VEC, 4, 4>(s, quota, p, qkv, O, lse, dO, dqkv, delta);
    if (split_items(p)) return bwd_split_t<T, DB, VEC, 4, 1>(s, quota, p, qkv, O, lse, dO, dqkv, delta);
  }
  return bwd_split_t<T, DB, VEC, 1, 1>(s, quota, p, qkv, O, lse, dO, dqkv, delta);
}

// column blocks of 16 that a head needs, rounded up to an instantiated count
#define WITH_BLOCKS(CALL)                       \
  if (p.d <= 16) return CALL(1);                \
  if (p.d <= 32) return CALL(2);                \
  if (p.d <= 64) return CALL(4);                \
  return CALL(8)

template <typename T, bool VEC>
mosaic_status fwd_d(hipStream_t s, int quota, const AttnArgs& p, const void* qkv, void* O, float* lse) {
#define CALL(DB) (fwd_t<T, DB, VEC>(s, quota, p, qkv, O, lse))
  WITH_BLOCKS(CALL);
#undef CALL
}

template <typename T, bool VEC>
mosaic_status bwd_d(hipStream_t s, int quota, const AttnArgs& p, const void* qkv, const void* O, const float* lse, const void* dO,
                    void* dqkv, float* delta) {
#define CALL(DB) (bwd_t<T, DB, VEC>(s, quota, p, qkv, O, lse, dO, dqkv, delta))
  WITH_BLOCKS(CALL);
#undef CALL
}

AttnArgs attn_args(int B, int N, int H, int Hkv, int d, int causal) {
  return {B, N, H, Hkv, d, causal, 1.0f / sqrtf((float)d), (int)ceil_div(N, 16)};
}

}  // namespace

mosaic_status launch_attention_fwd_f32(hipStream_t s, int quota, int dtype, int B, int N, int H, int Hkv, int d,
                                       int causal, const void* qkv, void* O, float* lse) {
  const AttnArgs p = attn_args(B, N, H, Hkv, d, causal);
  if (dtype == MOSAIC_BF16)
    return four_columns<bf16>(d, qkv, O, O, O) ? fwd_d<bf16, true>(s, quota, p, qkv, O, lse) : fwd_d<bf16, false>(s, quota, p, qkv, O, lse);
  return four_columns<float>(d, qkv, O, O, O) ? fwd_d<float, true>(s, quota, p, qkv, O, lse) : fwd_d<float, false>(s, quota, p, qkv, O, lse);
}

mosaic_status launch_attention_bwd_f32(hipStream_t s, int quota, int dtype, int B, int N, int H, int Hkv, int d,
                                       int causal, const void* qkv, const void* O, const float* lse,
                                       const void* dO, void* dqkv, float* delta) {
  const AttnArgs p = attn_args(B, N, H, Hkv, d, causal);
  if (dtype == MOSAIC_BF16)
    return four_columns<bf16>(d, qkv, O, dO, dqkv) ? bwd_d<bf16, true>(s, quota, p, qkv, O, lse, dO, dqkv, delta)
                                                   : bwd_d<bf16, false>(s, quota, p, qkv, O, lse, dO, dqkv, delta);
  return four_columns<float>(d, qkv, O, dO, dqkv) ? bwd_d<float, true>(s, quota, p, qkv, O, lse, dO, dqkv, delta)
                                                  : bwd_d<float, false>(s, quota, p, qkv, O, lse, dO, dqkv, delta);
}
