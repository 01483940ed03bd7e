// Contractions with fp32 arithmetic: the fp32 path, and the bf16 shapes that the bf16 kernels do
// not take (widths that are not a multiple of 8, unaligned tensors, extents beyond 32 bits).
//
// v_mfma_f32_16x16x4_f32: fp32 products and sums, no narrower type anywhere.  Four waves share a
// square output tile.  A lane's four consecutive k-values feed four consecutive instructions:
// instruction s of a 16-wide k-step contracts k = s, 4+s, 8+s, 12+s; both operands agree on that
// order, so each output is a fixed sum that depends on the sizes alone.
//
// What bounds it: the fp32 workloads are a few hundred rows wide, every product is a chain of
// latencies (load, barrier, matrix instructions, store) behind a launch that costs 4 us or more whatever it does.  So what stands
// around a product in a layer (norm in front, activation or its derivative behind) shares its launch; tiles are small
// enough to give most CUs one; and products of up to 512 blocks of 16 x 16 are summed in shares of the contraction, which
// eight waves take side by side where the CUs hold all blocks (gemm_f32_share_tile).  32 x 32 tiles: four waves, a K-tile is 64 deep and
// the next one is requested before the current one is multiplied.  Products with at least two 64 x 64 tiles per CU take those:
// twice the flops per LDS byte (rule and figures in launch_t).
// A decoder layer of 256 rows, width 128, MLP 384 (forward, loss, backward): 19 launches, 92.8 us -> 14, 62.3.
#include <algorithm>
#include <type_traits>
#include "activations.h"
#include "kernels.h"

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

struct F32Gemm {
  const void *A, *B, *bias, *R;
  void* C;
  int M, N, K;
  int64_t lda, ldb, ldc;
  int tiles_m, tiles_n;
  bool in_shares;            // the order of the sums (share_order)
  // what the epilogues and the norm in front take (fp32 tensors, rows of whole 16-byte pieces)
  const float* Z;            // the stored input of the activation whose derivative is applied
  float* C2;                 // the activation, or the gradient behind the derivative
  float* sums;               // column sums of C2 over 8 rows each, [M / 8 rounded up][N]
  int f;                     // SwiGLU: width of the gate half
  const float *gamma, *beta; // A is the normalised input: U = norm(A) is formed here
  float *U, *stats;
  float eps;
};

// EPI: what follows the product.  F32_GELU: C2 = gelu(C).  F32_SWIGLU: C is [gate | up], C2 = silu(gate) * up; a tile holds 16 columns of either
// half.  F32_DGELU / F32_DSWIGLU: the product is the gradient of the activation; it is not stored, C2 is the gradient in front.
enum { F32_PLAIN, F32_GELU, F32_SWIGLU, F32_DGELU, F32_DSWIGLU };
// widest row that the norm in front of a product keeps in LDS (32 rows)
constexpr int kF32NormMax = 256;
constexpr int kF32NormPitch = kF32NormMax + 4;

// four consecutive elements as fp32; elements from `n` on are zero
template <typename T, bool VEC>
__device__ __forceinline__ f32x4 load4(const T* p, int n) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if constexpr (VEC) {
    if (n > 0) {
      typedef T vec __attribute__((ext_vector_type(4)));
      const vec x = *reinterpret_cast<const vec*>(p);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = (float)x[i];
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) if (i < n) v[i] = to_f32(p[i]);
  }
  return v;
}

// One operand tile of BT rows x KS k-values: global -> registers -> LDS.
//   K contiguous: LDS [row][k], pitch KS + 4; a fragment is one 16-byte read.
//   K strided:    LDS [k][row], pitch BT + 4; a fragment is four 4-byte reads (16 lanes side by
//                 side, the four lane groups 4 * (BT + 4) floats apart: all 64 banks once).
template <typename T, int BT, int KS, bool KC, bool VEC>
struct F32Tile {
  static constexpr int NCH = BT * KS / 1024;                       // 4-element chunks per thread
  static constexpr int PITCH = (KC ? KS : BT) + 4;
  static constexpr int FLOATS = (KC ? BT : KS) * PITCH;
  f32x4 reg[NCH];
  // half > 0: the tile's upper 16 columns lie that far behind column x0, the lower 16 at x0 (K strided)
  __device__ __forceinline__ void request(const T* base, int64_t ld, int x0, int X, int k0, int K, int half = 0) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int q = threadIdx.x + 256 * i;
      if constexpr (KC) {
        const int r = x0 + q / (KS / 4), k = k0 + q % (KS / 4) * 4;
        reg[i] = load4<T, VEC>(base + (int64_t)r * ld + k, r < X ? K - k : 0);
      } else {
        const int k = k0 + q / (BT / 4), c = q % (BT / 4) * 4, x = half ? x0 + c % 16 : x0 + c;
        reg[i] = load4<T, VEC>(base + (int64_t)k * ld + x + (half && c >= 16 ? half : 0), k < K ? (half ? half : X) - x : 0);
      }
    }
  }
  __device__ __forceinline__ void put(float* lds) const {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int q = threadIdx.x + 256 * i;
      constexpr int W = (KC ? KS : BT) / 4;
      *reinterpret_cast<f32x4*>(lds + q / W * PITCH + q % W * 4) = reg[i];
    }
  }
  // k-values 16*ks + 4*g .. +3 of row x
  __device__ static __forceinline__ f32x4 frag(const float* lds, int x, int ks, int g) {
    if constexpr (KC) return *reinterpret_cast<const f32x4*>(lds + x * PITCH + 16 * ks + 4 * g);
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = lds[(16 * ks + 4 * g + e) * PITCH + x];
    return v;
  }
};

// y = norm(x) of the tile's 32 rows into `panel` (zeros behind the row's end); the workgroup of the first tile column stores it too.
// Eight lanes a row; mean first, then the squares around it, as in the norm's own kernel.
template <int NORM>
__device__ __forceinline__ void f32_norm_panel(const F32Gemm& p, int m0, bool first, float* panel) {
  constexpr int NV = kF32NormMax / 32;
  const int r = threadIdx.x >> 3, l = threadIdx.x & 7, row = m0 + r, h = p.K;
  const float* x = (const float*)p.A + (int64_t)row * p.lda;
  f32x4 v[NV], gm[NV], bt[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = (l + 8 * i) * 4;
    v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    gm[i] = v[i]; bt[i] = v[i];
    if (c < h) {
      if (row < p.M) v[i] = *reinterpret_cast<const f32x4*>(x + c);
      gm[i] = *reinterpret_cast<const f32x4*>(p.gamma + c);
      if (NORM == MOSAIC_LAYERNORM) bt[i] = *reinterpret_cast<const f32x4*>(p.beta + c);
    }
  }
  auto row_sum = [](float s) { s += __shfl_xor(s, 1, 64); s += __shfl_xor(s, 2, 64); return s + __shfl_xor(s, 4, 64); };
  const float inv_h = 1.0f / (float)h;
  float s = 0.f, mean = 0.f;
  if constexpr (NORM == MOSAIC_LAYERNORM) {
#pragma unroll
    for (int i = 0; i < NV; ++i) s += (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]);
    mean = row_sum(s) * inv_h;
    s = 0.f;
  }
#pragma unroll
  for (int i = 0; i < NV; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) { const float d = v[i][e] - mean; if ((l + 8 * i) * 4 < h) s += d * d; }
  const float rstd = 1.0f / sqrtf(row_sum(s) * inv_h + p.eps);
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = (l + 8 * i) * 4;
    f32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = c < h ? (v[i][e] - mean) * rstd * gm[i][e] + bt[i][e] : 0.f;      // mean * rstd may overflow
    *reinterpret_cast<f32x4*>(panel + r * kF32NormPitch + c) = o;
    if (first && row < p.M && c < h) *reinterpret_cast<f32x4*>(p.U + (int64_t)row * h + c) = o;
  }
  if (first && row < p.M && l == 0) { p.stats[2 * row] = mean; p.stats[2 * row + 1] = rstd; }
}

// What follows a product of fp32 tensors, for columns c .. c+3 of a row.  up: (SwiGLU) they belong to the up half, whose lanes hand them to
// the gate half's through `mail`; every lane of the workgroup comes here.  Lane (lr, g) of a wave: row lr of a block of 16 rows that starts
// at a multiple of 16, columns 4g .. 4g+3 of a block of 16.
template <int EPI>
__device__ __forceinline__ void f32_epilogue(const F32Gemm& p, f32x4 v, int row, int c, bool up, float* mail) {
  constexpr bool GU = EPI == F32_SWIGLU;
  const int width = GU ? p.f : p.N, col = up ? p.f + c : c;
  const bool in = row < p.M && c < width;
  f32x4 a2 = {0.f, 0.f, 0.f, 0.f};
  auto at = [&](const void* t, int64_t ld, int cc) { return reinterpret_cast<f32x4*>(const_cast<float*>((const float*)t) + (int64_t)row * ld + cc); };
  if constexpr (EPI == F32_PLAIN) {
    if (!in) return;
    if (p.bias) v += *reinterpret_cast<const f32x4*>((const float*)p.bias + c);
    if (p.R) v += *at(p.R, p.ldc, c);
    *at(p.C, p.ldc, c) = v;
  }
  if constexpr (EPI == F32_GELU || GU) {
    if (in && p.bias) v += *reinterpret_cast<const f32x4*>((const float*)p.bias + col);
    if (in) *at(p.C, p.ldc, col) = v;
  }
  if constexpr (EPI == F32_GELU) {
#pragma unroll
    for (int e = 0; e < 4; ++e) a2[e] = gelu_f(v[e]);
    if (in) *at(p.C2, p.N, c) = a2;
  }
  if constexpr (GU) {
    if (up) *reinterpret_cast<f32x4*>(mail) = v;
    __syncthreads();
    if (!up) {
      const f32x4 u = *reinterpret_cast<const f32x4*>(mail);
#pragma unroll
      for (int e = 0; e < 4; ++e) a2[e] = swiglu_f(v[e], u[e]);
      if (in) *at(p.C2, p.f, c) = a2;
    }
    __syncthreads();
  }
  if constexpr (EPI == F32_DGELU) {
    if (in) {
      const f32x4 z = *at(p.Z, p.N, c);
#pragma unroll
      for (int e = 0; e < 4; ++e) a2[e] = v[e] * gelu_grad_f(z[e]);
      *at(p.C2, p.N, c) = a2;
    }
    if (p.sums) {                                      // of what is stored, eight rows in ascending order: the partitions of launch_colsum
      const int first = threadIdx.x & 56;              // the lane of these columns in the first of the eight rows
      f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] += __shfl(a2[e], first + r, 64);
      if (in && (row & 7) == 0) *reinterpret_cast<f32x4*>(p.sums + (int64_t)(row >> 3) * p.N + c) = sum;
    }
  }
  if constexpr (EPI == F32_DSWIGLU) {
    if (!in) return;
    const f32x4 z = *at(p.Z, 2 * p.N, c), u = *at(p.Z, 2 * p.N, p.N + c);
    f32x4 du;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float dg, dp;
      swiglu_grad_f(z[e], u[e], v[e], &dg, &dp);
      a2[e] = dg; du[e] = dp;
    }
    *at(p.C2, 2 * p.N, c) = a2;
    *at(p.C2, 2 * p.N, p.N + c) = du;
  }
}

// k-values of a wave's share of a contraction (gemm_f32_share_tile): whole K-tiles of 64
constexpr int kShares = 8;
__device__ __host__ __forceinline__ int share_length(int K) { return (K + 64 * kShares - 1) / (64 * kShares) * 64; }

template <typename T, int BT, int KS, bool A_KC, bool B_KC, bool VEC, bool SHARES, int EPI = F32_PLAIN, int NORM = 0>
__device__ __forceinline__ void gemm_f32_tile(const F32Gemm& p, int tile, float* lds) {
  static_assert((EPI == F32_PLAIN && !SHARES) || BT == 32, "shares and the other epilogues exist for 32 x 32 tiles");
  constexpr bool GU = EPI == F32_SWIGLU;
  constexpr int TW = BT / 32;                                      // 16-wide blocks per wave and direction
  typedef F32Tile<T, BT, KS, A_KC, VEC> TA;
  typedef F32Tile<T, BT, KS, B_KC, VEC> TB;
  constexpr int AFLOATS = NORM ? 0 : TA::FLOATS, STAGE = AFLOATS + TB::FLOATS;
  float* const panel = lds + 2 * STAGE;  // NORM: the rows of A, normalised
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lr = lane & 15, g = lane >> 4;
  const int wm = (wave >> 1) * (BT / 2), wn = (wave & 1) * (BT / 2);
  const T *A = (const T*)p.A, *B = (const T*)p.B;
  const int tn = tile / p.tiles_m, tm = tile - tn * p.tiles_m;
  const int m0 = tm * BT, n0 = tn * (GU ? 16 : BT);
  TA ta; TB tb;
  // SHARES: the sum of gemm_f32_share_tile, a share of the contraction at a time
  const int share = p.in_shares ? share_length(p.K) : 0;
  f32x4 acc[TW][TW], sum = {-0.f, -0.f, -0.f, -0.f};        // -0 + x is x for every x
#pragma unroll
  for (int i = 0; i < TW; ++i)
#pragma unroll
    for (int j = 0; j < TW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  if constexpr (!NORM) ta.request(A, p.lda, m0, p.M, 0, p.K);
  tb.request(B, p.ldb, n0, p.N, 0, p.K, GU ? p.f : 0);
  if constexpr (NORM != 0) f32_norm_panel<NORM>(p, m0, tn == 0, panel);
  int st = 0, k0 = 0;
  // A share's K-tiles in a loop of their own, and the reads from LDS dealt out by hand: with a share's sum taken inside the loop the compiler kept
  // one pair of registers for B's fragments and waited for LDS eight times a K-tile.  Forward, us: 32 x 3072 x 768 on 32 CUs 34.9 -> 29.8 (29.8
  // without shares, 32.4 by the loop alone), 64 x 768 x 768 on 64 10.5 -> 9.5 (9.2), 512 x 512 x 512, not in shares, 7.7 -> 7.0; input gradient
  // 1024 x 1024 x 1024 27.0 -> 24.9.  All fragments before the first instruction: 32 x 3072 x 768 31.3, but 1024 x 1024 x 1024 29.1.
  do {
    const int k_end = SHARES && share ? min(p.K, k0 + share) : p.K;
    for (; k0 < k_end; k0 += KS, st ^= 1) {
      float* a = lds + st * STAGE;
      float* b = a + AFLOATS;
      if constexpr (!NORM) ta.put(a);
      tb.put(b);
      __syncthreads();                     // the other stage was read before this barrier, and is written after the next
      if (k0 + KS < p.K) {
        if constexpr (!NORM) ta.request(A, p.lda, m0, p.M, k0 + KS, p.K);
        tb.request(B, p.ldb, n0, p.N, k0 + KS, p.K, GU ? p.f : 0);
      }
#pragma unroll
      for (int ks = 0; ks < KS / 16; ++ks) {
        f32x4 fa[TW], fb[TW];
#pragma unroll
        for (int i = 0; i < TW; ++i) {
          if constexpr (NORM != 0) fa[i] = *reinterpret_cast<const f32x4*>(panel + (wm + 16 * i + lr) * kF32NormPitch + k0 + 16 * ks + 4 * g);
          else fa[i] = TA::frag(a, wm + 16 * i + lr, ks, g);
          fb[i] = TB::frag(b, wn + 16 * i + lr, ks, g);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < TW; ++i)
#pragma unroll
            for (int j = 0; j < TW; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[j][e], fa[i][e], acc[i][j], 0, 0, 0);
      }
      if constexpr (TW == 1) {
        // a step's fragments are read from LDS two steps before they are multiplied
        constexpr int READS = (NORM || A_KC ? 1 : 2) + (B_KC ? 1 : 2);
        __builtin_amdgcn_sched_group_barrier(0x100, 2 * READS, 0);
#pragma unroll
        for (int ks = 0; ks < KS / 16; ++ks) {
          __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
          if (ks + 2 < KS / 16) __builtin_amdgcn_sched_group_barrier(0x100, READS, 0);
        }
      }
    }
    if constexpr (SHARES) { sum += acc[0][0]; acc[0][0] = f32x4{0.f, 0.f, 0.f, 0.f}; }
  } while (SHARES && k0 < p.K);
  if constexpr (SHARES) acc[0][0] = sum;
  __syncthreads();                       // the next tile writes stage 0
  // acc[i][j][e] is output (row m0+wm+16i+lr, column n0+wn+16j+4g+e)
  if constexpr (EPI != F32_PLAIN) {
    f32_epilogue<EPI>(p, acc[0][0], m0 + wm + lr, n0 + (GU ? 0 : wn) + 4 * g, GU && wn, lds + (wm + lr) * 20 + 4 * g);
    return;
  }
  const T *bias = (const T*)p.bias, *R = (const T*)p.R;
  T* C = (T*)p.C;
#pragma unroll
  for (int i = 0; i < TW; ++i) {
    const int row = m0 + wm + 16 * i + lr;
    if (row >= p.M) continue;
#pragma unroll
    for (int j = 0; j < TW; ++j) {
      const int col = n0 + wn + 16 * j + 4 * g;
      const int n = p.N - col;
      if (n <= 0) continue;
      f32x4 v = acc[i][j];
      if (bias) v += load4<T, VEC>(bias + col, n);
      if (R) v += load4<T, VEC>(R + (int64_t)row * p.ldc + col, n);
      T* dst = C + (int64_t)row * p.ldc + col;
      if constexpr (VEC) {
        typedef T vec __attribute__((ext_vector_type(4)));
        vec o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (T)v[e];
        *reinterpret_cast<vec*>(dst) = o;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) if (e < n) dst[e] = from_f32<T>(v[e]);
      }
    }
  }
}

template <typename T, int BT, int KS, bool A_KC, bool B_KC, bool VEC, bool SHARES>
__global__ __launch_bounds__(256) void gemm_f32_kernel(F32Gemm p) {
  constexpr int STAGE = F32Tile<T, BT, KS, A_KC, VEC>::FLOATS + F32Tile<T, BT, KS, B_KC, VEC>::FLOATS;
  __shared__ __align__(16) float lds[2 * STAGE];
  for (int tile = blockIdx.x; tile < p.tiles_m * p.tiles_n; tile += gridDim.x) gemm_f32_tile<T, BT, KS, A_KC, B_KC, VEC, SHARES>(p, tile, lds);
}

// ------------------------------------------------- 16 x 16 tiles of fp32 tensors, a share of the contraction per wave
constexpr int kSharePitch = 20;
constexpr int kShareFloats = kShares * 16 * kSharePitch;
constexpr int kOutside = (int)0xFFFFFFF0u;     // a byte offset beyond every descriptor's range: reads zero

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

// Fragments of 16 rows of an operand, 16 k-values per step: lane (lr, g) holds k = 4g .. 4g+3 of row lr.  Requests are
// unconditional, so that the compiler counts them and waits for each only where it is used; what lies outside reads zero.
template <bool KC>
struct ShareOperand {
  __amdgpu_buffer_rsrc_t rsrc;
  int off[KC ? 1 : 4];           // byte offset of this lane's accesses at k = 0
  int step;                      // bytes per k-value
  int k4;
  __device__ __forceinline__ void init(const float* base, int64_t ld, int x0, int X, int K, int lr, int g) {
    const int64_t skip = KC ? (int64_t)x0 * ld : x0, all = KC ? (int64_t)(X - 1) * ld + K : (int64_t)(K - 1) * ld + X;
    rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base) + skip, 0, (int)(uint32_t)((all - skip) * 4), 0x00020000);
    step = KC ? 4 : (int)(ld * 4);
    k4 = 4 * g;
#pragma unroll
    for (int e = 0; e < (KC ? 1 : 4); ++e) off[e] = (int)(uint32_t)((KC ? (int64_t)lr * ld + 4 * g : (int64_t)(4 * g + e) * ld + lr) * 4);
  }
  __device__ __forceinline__ f32x4 request(int k, int ke) const {
    if constexpr (KC) return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, k + k4 < ke ? off[0] + k * 4 : kOutside, 0, 0));
    f32x4 f;
#pragma unroll
    for (int e = 0; e < (KC ? 1 : 4); ++e) f[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, k + k4 + e < ke ? off[e] + k * step : kOutside, 0, 0));
    return f;
  }
};

// A tile is one block of 16 x 16 outputs; each of eight waves takes an eighth of the contraction (share_length), its fragments straight from
// memory, and the eight sums meet in LDS, added in wave order.  For long contractions over few tiles, which are one chain of
// latencies: 128 x 256 outputs, K 768 (384): tiles of 32 x 32 8.8 us (5.6), this 5.3 (4.1); 100 x 64, K 1500 16.3 -> 5.7.
template <bool A_KC, bool B_KC, int EPI>
__device__ __forceinline__ void gemm_f32_share_tile(const F32Gemm& p, int tile, float* lds) {
  constexpr int STEPS = 2;                     // k-steps of 16 requested together
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, g = lane >> 4;
  const int tn = tile / p.tiles_m, tm = tile - tn * p.tiles_m;
  const int m0 = tm * 16, n0 = tn * 16;
  const int per = share_length(p.K), kb = wave * per, ke = min(p.K, kb + per);
  ShareOperand<A_KC> A;
  ShareOperand<B_KC> B;
  A.init((const float*)p.A, p.lda, m0, p.M, p.K, lr, g);
  B.init((const float*)p.B, p.ldb, n0, p.N, p.K, lr, g);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  f32x4 fa[2][STEPS], fb[2][STEPS];            // [buffer][step]
  auto request = [&](auto buf_, int k0) {
    constexpr int buf = decltype(buf_)::value;
#pragma unroll
    for (int t = 0; t < STEPS; ++t) { fa[buf][t] = A.request(k0 + 16 * t, ke); fb[buf][t] = B.request(k0 + 16 * t, ke); }
  };
  auto multiply = [&](auto buf_, int k0) {
    constexpr int buf = decltype(buf_)::value;
#pragma unroll
    for (int t = 0; t < STEPS; ++t) {
      if (k0 + 16 * t >= ke) break;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[buf][t][e], fa[buf][t][e], acc, 0, 0, 0);
    }
  };
  typedef std::integral_constant<int, 0> B0;
  typedef std::integral_constant<int, 1> B1;
  request(B0{}, kb);
  for (int k0 = kb; k0 < ke; k0 += 32 * STEPS) {
    request(B1{}, k0 + 16 * STEPS);
    multiply(B0{}, k0);
    request(B0{}, k0 + 32 * STEPS);
    multiply(B1{}, k0 + 16 * STEPS);
  }
  // acc[e] is output (row lr, column 4g + e)
  *reinterpret_cast<f32x4*>(lds + (wave * 16 + lr) * kSharePitch + 4 * g) = acc;
  __syncthreads();
  if (wave == 0) {
    f32x4 v = acc;
#pragma unroll
    for (int w = 1; w < kShares; ++w) v += *reinterpret_cast<const f32x4*>(lds + (w * 16 + lr) * kSharePitch + 4 * g);
    f32_epilogue<EPI>(p, v, m0 + lr, n0 + 4 * g, false, nullptr);
  }
  __syncthreads();                             // the next tile's sums take the same place
}

template <bool A_KC, bool B_KC, int EPI>
__global__ __launch_bounds__(64 * kShares) void gemm_f32_share_kernel(F32Gemm p) {
  static_assert(EPI != F32_SWIGLU, "a tile of 16 columns holds one half");
  __shared__ __align__(16) float lds[kShareFloats];
  for (int tile = blockIdx.x; tile < p.tiles_m * p.tiles_n; tile += gridDim.x) gemm_f32_share_tile<A_KC, B_KC, EPI>(p, tile, lds);
}

template <int EPI>
__global__ __launch_bounds__(64 * kShares) void gemm_f32_share_pair_kernel(F32Gemm d, F32Gemm w, int w_first) {
  __shared__ __align__(16) float lds[kShareFloats];
  const int nd = d.tiles_m * d.tiles_n, nw = w.tiles_m * w.tiles_n;
  for (int u = blockIdx.x; u < nd + nw; u += gridDim.x) {
    const int td = w_first ? u - nw : u, tw = w_first ? u : u - nd;
    if (td >= 0 && td < nd) gemm_f32_share_tile<true, true, EPI>(d, td, lds);
    else gemm_f32_share_tile<false, false, F32_PLAIN>(w, tw, lds);
  }
}

// Which products are summed in shares, by whatever kernel: a function of the shape (512: two workgroups to a CU of the whole device; operands
// that 32-bit offsets reach).  They are computed in 16 x 16 tiles where two workgroups to a CU take all of them and a wave
// has work for its latency; below 128 k-values 32 x 32 tiles are as fast.
int64_t share_tiles(const F32Gemm& p) { return ceil_div(p.M, 16) * ceil_div(p.N, 16); }
bool share_order(const F32Gemm& p) {
  const int64_t rows_a = (int64_t)std::max(p.M, p.K) + 32, rows_b = (int64_t)std::max(p.N, p.K) + 32, lim = (int64_t)1 << 29;
  return share_tiles(p) <= 512 && rows_a * p.lda + p.K < lim && rows_b * p.ldb + p.K < lim;
}
void share_layout(F32Gemm* p) { p->tiles_m = (int)ceil_div(p->M, 16); p->tiles_n = (int)ceil_div(p->N, 16); }

// The input gradient (both operands K-contiguous) and the weight gradient (both K-strided) of a linear layer in one
// launch of 32 x 32 tiles, those with the longer contraction first: each is a chain of a few tiles' latency that leaves
// most CUs idle.  Products of a decoder layer of 256 rows, width 128: 6.1 + 5.6 us in two launches, 7.0 in one (a launch less
// to wait for besides: with the attention's, the layer's step 120 -> 92 us; with the norms', the activations' and the shares 62).
template <int EPI, bool SHARES>
__global__ __launch_bounds__(256) void gemm_f32_pair_kernel(F32Gemm d, F32Gemm w, int w_first) {
  typedef F32Tile<float, 32, 64, true, true> Contiguous;
  typedef F32Tile<float, 32, 64, false, true> Strided;
  constexpr int STAGE = 2 * (Contiguous::FLOATS > Strided::FLOATS ? Contiguous::FLOATS : Strided::FLOATS);
  __shared__ __align__(16) float lds[2 * STAGE];
  const int nd = d.tiles_m * d.tiles_n, nw = w.tiles_m * w.tiles_n;
  for (int u = blockIdx.x; u < nd + nw; u += gridDim.x) {
    const int td = w_first ? u - nw : u, tw = w_first ? u : u - nd;
    if (td >= 0 && td < nd) gemm_f32_tile<float, 32, 64, true, true, true, SHARES, EPI>(d, td, lds);
    else gemm_f32_tile<float, 32, 64, false, false, true, SHARES>(w, tw, lds);
  }
}

// The forward product with what stands before and behind it in a layer of the fp32 path: a launch costs 4 us or more however little
// it does.  The norm is formed again by every tile column (rows of at most kF32NormMax values, read once more from the caches).
template <int EPI, int NORM, bool SHARES>
__global__ __launch_bounds__(256) void gemm_f32_layer_kernel(F32Gemm p) {
  constexpr int STAGE = (NORM ? 0 : F32Tile<float, 32, 64, true, true>::FLOATS) + F32Tile<float, 32, 64, false, true>::FLOATS;
  __shared__ __align__(16) float lds[2 * STAGE + (NORM ? 32 * kF32NormPitch : 0)];
  for (int tile = blockIdx.x; tile < p.tiles_m * p.tiles_n; tile += gridDim.x) gemm_f32_tile<float, 32, 64, true, false, true, SHARES, EPI, NORM>(p, tile, lds);
}

// a function of the shape alone; the order of every sum is the same in both.  Figures in launch_t.
bool large_tiles(int64_t M, int64_t N) { return ceil_div(M, 64) * ceil_div(N, 64) >= 512; }

template <typename T, bool A_KC, bool B_KC, bool VEC>
mosaic_status launch_t(hipStream_t s, int quota, F32Gemm p) {
  // A function of the shape alone; the order of every sum is the same in both.  Measured, forward, tiles of 32 / of 64
  // on 256 CUs (on 64): 256 tiles of 64 (1024 x 512 x 1024) 15.7 / 16.8 us (22.6 / 16.6), 512 (1024 x 512 x 2048)
  // 28.7 / 26.0 (43.9 / 31.1), 576 31.1 / 34.1 (48.9 / 45.2), 1024 53.1 / 44.3 (84.9 / 59.7), 4096 386 / 312; input gradient,
  // 192 tiles 31.0 / 41.8.  bf16 tensors, 256 tiles 33.0 / 39.3, 576 76.5 / 66.0, 1024 122.6 / 82.2.
  const bool large = large_tiles(p.M, p.N);
  p.in_shares = std::is_same<T, float>::value && !large && share_order(p);
  // (an output on an operand stays with the larger tiles, of which there may be only one: it then reads everything before it stores)
  const int64_t ab = (A_KC ? (int64_t)(p.M - 1) * p.lda + p.K : (int64_t)(p.K - 1) * p.lda + p.M) * 4;
  const int64_t bb = (B_KC ? (int64_t)(p.N - 1) * p.ldb + p.K : (int64_t)(p.K - 1) * p.ldb + p.N) * 4, cb = ((int64_t)(p.M - 1) * p.ldc + p.N) * 4;
  if constexpr (std::is_same<T, float>::value && VEC) {
    if (p.in_shares && p.K >= 128 && share_tiles(p) <= 2 * (int64_t)quota && !overlap(p.C, cb, p.A, ab) && !overlap(p.C, cb, p.B, bb)) {
      share_layout(&p);
      gemm_f32_share_kernel<A_KC, B_KC, F32_PLAIN><<<p.tiles_m * p.tiles_n, 64 * kShares, 0, s>>>(p);
      MOSAIC_LAUNCH_CHECK();
      return MOSAIC_OK;
    }
  }
  const int bt = large ? 64 : 32;
  const int64_t tm = ceil_div(p.M, bt), tn = ceil_div(p.N, bt);
  if (tm * tn > INT32_MAX / 2) MOSAIC_FAIL(MOSAIC_EUNSUPPORTED, "too many output tiles");
  p.tiles_m = (int)tm; p.tiles_n = (int)tn;
  const int grid = grid_for(quota, 4, tm * tn);
  if (large) {
    gemm_f32_kernel<T, 64, 32, A_KC, B_KC, VEC, false><<<grid, 256, 0, s>>>(p);
  } else {
    if constexpr (std::is_same<T, float>::value)
      if (p.in_shares) gemm_f32_kernel<T, 32, 64, A_KC, B_KC, VEC, true><<<grid, 256, 0, s>>>(p);
    if (!p.in_shares) gemm_f32_kernel<T, 32, 64, A_KC, B_KC, VEC, false><<<grid, 256, 0, s>>>(p);
  }
  MOSAIC_LAUNCH_CHECK();
  return MOSAIC_OK;
}

template <typename T>
mosaic_status launch_form(hipStream_t s, int quota, bool a_kc, bool b_kc, const F32Gemm& p) {
  const uintptr_t mask = 4 * sizeof(T) - 1;                        // four elements per access where every row allows it
  const bool vec = p.lda % 4 == 0 && p.ldb % 4 == 0 && p.ldc % 4 == 0 && p.N % 4 == 0 && (a_kc ? p.K : p.M) % 4 == 0 &&
                   (b_kc ? p.K : p.N) % 4 == 0 &&
                   (((uintptr_t)p.A | (uintptr_t)p.B | (uintptr_t)p.C | (uintptr_t)p.bias | (uintptr_t)p.R) & mask) == 0;
#define FORM(AK, BK_) (vec ? launch_t<T, AK, BK_, true>(s, quota, p) : launch_t<T, AK, BK_, false>(s, quota, p))
  if (a_kc) return b_kc ? FORM(true, true) : FORM(true, false);
  return b_kc ? FORM(false, true) : FORM(false, false);
#undef FORM
}

}  // namespace

// (norm and) product (and activation) of fp32 tensors, dense rows, no output on an input or on another; *taken: in one launch
mosaic_status launch_layer_fwd_f32(hipStream_t s, int quota, int norm, int act, int64_t T, int64_t k, int64_t n, float eps, const void* X, const void* gamma,
                                   const void* beta, void* U, float* stats, const void* W, const void* bias, void* Z, void* A, bool* taken) {
  *taken = false;
  const bool glu = act == MOSAIC_SWIGLU;
  const int64_t f = glu ? n / 2 : n;
  const uintptr_t all = (uintptr_t)X | (uintptr_t)gamma | (uintptr_t)beta | (uintptr_t)U | (uintptr_t)W | (uintptr_t)bias | (uintptr_t)Z | (uintptr_t)A;
  if (T <= 0 || k <= 0 || n <= 0 || T > INT32_MAX || k > INT32_MAX || n > INT32_MAX || k % 4 || f % 4 || all % 16 || large_tiles(T, n)) return MOSAIC_OK;
  if (act != -1 && act != MOSAIC_GELU && !glu) return MOSAIC_OK;
  if (norm && (k > kF32NormMax || (norm != MOSAIC_LAYERNORM && norm != MOSAIC_RMSNORM))) return MOSAIC_OK;
  // The norm, formed again by every tile column, shares the launch up to two tiles to a CU of the device: a function of the shape, because its bits
  // are not those of the norm's own kernel.  In the product's launch / apart, us: encoder layer of 2048 rows, width 256, 1536 tiles, 338 / 335, on 32 CUs
  // 1524 / 1482; decoder layer of 1024 rows, width 256, 768 and 1536 tiles, on 64 391 / 372; 256 rows, width 128, 96 tiles, 62 / 70.
  if (norm && ceil_div(T, 32) * (glu ? ceil_div(f, 16) : ceil_div(n, 32)) > 512) return MOSAIC_OK;
  // A tile's outputs are stored while other tiles still read the inputs: an output that lies on an input, which the order of separate
  // launches allows (the activation on X or W), keeps them, and so does an activation on Z
  struct Span { const void* p; int64_t n; };
  const Span in[] = {{X, T * k * 4}, {W, k * n * 4}, {bias, n * 4}, {gamma, k * 4}, {beta, k * 4}}, out[] = {{Z, T * n * 4}, {A, T * f * 4}, {U, T * k * 4}, {stats, T * 8}};
  for (const Span& o : out)
    for (const Span& i : in) if (overlap(o.p, o.n, i.p, i.n)) return MOSAIC_OK;
  if (overlap(Z, T * n * 4, A, T * f * 4)) return MOSAIC_OK;
  F32Gemm p = {};
  p.A = X; p.B = W; p.bias = bias; p.C = Z; p.C2 = (float*)A; p.M = (int)T; p.N = (int)n; p.K = (int)k; p.lda = k; p.ldb = n; p.ldc = n; p.f = (int)f;
  p.tiles_m = (int)ceil_div(T, 32); p.tiles_n = (int)(glu ? ceil_div(f, 16) : ceil_div(n, 32));
  p.in_shares = share_order(p);
  p.gamma = (const float*)gamma; p.beta = (const float*)beta; p.U = (float*)U; p.stats = stats; p.eps = eps;
  const int grid = grid_for(quota, 4, (int64_t)p.tiles_m * p.tiles_n);
  auto go = [&](auto epi, auto shares) {
    constexpr int EPI = decltype(epi)::value;
    constexpr bool SHARES = decltype(shares)::value;
    if (norm == MOSAIC_LAYERNORM) gemm_f32_layer_kernel<EPI, MOSAIC_LAYERNORM, SHARES><<<grid, 256, 0, s>>>(p);
    else if (norm) gemm_f32_layer_kernel<EPI, MOSAIC_RMSNORM, SHARES><<<grid, 256, 0, s>>>(p);
    else gemm_f32_layer_kernel<EPI, 0, SHARES><<<grid, 256, 0, s>>>(p);
  };
  auto launch = [&](auto epi) { if (p.in_shares) go(epi, std::true_type{}); else go(epi, std::false_type{}); };
  if (glu) launch(std::integral_constant<int, F32_SWIGLU>{});
  else if (act == MOSAIC_GELU) launch(std::integral_constant<int, F32_GELU>{});
  else launch(std::integral_constant<int, F32_PLAIN>{});
  MOSAIC_LAUNCH_CHECK();
  *taken = true;
  return MOSAIC_OK;
}

// dX[T,k] = dY W^T and dW[k,n] = X^T dY of fp32 tensors, dense rows, no output on an input; *taken: in one launch.  act >= 0: X is an
// activation, the gradient goes on to its input, dZ[T, k] (SwiGLU: [T, 2k]) = act'(Z) dX, and dX is not written; sums (may be null): column sums
// of dZ over 8 rows each.
mosaic_status launch_linear_bwd_f32(hipStream_t s, int quota, int64_t T, int64_t k, int64_t n, const void* X, const void* dY, const void* W,
                                    void* dX, void* dW, bool* taken, int act, const void* Z, void* dZ, float* sums) {
  *taken = false;
  const uintptr_t all = (uintptr_t)X | (uintptr_t)dY | (uintptr_t)W | (uintptr_t)dX | (uintptr_t)dW | (uintptr_t)Z | (uintptr_t)dZ | (uintptr_t)sums;
  if (T > INT32_MAX || k > INT32_MAX || n > INT32_MAX || k % 4 || n % 4 || all % 16 || large_tiles(T, k) || large_tiles(k, n)) return MOSAIC_OK;
  if (act != -1 && act != MOSAIC_GELU && act != MOSAIC_SWIGLU) return MOSAIC_OK;
  auto product = [](const void* A, int64_t lda, const void* B, int64_t ldb, void* C, int64_t M, int64_t N, int64_t K) {
    F32Gemm p = {};
    p.A = A; p.B = B; p.C = C; p.M = (int)M; p.N = (int)N; p.K = (int)K; p.lda = lda; p.ldb = ldb; p.ldc = N;
    p.tiles_m = (int)ceil_div(M, 32); p.tiles_n = (int)ceil_div(N, 32);
    return p;
  };
  F32Gemm d = product(dY, n, W, n, dX, T, k, n), w = product(X, k, dY, n, dW, k, n, T);
  d.Z = (const float*)Z; d.C2 = (float*)dZ; d.sums = sums;
  d.in_shares = share_order(d);
  w.in_shares = share_order(w);
  const bool share = d.in_shares && w.in_shares && std::max(T, n) >= 128 && share_tiles(d) + share_tiles(w) <= 2 * (int64_t)quota;
  auto launch = [&](auto epi) {
    constexpr int EPI = decltype(epi)::value;
    if (share) {
      share_layout(&d);
      share_layout(&w);
      gemm_f32_share_pair_kernel<EPI><<<d.tiles_m * d.tiles_n + w.tiles_m * w.tiles_n, 64 * kShares, 0, s>>>(d, w, T > n);
    } else {
      const int grid = grid_for(quota, 4, (int64_t)d.tiles_m * d.tiles_n + (int64_t)w.tiles_m * w.tiles_n);
      if (d.in_shares || w.in_shares) gemm_f32_pair_kernel<EPI, true><<<grid, 256, 0, s>>>(d, w, T > n);
      else gemm_f32_pair_kernel<EPI, false><<<grid, 256, 0, s>>>(d, w, T > n);
    }
  };
  if (act == MOSAIC_SWIGLU) launch(std::integral_constant<int, F32_DSWIGLU>{});
  else if (act == MOSAIC_GELU) launch(std::integral_constant<int, F32_DGELU>{});
  else launch(std::integral_constant<int, F32_PLAIN>{});
  MOSAIC_LAUNCH_CHECK();
  *taken = true;
  return MOSAIC_OK;
}

mosaic_status launch_gemm_f32(hipStream_t s, int quota, int dtype, bool a_kc, bool b_kc, int M, int N, int K, const void* A,
                              int64_t lda, const void* B, int64_t ldb, void* C, int64_t ldc, const void* bias, const void* R) {
  F32Gemm p = {};
  p.A = A; p.B = B; p.bias = bias; p.R = R; p.C = C; p.M = M; p.N = N; p.K = K; p.lda = lda; p.ldb = ldb; p.ldc = ldc;
  return dtype == MOSAIC_BF16 ? launch_form<bf16>(s, quota, a_kc, b_kc, p) : launch_form<float>(s, quota, a_kc, b_kc, p);
}
