// Contractions with fp32 arithmetic: the fp32 path, and the bf16 shapes that the bf16 kernels do
// not take (widths that are not a multiple of 8, unaligned tensors, extents beyond 32 bits).
//
// v_mfma_f32_16x16x4_f32: fp32 products and sums, no narrower type anywhere.  Four waves share a
// square output tile.  A lane's four consecutive k-values feed four consecutive instructions:
// instruction s of a 16-wide k-step contracts k = s, 4+s, 8+s, 12+s; both operands agree on that
// order, so each output is a fixed sum that depends on K alone.
//
// What bounds it: the fp32 workloads are a few hundred rows wide, every product is a chain of
// latencies (load, barrier, matrix instructions, store), so tiles are small enough to give most
// CUs one (32 x 32), a K-tile is 64 deep and the next one is requested before the current one
// is multiplied.  Products with at least two 64 x 64 tiles per CU take those: twice the flops per
// LDS byte (rule and figures in launch_t).  256 x 128 x 384 (M x K x N) and the like: 47 us with 64 x 64 tiles of scalar FMA, 16 deep,
// before; 4.8 to 5.9 now (launch included).
#include "kernels.h"

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

struct F32Gemm {
  const void *A, *B, *bias, *R;
  void* C;
  int M, N, K;
  int64_t lda, ldb, ldc;
  int tiles_m, tiles_n;
};

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
  __device__ __forceinline__ void request(const T* base, int64_t ld, int x0, int X, int k0, int K) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int q = threadIdx.x + 256 * i;
      if constexpr (KC) {
        const int r = x0 + q / (KS / 4), k = k0 + q % (KS / 4) * 4;
        reg[i] = load4<T, VEC>(base + (int64_t)r * ld + k, r < X ? K - k : 0);
      } else {
        const int k = k0 + q / (BT / 4), x = x0 + q % (BT / 4) * 4;
        reg[i] = load4<T, VEC>(base + (int64_t)k * ld + x, k < K ? X - x : 0);
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

template <typename T, int BT, int KS, bool A_KC, bool B_KC, bool VEC>
__device__ __forceinline__ void gemm_f32_tile(const F32Gemm& p, int tile, float* lds) {
  constexpr int TW = BT / 32;                                      // 16-wide blocks per wave and direction
  typedef F32Tile<T, BT, KS, A_KC, VEC> TA;
  typedef F32Tile<T, BT, KS, B_KC, VEC> TB;
  constexpr int STAGE = TA::FLOATS + TB::FLOATS;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lr = lane & 15, g = lane >> 4;
  const int wm = (wave >> 1) * (BT / 2), wn = (wave & 1) * (BT / 2);
  const T *A = (const T*)p.A, *B = (const T*)p.B;
  const int tn = tile / p.tiles_m, tm = tile - tn * p.tiles_m;
  const int m0 = tm * BT, n0 = tn * BT;
  TA ta; TB tb;
  f32x4 acc[TW][TW];
#pragma unroll
  for (int i = 0; i < TW; ++i)
#pragma unroll
    for (int j = 0; j < TW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  ta.request(A, p.lda, m0, p.M, 0, p.K);
  tb.request(B, p.ldb, n0, p.N, 0, p.K);
  int st = 0;
  for (int k0 = 0; k0 < p.K; k0 += KS, st ^= 1) {
    float* a = lds + st * STAGE;
    float* b = a + TA::FLOATS;
    ta.put(a);
    tb.put(b);
    __syncthreads();                     // the other stage was read before this barrier, and is written after the next
    if (k0 + KS < p.K) {
      ta.request(A, p.lda, m0, p.M, k0 + KS, p.K);
      tb.request(B, p.ldb, n0, p.N, k0 + KS, p.K);
    }
#pragma unroll
    for (int ks = 0; ks < KS / 16; ++ks) {
      f32x4 fa[TW], fb[TW];
#pragma unroll
      for (int i = 0; i < TW; ++i) { fa[i] = TA::frag(a, wm + 16 * i + lr, ks, g); fb[i] = TB::frag(b, wn + 16 * i + lr, ks, g); }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < TW; ++i)
#pragma unroll
          for (int j = 0; j < TW; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[j][e], fa[i][e], acc[i][j], 0, 0, 0);
    }
  }
  __syncthreads();                       // the next tile writes stage 0
  // acc[i][j][e] is output (row m0+wm+16i+lr, column n0+wn+16j+4g+e)
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

template <typename T, int BT, int KS, bool A_KC, bool B_KC, bool VEC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(F32Gemm p) {
  constexpr int STAGE = F32Tile<T, BT, KS, A_KC, VEC>::FLOATS + F32Tile<T, BT, KS, B_KC, VEC>::FLOATS;
  __shared__ __align__(16) float lds[2 * STAGE];
  for (int tile = blockIdx.x; tile < p.tiles_m * p.tiles_n; tile += gridDim.x) gemm_f32_tile<T, BT, KS, A_KC, B_KC, VEC>(p, tile, lds);
}

// The input gradient (both operands K-contiguous) and the weight gradient (both K-strided) of a linear layer in one
// launch of 32 x 32 tiles, those with the longer contraction first: each is a chain of a few tiles' latency that leaves
// most CUs idle.  Products of a decoder layer of 256 rows, width 128: 6.1 + 5.6 us in two launches, 7.0 in one (a launch less
// to wait for besides: with the attention's, the layer's step 120 -> 92 us).
__global__ __launch_bounds__(256) void gemm_f32_pair_kernel(F32Gemm d, F32Gemm w, int w_first) {
  typedef F32Tile<float, 32, 64, true, true> Contiguous;
  typedef F32Tile<float, 32, 64, false, true> Strided;
  constexpr int STAGE = 2 * (Contiguous::FLOATS > Strided::FLOATS ? Contiguous::FLOATS : Strided::FLOATS);
  __shared__ __align__(16) float lds[2 * STAGE];
  const int nd = d.tiles_m * d.tiles_n, nw = w.tiles_m * w.tiles_n;
  for (int u = blockIdx.x; u < nd + nw; u += gridDim.x) {
    const int td = w_first ? u - nw : u, tw = w_first ? u : u - nd;
    if (td >= 0 && td < nd) gemm_f32_tile<float, 32, 64, true, true, true>(d, td, lds);
    else gemm_f32_tile<float, 32, 64, false, false, true>(w, tw, lds);
  }
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
  const int bt = large ? 64 : 32;
  const int64_t tm = ceil_div(p.M, bt), tn = ceil_div(p.N, bt);
  if (tm * tn > INT32_MAX / 2) MOSAIC_FAIL(MOSAIC_EUNSUPPORTED, "too many output tiles");
  p.tiles_m = (int)tm; p.tiles_n = (int)tn;
  const int grid = grid_for(quota, 4, tm * tn);
  if (large) gemm_f32_kernel<T, 64, 32, A_KC, B_KC, VEC><<<grid, 256, 0, s>>>(p);
  else gemm_f32_kernel<T, 32, 64, A_KC, B_KC, VEC><<<grid, 256, 0, s>>>(p);
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

// dX[T,k] = dY W^T and dW[k,n] = X^T dY of fp32 tensors, dense rows, no output on an input; *taken: in one launch
mosaic_status launch_linear_bwd_f32(hipStream_t s, int quota, int64_t T, int64_t k, int64_t n, const void* X, const void* dY, const void* W,
                                    void* dX, void* dW, bool* taken) {
  *taken = false;
  const uintptr_t all = (uintptr_t)X | (uintptr_t)dY | (uintptr_t)W | (uintptr_t)dX | (uintptr_t)dW;
  if (T > INT32_MAX || k > INT32_MAX || n > INT32_MAX || k % 4 || n % 4 || all % 16 || large_tiles(T, k) || large_tiles(k, n)) return MOSAIC_OK;
  auto product = [](const void* A, int64_t lda, const void* B, int64_t ldb, void* C, int64_t M, int64_t N, int64_t K) {
    return F32Gemm{A, B, nullptr, nullptr, C, (int)M, (int)N, (int)K, lda, ldb, N, (int)ceil_div(M, 32), (int)ceil_div(N, 32)};
  };
  const F32Gemm d = product(dY, n, W, n, dX, T, k, n), w = product(X, k, dY, n, dW, k, n, T);
  gemm_f32_pair_kernel<<<grid_for(quota, 4, (int64_t)d.tiles_m * d.tiles_n + (int64_t)w.tiles_m * w.tiles_n), 256, 0, s>>>(d, w, T > n);
  MOSAIC_LAUNCH_CHECK();
  *taken = true;
  return MOSAIC_OK;
}

mosaic_status launch_gemm_f32(hipStream_t s, int quota, int dtype, bool a_kc, bool b_kc, int M, int N, int K, const void* A,
                              int64_t lda, const void* B, int64_t ldb, void* C, int64_t ldc, const void* bias, const void* R) {
  const F32Gemm p = {A, B, bias, R, C, M, N, K, lda, ldb, ldc, 0, 0};
  return dtype == MOSAIC_BF16 ? launch_form<bf16>(s, quota, a_kc, b_kc, p) : launch_form<float>(s, quota, a_kc, b_kc, p);
}
