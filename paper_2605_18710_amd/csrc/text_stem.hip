// Text stem: image-token rows and embedding rows assembled into sequences, and the way back.
//
// Forward and the image-token gradient are row copies (HBM-bound).  The embedding gradient
// needs, for every table row, the sum of the output gradients at the positions that hold it:
//   1. the T positions are sorted by id with a stable radix sort (8 bits a pass), so the occurrences of an id are
//      one run in ascending position: by one workgroup in its LDS while the others fill the table rows that nobody
//      used and copy the image-token gradient (up to 8192 positions), else in two launches a pass;
//   2. the sorted list is cut into segments of kSeg entries; a workgroup requests all rows of
//      its segment at once and adds them run by run, so the work is balanced however often an
//      id occurs; runs inside a segment go straight to the table, pieces of longer runs to scratch;
//   3. the pieces of a run are added by the segment it starts in.  After the sort in several launches, rows that nobody
//      used are found by bisection in the sorted list and filled with zeros beside step 2.
// Every sum has one owner and an order fixed by the ids alone: repeated ids need no atomics and
// the bits do not depend on the grid.
//
// The order: segments of 16 positions ascending, then the pieces of a run that spans segments, as
// four quarters added in turn.
//
// What bounds it: the table is written whole (V x h; 131 MB at V 32000, h 2048) and dy read once.
// At B 8, N 1024, h 2048, V 32000, bf16, 196 or fewer image tokens: sort and fill 23 us, sums 11, joins 7 (forward 12); in six
// launches of the sort, sums with the fill beside them, a join with a bisection per run and a launch for the image
// tokens the whole pass took 100 us instead of 67, forward included.
// A walk over all positions by the owner of every table row (V x T id reads) takes 2000 us there, but is one launch,
// and still what small calls take (scan_is_faster).
#include "kernels.h"
#include "sample_index.h"

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

// Token ids and image-token counts.  Without per-sample counts every sample has n_img image
// tokens and ids holds the N - n_img text ids of a sample, [B, N - n_img].  With counts
// (int32 [B], clamped to [0, n_img]) sample b takes its first counts[b] image tokens and ids
// holds one id per sequence position, [B, N], read at positions counts[b] .. N-1.
__device__ __forceinline__ int stem_n_img(const int32_t* counts, int b, int n_img) {
  if (!counts) return n_img;
  const int c = counts[b];
  return c < 0 ? 0 : (c > n_img ? n_img : c);
}
__device__ __forceinline__ int stem_id(const int32_t* ids, const int32_t* counts, int b, int t, int N, int n_img, int vocab) {
  // an id outside the table is clamped rather than followed out of bounds (forward and backward alike)
  const int id = counts ? ids[(int64_t)b * N + t] : ids[(int64_t)b * (N - n_img) + (t - n_img)];
  return id < 0 ? 0 : (id >= vocab ? vocab - 1 : id);
}

// One wave per row: one division per row, 16 bytes per lane and access.  (A kernel with one element
// per thread spent its time on three 64-bit divisions per element: 51 us at B8 N1024 h2048.)
template <typename T, int V>
__global__ __launch_bounds__(kThreads) void text_stem_fwd_kernel(const T* __restrict__ img_tok, const int32_t* __restrict__ ids,
                                                                 const int32_t* __restrict__ counts,
                                                                 const T* __restrict__ table, T* __restrict__ out,
                                                                 int B, int N, int n_img, int h, int vocab) {
  typedef typename Pack<T, V>::type vec;
  const int lane = threadIdx.x & 63;
  const int64_t rows = (int64_t)B * N;
  for (int64_t row = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6); row < rows; row += (int64_t)gridDim.x * kWaves) {
    const int b = (int)(row / N), t = (int)(row - (int64_t)b * N);
    const T* src = t < stem_n_img(counts, b, n_img) ? img_tok + ((int64_t)b * n_img + t) * h
                                                     : table + (int64_t)stem_id(ids, counts, b, t, N, n_img, vocab) * h;
    T* dst = out + row * h;
    for (int c = lane * V; c < h; c += 64 * V) *reinterpret_cast<vec*>(dst + c) = *reinterpret_cast<const vec*>(src + c);
  }
}

// gradient of the image tokens: rows the sample did not use get zero
template <typename T, int V>
__global__ __launch_bounds__(kThreads) void split_img_kernel(const T* __restrict__ dy, const int32_t* __restrict__ counts,
                                                             T* __restrict__ d_img, int B, int N, int n_img, int h) {
  typedef typename Pack<T, V>::type vec;
  const int lane = threadIdx.x & 63;
  const int64_t rows = (int64_t)B * n_img;
  for (int64_t row = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6); row < rows; row += (int64_t)gridDim.x * kWaves) {
    const int b = (int)(row / n_img), t = (int)(row - (int64_t)b * n_img);
    const bool used = t < stem_n_img(counts, b, n_img);
    const T* src = dy + ((int64_t)b * N + t) * h;
    T* dst = d_img + row * h;
    for (int c = lane * V; c < h; c += 64 * V) *reinterpret_cast<vec*>(dst + c) = used ? *reinterpret_cast<const vec*>(src + c) : vec{};
  }
}

// --------------------------------------------------------------------- sort by id
constexpr int kDigit = 8, kBins = 1 << kDigit;       // a thread per bin
constexpr int kRounds = 8;                            // keys per thread
constexpr int kChunk = kThreads * kRounds;            // keys per workgroup
static_assert(kBins == kThreads, "the scatter kernel gives every bin a thread");

// where a sort pass takes its keys from: the token ids (first pass; positions that hold an
// image token get the key `vocab`, beyond every id), or the pass before
struct SortInput {
  const int32_t *key, *pos;                           // null key: the token ids
  const int32_t *ids, *counts;
  int N, n_img, vocab;
  __device__ __forceinline__ int key_of(int e) const {
    if (key) return key[e];
    const int b = e / N, t = e - b * N;
    return t >= stem_n_img(counts, b, n_img) ? stem_id(ids, counts, b, t, N, n_img, vocab) : vocab;
  }
  __device__ __forceinline__ int pos_of(int e) const { return key ? pos[e] : e; }
};

// digit counts of every chunk: hist[chunk][bin]
__global__ __launch_bounds__(kThreads) void sort_hist_kernel(SortInput in, int shift, int total, int chunks, int* __restrict__ hist) {
  __shared__ int cnt[kBins];
  for (int c = blockIdx.x; c < chunks; c += gridDim.x) {
    cnt[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      const int e = c * kChunk + r * kThreads + threadIdx.x;
      if (e < total) atomicAdd(&cnt[(in.key_of(e) >> shift) & (kBins - 1)], 1);
    }
    __syncthreads();
    hist[c * kBins + threadIdx.x] = cnt[threadIdx.x];
    __syncthreads();
  }
}

// A chunk's keys go to their places: entries with a smaller digit, the same digit in earlier
// chunks, in earlier waves of the chunk (a wave owns 512 consecutive entries), in earlier rounds
// of the wave, in earlier lanes of the round.
__global__ __launch_bounds__(kThreads) void sort_scatter_kernel(SortInput in, int shift, int total, int chunks,
                                                                const int* __restrict__ hist, int32_t* __restrict__ key_out,
                                                                int32_t* __restrict__ pos_out) {
  __shared__ int place[kWaves][kBins];
  __shared__ int wave_total[kWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int c = blockIdx.x; c < chunks; c += gridDim.x) {
    int key[kRounds];
    const int first = c * kChunk + wave * (64 * kRounds) + lane;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) place[w][threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      const int e = first + 64 * r;
      key[r] = e < total ? in.key_of(e) : -1;
      if (e < total) atomicAdd(&place[wave][(key[r] >> shift) & (kBins - 1)], 1);
    }
    // this thread's bin: entries in all chunks, and in the chunks before this one
    int all = 0, before = 0;
    for (int k = 0; k < chunks; ++k) {
      const int v = hist[k * kBins + threadIdx.x];
      if (k < c) before += v;
      all += v;
    }
    int scan = all;                                   // inclusive over the bins
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(scan, o, 64);
      if (lane >= o) scan += v;
    }
    if (lane == 63) wave_total[wave] = scan;
    __syncthreads();
    int at = scan - all + before;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) if (w < wave) at += wave_total[w];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) { const int v = place[w][threadIdx.x]; place[w][threadIdx.x] = at; at += v; }
    __syncthreads();
    volatile int* mine = place[wave];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      const int e = first + 64 * r;
      const bool live = e < total;
      const int dgt = (key[r] >> shift) & (kBins - 1);
      unsigned long long same = __ballot(live);       // lanes of this round with the same digit
#pragma unroll
      for (int b = 0; b < kDigit; ++b) {
        const unsigned long long m = __ballot((dgt >> b) & 1);
        same &= ((dgt >> b) & 1) ? m : ~m;
      }
      const int rank = __popcll(same & ((1ull << lane) - 1ull));
      const int base = live ? mine[dgt] : 0;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();                // every lane has read its base before a leader moves it
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if (live) {
        if (rank == 0) mine[dgt] = base + __popcll(same);
        key_out[base + rank] = key[r];
        pos_out[base + rank] = in.pos_of(e);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    __syncthreads();
  }
}

// Keys of the positions first + r * step, r < rounds, all of them requested together (conditional loads would wait for each
// other); -1 past the end.  Positions without an id to read are requested outside the buffer, which reads nothing.  An integer division a
// key would cost more than the loads (sample_of).
template <int R, int N>
__device__ __forceinline__ void keys_at(const SortInput& in, int first, int step, int rounds, int total, int (&key)[N]) {
  if constexpr (R > 1) {
    if (rounds <= R / 2) return keys_at<R / 2>(in, first, step, rounds, total, key);        // alike for all threads
  }
  constexpr int kOutside = INT32_MIN;
  const __amdgpu_buffer_rsrc_t ids = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(in.ids), 0, in.ids ? total * 4 : 0, 0x00020000);
  const __amdgpu_buffer_rsrc_t counts = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(in.counts), 0, in.counts ? total * 4 : 0, 0x00020000);
  const float inv = 1.f / (float)in.N;
  int t[R], img[R], id[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int e = first + r * step, b = sample_of(e, inv);
    const bool live = r < rounds && e < total;
    t[r] = live ? e - b * in.N : -1;
    img[r] = in.counts ? (int)__builtin_amdgcn_raw_buffer_load_b32(counts, live ? b * 4 : kOutside, 0, 0) : in.n_img;
    const bool read = in.counts ? live : t[r] >= in.n_img && live;
    id[r] = (int)__builtin_amdgcn_raw_buffer_load_b32(ids, read ? (in.counts ? e : b * (in.N - in.n_img) + t[r] - in.n_img) * 4 : kOutside, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < N; ++r) {
    key[r] = -1;
    if (r < R && t[r % R] >= 0) key[r] = t[r % R] >= min(max(img[r % R], 0), in.n_img) ? min(max(id[r % R], 0), in.vocab - 1) : in.vocab;
  }
}

// Sort, fill and image-token gradient in one launch.  Workgroup 0 sorts: a key and its position share 32 bits, a thread
// holds up to 8 of them, and a pass scatters them through LDS in the order of sort_scatter_kernel, so the lists are the
// same.  The others (all, if there is one) take table rows and image-token rows; which table rows are used they find
// out by a walk over the ids, 2048 rows at a time.  What bounds it is the fill of what nobody used (106 of 131 MB), which covers
// the sort's 10 to 20 us of short dependent steps, and the ids before it: eight conditional reads a thread, one after the other,
// took 5 us of which keys_at leaves half (the whole pass with buffers in cache 54.7 -> 52.3 us; 1400 positions, 1000 x 512, 18.7 -> 18.5).
constexpr int kOneThreads = 1024, kOneWaves = kOneThreads / 64, kFlagRows = 2048;
constexpr int kOneMax = 8 * kOneThreads;              // positions that one workgroup sorts
static_assert(kFlagRows <= kOneWaves * kBins + kOneMax, "flags");
static_assert(2 * kOneMax <= kSampleMax, "sample_of, positions past the end (fewer than as many again) included");
template <typename T, int V>
__global__ __launch_bounds__(kOneThreads) void embed_prepare_kernel(SortInput in, const T* __restrict__ dy, T* __restrict__ d_img, T* __restrict__ dtable,
                                                                    int B, int h, int total, int pos_bits, int32_t* __restrict__ key_out,
                                                                    int32_t* __restrict__ pos_out) {
  typedef typename Pack<T, V>::type vec;
  __shared__ int lds[kOneWaves * kBins + kOneMax];    // workgroup 0: digit places [16 waves][256 bins], entries; others: flags of kFlagRows rows
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (blockIdx.x == 0) {
    int* const place = lds;
    int* const entry = lds + kOneWaves * kBins;
    constexpr int R = kOneMax / kOneThreads;
    __shared__ int wave_total[kWaves];
    const int rounds = (total + kOneThreads - 1) / kOneThreads, first = wave * 64 * rounds + lane;
    unsigned x[R];
    int key[R];
    keys_at<R>(in, first, 64, rounds, total, key);
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = r < rounds && first + 64 * r < total ? ((unsigned)key[r] << pos_bits) | (unsigned)(first + 64 * r) : 0u;
    for (int shift = 0; shift == 0 || (in.vocab >> shift) > 0; shift += kDigit) {      // the largest key is `vocab`
      const int at_bit = pos_bits + shift;
#pragma unroll
      for (int u = 0; u < kOneWaves * kBins / kOneThreads; ++u) place[u * kOneThreads + threadIdx.x] = 0;
      __syncthreads();
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (r < rounds && first + 64 * r < total) atomicAdd(&place[wave * kBins + ((x[r] >> at_bit) & (kBins - 1))], 1);
      __syncthreads();
      int all = 0, scan = 0;
      if (threadIdx.x < kBins) {
#pragma unroll
        for (int w = 0; w < kOneWaves; ++w) all += place[w * kBins + threadIdx.x];
        scan = all;                                    // inclusive over the bins
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int v = __shfl_up(scan, o, 64);
          if (lane >= o) scan += v;
        }
        if (lane == 63) wave_total[wave] = scan;
      }
      __syncthreads();
      if (threadIdx.x < kBins) {
        int at = scan - all;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) if (w < wave) at += wave_total[w];
#pragma unroll
        for (int w = 0; w < kOneWaves; ++w) { const int v = place[w * kBins + threadIdx.x]; place[w * kBins + threadIdx.x] = at; at += v; }
      }
      __syncthreads();
      volatile int* mine = place + wave * kBins;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (r < rounds) {
          const bool live = first + 64 * r < total;
          const int dgt = (x[r] >> at_bit) & (kBins - 1);
          unsigned long long same = __ballot(live);      // lanes of this round with the same digit
#pragma unroll
          for (int b = 0; b < kDigit; ++b) {
            const unsigned long long m = __ballot((dgt >> b) & 1);
            same &= ((dgt >> b) & 1) ? m : ~m;
          }
          const int rank = __popcll(same & ((1ull << lane) - 1ull));
          const int base = live ? mine[dgt] : 0;
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();               // every lane has read its base before a leader moves it
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
          if (live) {
            if (rank == 0) mine[dgt] = base + __popcll(same);
            entry[base + rank] = (int)x[r];
          }
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < R; ++r) if (r < rounds && first + 64 * r < total) x[r] = (unsigned)entry[first + 64 * r];
    }
    for (int e = threadIdx.x; e < total; e += kOneThreads) {
      const unsigned v = (unsigned)entry[e];
      key_out[e] = (int32_t)(v >> pos_bits);
      pos_out[e] = (int32_t)(v & ((1u << pos_bits) - 1u));
    }
    if (gridDim.x > 1) return;
    __syncthreads();
  }
  const int workers = gridDim.x > 1 ? gridDim.x - 1 : 1, me = gridDim.x > 1 ? (int)blockIdx.x - 1 : 0;
  const int per = (in.vocab + workers - 1) / workers, v0 = me * per, v1 = min(v0 + per, in.vocab);
  int key[kOneMax / kOneThreads];
  keys_at<kOneMax / kOneThreads>(in, threadIdx.x, kOneThreads, (total + kOneThreads - 1) / kOneThreads, total, key);
  for (int r0 = v0; r0 < v1; r0 += kFlagRows) {
    const int n = min(kFlagRows, v1 - r0);
    for (int i = threadIdx.x; i < n; i += kOneThreads) lds[i] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kOneMax / kOneThreads; ++r) {
      const int k = key[r] - r0;
      if (k >= 0 && k < n) lds[k] = 1;
    }
    __syncthreads();
    for (int r = wave; r < n; r += kOneWaves) {
      if (lds[r]) continue;
      for (int c = lane * V; c < h; c += 64 * V) *reinterpret_cast<vec*>(dtable + (int64_t)(r0 + r) * h + c) = vec{};
    }
    __syncthreads();
  }
  if (!d_img) return;
  // image-token rows: those that the sample did not use get zero
  for (int row = me * kOneWaves + wave; row < B * in.n_img; row += workers * kOneWaves) {
    const int b = row / in.n_img, t = row - b * in.n_img;
    const bool used = t < stem_n_img(in.counts, b, in.n_img);
    const T* src = dy + ((int64_t)b * in.N + t) * h;
    for (int c = lane * V; c < h; c += 64 * V) *reinterpret_cast<vec*>(d_img + (int64_t)row * h + c) = used ? *reinterpret_cast<const vec*>(src + c) : vec{};
  }
}

// ---------------------------------------------------------------- sums over the runs
constexpr int kSeg = 16;         // entries of a segment: as many rows as a thread holds in registers at once
constexpr int kFillRows = 16;    // table rows a wave looks up and, where nobody used them, fills

template <typename T, int V>
__device__ __forceinline__ void store_row(T* dst, const float* acc) {
  typename Pack<T, V>::type o = {};
#pragma unroll
  for (int k = 0; k < V; ++k) pack_set<T, V>(o, k, acc[k]);
  *reinterpret_cast<typename Pack<T, V>::type*>(dst) = o;
}

// Items [0, segs * ctiles): segment x tile of kThreads * V columns.  Items after that: fills.
// part[segment][0][h] is the piece of the run that reaches into the segment from the one before,
// part[segment][1][h] the piece of a run that starts in it and goes on in the next.
template <typename T, int V>
__global__ __launch_bounds__(kThreads) void embed_sum_kernel(const T* __restrict__ dy, const int32_t* __restrict__ key,
                                                             const int32_t* __restrict__ pos, T* __restrict__ dtable,
                                                             float* __restrict__ part, int total, int h, int vocab,
                                                             int segs, int ctiles, int fills) {
  typedef typename Pack<T, V>::type vec;
  const int sums = segs * ctiles;
  const int lane = threadIdx.x & 63;
  for (int item = blockIdx.x; item < sums + fills; item += gridDim.x) {
    if (item >= sums) {
      const int r0 = ((item - sums) * kWaves + (threadIdx.x >> 6)) * kFillRows;
      const int row = r0 + lane;
      bool empty = false;
      if (lane < kFillRows && row < vocab) {
        int lo = 0, hi = total;                        // first entry whose key is not below `row`
        while (lo < hi) { const int mid = (lo + hi) >> 1; if (key[mid] < row) lo = mid + 1; else hi = mid; }
        empty = lo >= total || key[lo] != row;
      }
      unsigned long long m = __ballot(empty);
      while (m) {
        const int r = r0 + __ffsll(m) - 1;
        m &= m - 1;
        for (int c = lane * V; c < h; c += 64 * V) *reinterpret_cast<vec*>(dtable + (int64_t)r * h + c) = vec{};
      }
      continue;
    }
    const int seg = item / ctiles, c = ((item - seg * ctiles) * kThreads + (int)threadIdx.x) * V;
    const int e0 = seg * kSeg, e1 = min(e0 + kSeg, total);
    int k[kSeg + 2];                                   // keys of the entry before, the segment, the entry after; -1: none
#pragma unroll
    for (int i = 0; i < kSeg + 2; ++i) {
      const int e = e0 + i - 1;
      k[i] = e >= 0 && e < total && e <= e1 ? key[e] : -1;
    }
    if (c >= h) continue;
    vec v[kSeg];
#pragma unroll
    for (int i = 0; i < kSeg; ++i) {
      v[i] = vec{};
      if (k[i + 1] >= 0 && k[i + 1] < vocab) v[i] = *reinterpret_cast<const vec*>(dy + (int64_t)pos[e0 + i] * h + c);
    }
    float acc[V];
#pragma unroll
    for (int q = 0; q < V; ++q) acc[q] = 0.f;
    bool from_before = k[0] == k[1];
#pragma unroll
    for (int i = 0; i < kSeg; ++i) {
      if (k[i + 1] < 0 || k[i + 1] >= vocab) continue;  // past the list, or an image token
#pragma unroll
      for (int q = 0; q < V; ++q) acc[q] += pack_get<T, V>(v[i], q);
      if (i + 1 < kSeg && k[i + 2] == k[i + 1]) continue;
      const bool goes_on = i + 1 == kSeg && k[i + 2] == k[i + 1];
      if (from_before || goes_on) {
        float* dst = part + ((int64_t)seg * 2 + (from_before ? 0 : 1)) * h + c;
#pragma unroll
        for (int q = 0; q < V; ++q) dst[q] = acc[q];
      } else {
        store_row<T, V>(dtable + (int64_t)k[i + 1] * h + c, acc);
      }
      from_before = false;
#pragma unroll
      for (int q = 0; q < V; ++q) acc[q] = 0.f;
    }
  }
}

// Runs that leave the segment they start in: the first piece plus the head pieces of the
// segments that follow, each wave a quarter of those in ascending order, the waves added in
// order.  Item = segment x 64 columns.
template <typename T>
__global__ __launch_bounds__(kThreads) void embed_join_kernel(const int32_t* __restrict__ key, const float* __restrict__ part,
                                                              T* __restrict__ dtable, int total, int h, int vocab, int segs,
                                                              int ctiles) {
  __shared__ float red[kWaves][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int items = segs * ctiles;
  // 64 of this workgroup's items are looked at together, a lane each (every wave comes to the same): few have work to do,
  // and the key loads of one after the other were most of this kernel
  for (int64_t first = blockIdx.x; first < items; first += 64ll * gridDim.x) {
    const int64_t mine = first + (int64_t)lane * gridDim.x;
    bool starts = false;                               // a run that starts in the segment goes on behind it
    if (mine < items) {
      const int seg = (int)mine / ctiles, e0 = seg * kSeg, next = e0 + kSeg;
      if (next < total) {
        const int id = key[next - 1], after = key[next], head = key[e0], before = e0 > 0 ? key[e0 - 1] : -1;
        starts = id < vocab && after == id && !(head == id && before == id);
      }
    }
    unsigned long long todo = __ballot(starts);
    while (todo) {
      const int item = (int)(first + (int64_t)(__ffsll(todo) - 1) * gridDim.x);
      todo &= todo - 1;
      const int seg = item / ctiles, c = (item - seg * ctiles) * 64 + lane;
      const int id = key[seg * kSeg + kSeg - 1];
      // segments that follow: those whose first entry is the run's, 64 looked at together
      int n = 0;
      for (bool all = true; all; ) {
        const int64_t e = (int64_t)(seg + 1 + n + lane) * kSeg;
        const unsigned long long m = ~__ballot(e < total && key[e] == id);
        all = m == 0;
        n += all ? 64 : __ffsll(m) - 1;
      }
      const int per = (n + kWaves - 1) / kWaves;
      const int s0 = seg + 1 + wave * per, s1 = min(s0 + per, seg + 1 + n);
      float acc = 0.f;
      if (c < h) {
        if (wave == 0) acc = part[((int64_t)seg * 2 + 1) * h + c];
        for (int s = s0; s < s1; s += 8) {
          float v[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) v[u] = s + u < s1 ? part[(int64_t)(s + u) * 2 * h + c] : 0.f;
#pragma unroll
          for (int u = 0; u < 8; ++u) if (s + u < s1) acc += v[u];
        }
      }
      red[wave][lane] = acc;
      __syncthreads();
      if (wave == 0 && c < h) {
#pragma unroll
        for (int w = 1; w < kWaves; ++w) acc += red[w][lane];
        dtable[(int64_t)id * h + c] = from_f32<T>(acc);
      }
      __syncthreads();
    }
  }
}

// Small calls: the workgroup that owns a table row walks all positions, 256 at a time, gathers
// those that hold its id into a list in LDS in ascending order (waves in order, lanes in order, by ballot
// and prefix count) and adds the listed rows of dy in that order, all columns of a row in registers: COLS of them a thread, ROWS
// rows requested together.  Bound by an id's rows, one batch after the other: T 128 h 64, one id for all, 58 us row by row with 32
// columns a thread, now 24; with the frequencies of running text T 128 h 512 V 1000 13.6 -> 7.5, T 96 h 64 V 32 11.9 -> 5.6.
constexpr int kScanPositions = 128, kScanCols = 32;  // columns per thread: rows of up to 8192 elements
template <typename T, int COLS, int ROWS>
__global__ __launch_bounds__(kThreads) void embed_scan_kernel(const T* __restrict__ dy, const int32_t* __restrict__ ids,
                                                              const int32_t* __restrict__ counts, T* __restrict__ dtable,
                                                              int B, int N, int n_img, int h, int vocab) {
  __shared__ int list[kScanPositions];
  __shared__ int wave_hits[kWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int total = B * N;
  for (int v = blockIdx.x; v < vocab; v += gridDim.x) {
    int n_list = 0;                                    // the same in every thread
    for (int p0 = 0; p0 < total; p0 += kThreads) {
      const int p = p0 + threadIdx.x;
      bool hit = false;
      if (p < total) {
        const int b = p / N, t = p - b * N;
        hit = t >= stem_n_img(counts, b, n_img) && stem_id(ids, counts, b, t, N, n_img, vocab) == v;
      }
      const unsigned long long m = __ballot(hit);
      if (lane == 0) wave_hits[wave] = __popcll(m);
      __syncthreads();
      int before = n_list, all = 0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) { if (w < wave) before += wave_hits[w]; all += wave_hits[w]; }
      if (hit) list[before + __popcll(m & ((1ull << lane) - 1ull))] = p;
      n_list += all;
      __syncthreads();                                 // list entries visible; wave_hits free for the next chunk
    }
    float acc[COLS] = {};
    for (int e = 0; e < n_list; e += ROWS) {
      float v[ROWS][COLS] = {};
#pragma unroll
      for (int u = 0; u < ROWS; ++u)
        if (e + u < n_list) {
          const T* row = dy + (int64_t)list[e + u] * h;
#pragma unroll
          for (int j = 0; j < COLS; ++j) {
            const int c = j * kThreads + threadIdx.x;
            if (c < h) v[u][j] = to_f32(row[c]);
          }
        }
#pragma unroll
      for (int u = 0; u < ROWS; ++u)
        if (e + u < n_list) {
#pragma unroll
          for (int j = 0; j < COLS; ++j) acc[j] += v[u][j];
        }
    }
    __syncthreads();                                   // everybody is done with the list
#pragma unroll
    for (int j = 0; j < COLS; ++j) {
      const int c = j * kThreads + threadIdx.x;
      if (c < h) dtable[(int64_t)v * h + c] = from_f32<T>(acc[j]);
    }
  }
}

// One launch of the scan against three of the sort, whatever the CUs (the orders of the sums
// differ, so the rule is one of the shape).  The scan takes a pass over the ids per table row and the rows of an id in batches one
// after the other: it loses with many rows, on few CUs first, and with many positions to an id.  Measured on 256 CUs (on 64, on 32),
// bf16, ids with the frequencies of running text, scan / sort in us:
//   T 16 h 64 V 32  4.0 / 12.2     T 96 h 512 V 1000  5.4 (5.9, 6.8) / 14.5      h 2048 V 4000  13.4 (17.4, 24.0) / 15.6
//   T 112 h 64 V 128  6.3 / 11.7   h 64 V 2000  4.0 (5.1, 7.9) / 13.4            V 4000  6.8 (17.8, 32.4) row by row / 12.9 (12.5, 12.9)
//   T 128 h 512 V 1000  7.5 (7.9, 8.9) / 12.9 (12.7, 15.3)   V 2000  6.7 (6.4, 8.4) / 12.9   h 2048 V 1000  21.7 row by row / 13.7
// and with one id for all positions: T 96 h 64  18.5 / 12;  T 128 h 64  24 / 12, h 400  36 / 12;  T 200 h 64  37 / 14, h 400  55 / 13, which is
// why more positions are sorted although T 160 h 64 V 1000 takes the scan 5.6 and the sort 13.2.
inline bool scan_is_faster(int64_t T, int64_t h, int64_t vocab) {
  if (T <= 96) return vocab <= 8192 && T <= 4 * vocab && T * h <= 1 << 18 && h <= kScanCols * kThreads;
  return T <= kScanPositions && T < vocab && vocab <= 2048 && T * h <= 1 << 16;
}

struct EmbedScratch {
  size_t key[2], pos[2], hist, part, bytes;
  EmbedScratch(int64_t total, int64_t h) {
    size_t cur = 0;
    auto take = [&](size_t n) { const size_t at = cur; cur = align_up(cur + n, 256); return at; };
    for (int i = 0; i < 2; ++i) { key[i] = take(total * 4); pos[i] = take(total * 4); }
    hist = take((size_t)ceil_div(total, kChunk) * kBins * 4);
    part = take((size_t)ceil_div(total, kSeg) * 2 * h * 4);
    bytes = cur;
  }
};

template <typename T, int V>
mosaic_status split_img(hipStream_t s, int quota, int B, int N, int n_img, int h, const T* dy, const int32_t* counts, T* d_img) {
  if (!d_img || n_img <= 0) return MOSAIC_OK;
  split_img_kernel<T, V><<<grid_for(quota, 8, ceil_div((int64_t)B * n_img, kWaves)), kThreads, 0, s>>>(dy, counts, d_img, B, N, n_img, h);
  MOSAIC_LAUNCH_CHECK();
  return MOSAIC_OK;
}

inline int bits_of(int v) { int n = 0; while (v >> n) ++n; return n; }
// One workgroup's LDS holds the positions, 32 bits a key (up to `vocab`) and its position.  One launch against five and
// more; one CU sorts, which tells at more positions.  Measured on 256 CUs, bf16, one / several launches in us:
//   T 2048 h 64 V 1048576  54 / 99     T 4096 h 2048 V 32000  33 / 54     T 8192 h 2048 V 32000  43 / 61     h 256 V 400  34 / 37
//   T 16384 h 2048 V 32000  76 / 72    h 512 V 500  63 / 43 (32 keys a thread)
// and on 64 and 8 CUs (masked streams; several launches with the join that they had): T 8192 h 2048 V 32000  59 / 111, 356 / 612;  h 256 V 400
// 40 / 47, 103 / 141;  T 1024 h 512 V 1000  16 / 28, 24 / 44;  T 2048 h 64 V 1048576  165 / 266, 1369 / 1775.
inline bool sorts_in_one(int64_t total, int64_t vocab) { return total <= kOneMax && bits_of((int)vocab) + bits_of((int)total - 1) <= 32; }

template <typename T, int V>
mosaic_status embed_grad_t(hipStream_t s, int quota, int B, int N, int n_img, int h, int vocab, const T* dy,
                           const int32_t* ids, const int32_t* counts, T* d_img, T* dtable, char* scratch) {
  const int total = B * N;
  if (scan_is_faster(total, h, vocab)) {
    MOSAIC_TRY((split_img<T, V>(s, quota, B, N, n_img, h, dy, counts, d_img)));
    const int grid = grid_for(quota, 8, vocab);
    if (h <= 2 * kThreads) embed_scan_kernel<T, 2, 8><<<grid, kThreads, 0, s>>>(dy, ids, counts, dtable, B, N, n_img, h, vocab);
    else if (h <= 8 * kThreads) embed_scan_kernel<T, 8, 4><<<grid, kThreads, 0, s>>>(dy, ids, counts, dtable, B, N, n_img, h, vocab);
    else embed_scan_kernel<T, kScanCols, 1><<<grid, kThreads, 0, s>>>(dy, ids, counts, dtable, B, N, n_img, h, vocab);
    MOSAIC_LAUNCH_CHECK();
    return MOSAIC_OK;
  }
  const int segs = (int)ceil_div(total, kSeg), ctiles = (int)ceil_div(h, kThreads * V), jtiles = (int)ceil_div(h, 64);
  const EmbedScratch sc(total, h);
  if (sorts_in_one(total, vocab)) {
    int32_t *key = (int32_t*)(scratch + sc.key[0]), *pos = (int32_t*)(scratch + sc.pos[0]);
    float* part = (float*)(scratch + sc.part);
    const SortInput in = {nullptr, nullptr, ids, counts, N, n_img, vocab};
    embed_prepare_kernel<T, V><<<grid_for(quota, 1, 1 + ceil_div(vocab, kOneWaves)), kOneThreads, 0, s>>>(in, dy, n_img > 0 ? d_img : nullptr, dtable, B, h,
                                                                                                         total, bits_of(total - 1), key, pos);
    MOSAIC_LAUNCH_CHECK();
    embed_sum_kernel<T, V><<<grid_for(quota, 8, (int64_t)segs * ctiles), kThreads, 0, s>>>(dy, key, pos, dtable, part, total, h, vocab, segs, ctiles, 0);
    MOSAIC_LAUNCH_CHECK();
    embed_join_kernel<T><<<grid_for(quota, 8, (int64_t)segs * jtiles), kThreads, 0, s>>>(key, part, dtable, total, h, vocab, segs, jtiles);
    MOSAIC_LAUNCH_CHECK();
    return MOSAIC_OK;
  }
  MOSAIC_TRY((split_img<T, V>(s, quota, B, N, n_img, h, dy, counts, d_img)));
  const int chunks = (int)ceil_div(total, kChunk);
  int32_t* key[2] = {(int32_t*)(scratch + sc.key[0]), (int32_t*)(scratch + sc.key[1])};
  int32_t* pos[2] = {(int32_t*)(scratch + sc.pos[0]), (int32_t*)(scratch + sc.pos[1])};
  int* hist = (int*)(scratch + sc.hist);
  float* part = (float*)(scratch + sc.part);
  int cur = 1;
  const int grid = grid_for(quota, 4, chunks);
  for (int shift = 0; shift == 0 || (shift < 32 && (vocab >> shift) > 0); shift += kDigit) {      // the largest key is `vocab`
    SortInput in = {shift ? key[cur] : nullptr, shift ? pos[cur] : nullptr, ids, counts, N, n_img, vocab};
    cur ^= 1;
    sort_hist_kernel<<<grid, kThreads, 0, s>>>(in, shift, total, chunks, hist);
    MOSAIC_LAUNCH_CHECK();
    sort_scatter_kernel<<<grid, kThreads, 0, s>>>(in, shift, total, chunks, hist, key[cur], pos[cur]);
    MOSAIC_LAUNCH_CHECK();
  }
  const int fills = (int)ceil_div(vocab, kWaves * kFillRows);
  if ((int64_t)segs * jtiles + fills > INT32_MAX) MOSAIC_FAIL(MOSAIC_EUNSUPPORTED, "embedding gradient over %d positions", total);
  embed_sum_kernel<T, V><<<grid_for(quota, 8, (int64_t)segs * ctiles + fills), kThreads, 0, s>>>(dy, key[cur], pos[cur], dtable, part, total, h,
                                                                                                vocab, segs, ctiles, fills);
  MOSAIC_LAUNCH_CHECK();
  embed_join_kernel<T><<<grid_for(quota, 8, (int64_t)segs * jtiles), kThreads, 0, s>>>(key[cur], part, dtable, total, h, vocab, segs, jtiles);
  MOSAIC_LAUNCH_CHECK();
  return MOSAIC_OK;
}

// 16-byte accesses where every row of every tensor starts on a 16-byte boundary (the width is a
// multiple of 16 bytes in a module); single elements for a caller's tensor that does not
template <typename T>
bool wide_rows(int h, const void* a, const void* b, const void* c) {
  return h % Vec16<T>::N == 0 && (((uintptr_t)a | (uintptr_t)b | (uintptr_t)c) & 15) == 0;
}

template <typename T>
mosaic_status text_stem_fwd_t(hipStream_t s, int quota, int B, int N, int n_img, int h, int vocab, const T* img_tok,
                              const int32_t* ids, const int32_t* counts, const T* table, T* out) {
  const int64_t rows = (int64_t)B * N;
  if (rows == 0 || h == 0) return MOSAIC_OK;
  const int grid = grid_for(quota, 8, ceil_div(rows, kWaves));
  if (wide_rows<T>(h, img_tok, table, out))
    text_stem_fwd_kernel<T, Vec16<T>::N><<<grid, kThreads, 0, s>>>(img_tok, ids, counts, table, out, B, N, n_img, h, vocab);
  else
    text_stem_fwd_kernel<T, 1><<<grid, kThreads, 0, s>>>(img_tok, ids, counts, table, out, B, N, n_img, h, vocab);
  MOSAIC_LAUNCH_CHECK();
  return MOSAIC_OK;
}

template <typename T>
mosaic_status text_stem_bwd_t(hipStream_t s, int quota, int B, int N, int n_img, int h, int vocab, const T* dy,
                              const int32_t* ids, const int32_t* counts, T* d_img, T* dtable, char* scratch) {
  const bool wide = wide_rows<T>(h, dy, d_img, dtable);
  if (wide) return embed_grad_t<T, Vec16<T>::N>(s, quota, B, N, n_img, h, vocab, dy, ids, counts, d_img, dtable, scratch);
  return embed_grad_t<T, 1>(s, quota, B, N, n_img, h, vocab, dy, ids, counts, d_img, dtable, scratch);
}

constexpr int kEmbedMaxWidth = kScanCols * kThreads;   // the widest rows that the entry point takes

}  // namespace

size_t text_stem_scratch_bytes(int64_t T, int64_t h) { return EmbedScratch(T, h).bytes; }

mosaic_status launch_text_stem_fwd(hipStream_t s, int quota, int dtype, int B, int N, int n_img, int h, int vocab,
                                   const void* img_tok, const int32_t* ids, const int32_t* counts, const void* table, void* out) {
  if (dtype == MOSAIC_BF16)
    return text_stem_fwd_t<bf16>(s, quota, B, N, n_img, h, vocab, (const bf16*)img_tok, ids, counts, (const bf16*)table, (bf16*)out);
  return text_stem_fwd_t<float>(s, quota, B, N, n_img, h, vocab, (const float*)img_tok, ids, counts, (const float*)table, (float*)out);
}

mosaic_status launch_text_stem_bwd(hipStream_t s, int quota, int dtype, int B, int N, int n_img, int h, int vocab,
                                   const void* dy, const int32_t* ids, const int32_t* counts, void* d_img, void* dtable, void* scratch) {
  if (h > kEmbedMaxWidth) MOSAIC_FAIL(MOSAIC_EUNSUPPORTED, "embedding rows of %d elements; the gradient takes up to %d", h, kEmbedMaxWidth);
  if (dtype == MOSAIC_BF16)
    return text_stem_bwd_t<bf16>(s, quota, B, N, n_img, h, vocab, (const bf16*)dy, ids, counts, (bf16*)d_img, (bf16*)dtable, (char*)scratch);
  return text_stem_bwd_t<float>(s, quota, B, N, n_img, h, vocab, (const float*)dy, ids, counts, (float*)d_img, (float*)dtable, (char*)scratch);
}
