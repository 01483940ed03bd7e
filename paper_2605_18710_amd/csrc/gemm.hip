// Linear-layer contractions (forward, input gradient, weight gradient) for gfx950.
//
// bf16 path: persistent MFMA kernels.  gemm_bf16_kernel serves every form: a workgroup of 8
// waves (256x256 tile, 128x64 per wave) or 4 waves (128x128 tile, 64x64 per wave; 64x128, 32x64 per wave) walks
// output tiles; gemm_bf16_w4_kernel (described at its definition) can take the 256x256 tiles of
// every product whose K-contiguous operands are whole 64-deep K-tiles long (the plans say when it does).  In both,
// the grid is sized to the module's CU quota.  Each output element is produced by exactly
// one wave that accumulates k in ascending order (v_mfma_f32_32x32x16_bf16 twice or
// v_mfma_f32_16x16x32_bf16 once per 32 k-values: the same bits), so the
// bits of the result do not depend on the grid, the tile shape, the tile order or the CU.
//
// Data movement (gemm_bf16_kernel)
//   * HBM -> LDS directly (buffer_load ... lds): no register staging and no LDS write
//     instructions.  A wave instruction fills 1 KB of consecutive LDS; each lane chooses
//     which 16 bytes of the tile it requests, which realises the bank swizzle.  The
//     descriptor's bounds check returns zeros for rows past the end, so ragged tiles need
//     no branches.
//   * an operand whose contraction index is contiguous in HBM sits in LDS as rows of 32
//     k-values (64 bytes), 16-byte chunks XOR-swizzled by (row/4)%4, and is read with
//     ds_read_b128.  An operand whose contraction index is the strided one (the weight in
//     the forward pass, both operands of the weight gradient) sits in LDS as it is in HBM,
//     k-row by k-row with 64-byte chunks XOR-swizzled by k%4, and its fragments come out
//     with the transposing read ds_read_b64_tr_b16 (two per fragment).
//   * five LDS stages: while K-tile t is multiplied, t+1 is visible (its first fragments
//     are fetched before the barrier), t+2 is complete or landing and t+3 / t+4 are in
//     flight.  One barrier per K-tile; before it every wave waits (vmcnt) for its own
//     requests of tile t+2.  The stream of K-tiles runs across output tiles, so a new
//     output tile starts without a pipeline refill.
//   * fragments are double-buffered in registers: the reads for the next batch of MFMAs
//     are issued under the current batch, one fragment and one request per MFMA slot
//     (a scheduling barrier after every slot keeps the written order).
//   * accumulators are kept transposed (the weight-side fragment is MFMA's first operand),
//     so a lane owns four consecutive output columns per register group; the epilogue
//     (bias, residual, bf16 rounding) is staged through the free LDS stage into
//     row-contiguous 16-byte stores that fill whole 128-byte lines of the output.
//   * tiles are handed out so that the workgroups running on one XCD at the same time
//     form a 4 x 8 patch of the tile grid and share operand panels in that XCD's L2.
//
// fp32 path, and shapes these kernels do not cover: gemm_f32.hip.
#include <stdlib.h>
#include <algorithm>
#include <mutex>
#include <type_traits>
#include "activations.h"
#include "gemm_plan.h"
#include "kernels.h"
#include "tile_queue.h"

namespace {

#pragma clang diagnostic ignored "-Winline-asm"   // m0 is named as a clobber on purpose

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;

constexpr int BK = 32;            // k-values per K-tile (64 bytes of a K-contiguous row); 64 where stated (BKT)
constexpr unsigned kOob = 0xFFFFFFF0u;   // byte offset beyond any descriptor's range

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}

typedef __attribute__((address_space(3))) unsigned char lds_byte;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;
constexpr int NS = 5;             // LDS stages
constexpr int AHEAD = 4;          // K-tiles between the load cursor and the compute cursor

// position of 16-byte chunk c of row r of a K-contiguous tile: c ^ kc_swizzle(r); 16 lanes that
// read one chunk of 16 consecutive rows touch every bank once
template <int BKT> __device__ __forceinline__ int kc_swizzle(int r) { return BKT == 64 ? (r >> 1) & 7 : (r >> 2) & 3; }

// Requests one operand tile (ROWS x BKT) from HBM straight into an LDS stage: every wave
// instruction moves 64 x 16 bytes to 1 KB of consecutive LDS; which 16 bytes of the tile a
// lane asks for is free, and that choice realises the swizzle.
//   K-contiguous operand: LDS rows of 64 bytes (32 k-values of one tile row; 128 bytes when
//     K-tiles are 64 deep), the 16-byte chunks of row r stored at position chunk ^ kc_swizzle(r).
//   K-strided operand: LDS rows of ROWS*2 bytes (one k-row of the tile), the 64-byte chunks
//     of k-row k stored at position chunk ^ k%4; fragments come out with transposing reads.
// GU (K-strided operand only): the tile's columns are not consecutive columns of the matrix.
// The matrix is [gate | up] halves of gu_f columns each; 32-column group c of the tile is
// group c/2 of the gate half (c even) or of the up half (c odd), counted from column x0/2,
// so that a wave's two 32-column accumulator blocks hold a gate column and its up column
// in the same lane and register.
template <int ROWS, bool KC, int NWAVES, bool GU = false, int BKT = BK>
struct DmaLoader {
  static constexpr int NI = ROWS * BKT / 512 / NWAVES;     // wave instructions per wave and K-tile
  static constexpr int ROWB = ROWS * 2;             // strided: bytes per k-row
  static constexpr int RPI = 1024 / ROWB;           // strided: k-rows per wave instruction
  struct Tile { unsigned org; unsigned oobmask; };

  unsigned rel[NI];     // byte offset of instruction j's chunk relative to the tile origin at K-tile 0
  unsigned kstep;       // bytes between consecutive K-tiles
  int kofs;             // KC: first k of this lane's chunk
  int xofs[NI];         // strided: first tile column of this lane's chunk
  int wave_base;        // LDS byte offset of this wave's first instruction inside the operand area

  __device__ __forceinline__ void init(int64_t ld, int gu_f = 0) {
    static_assert(!(GU && KC), "the gate/up column map exists for the K-strided operand");
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    wave_base = w * NI * 1024;
    kofs = 0;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      if constexpr (KC) {
        constexpr int CPR = BKT / 8;               // 16-byte chunks per row
        const int r = 64 / CPR * (w * NI + j) + lane / CPR, pos = lane % CPR;
        const int ch = pos ^ kc_swizzle<BKT>(r);
        if (j == 0) kofs = ch * 8;
        rel[j] = (unsigned)(((int64_t)r * ld + ch * 8) * 2);
        xofs[j] = 0;
        kstep = BKT * 2;
      } else {
        const int byte = 16 * lane;
        const int kr = (w * NI + j) * RPI + byte / ROWB, bp = byte % ROWB;
        const int c64 = (bp >> 6) ^ (kr & 3), p = (bp & 63) >> 4;
        xofs[j] = c64 * 32 + p * 8;
        int64_t gcol = xofs[j];
        if constexpr (GU) gcol = (c64 >> 1) * 32 + p * 8 + (int64_t)(c64 & 1) * gu_f;
        rel[j] = (unsigned)(((int64_t)kr * ld + gcol) * 2);
        kstep = (unsigned)(BKT * ld * 2);
      }
    }
  }

  __device__ __forceinline__ Tile tile(int64_t ld, int x0, int X) const {
    Tile tl;
    tl.oobmask = 0;
    if constexpr (KC) tl.org = (unsigned)((int64_t)x0 * ld * 2);
    else if constexpr (GU) tl.org = (unsigned)x0;      // column x0/2 of each half, 2 bytes each; halves are whole tiles wide
    else {
      tl.org = (unsigned)(x0 * 2);
#pragma unroll
      for (int j = 0; j < NI; ++j) if (x0 + xofs[j] >= X) tl.oobmask |= 1u << j;
    }
    return tl;
  }

  // K-tile kt (absolute index) of tile tl -> operand area `dst` of a stage; zeros when
  // !valid, at or past kt_lim, or outside the matrix (rows past the end fall outside the
  // descriptor's range).  prep() holds what the NI requests of one K-tile share; issue_j()
  // makes request j, so that the caller can spread the requests over its instruction stream.
  struct Prep { bool oob, oob_odd; unsigned base; };
  __device__ __forceinline__ Prep prep(const Tile& tl, int kt, int K, int kt_lim, bool valid) const {
    Prep p;
    p.oob = !valid || kt >= kt_lim;
    p.oob_odd = p.oob;
    if constexpr (KC) {
      // at 64 k-values a row the swizzle of odd instructions (8 rows on) differs in its top bit
      static_assert(BKT == 32 || NI % 2 == 0, "a wave starts on an even instruction");
      p.oob_odd = p.oob || (kt * BKT + (BKT == 64 ? kofs ^ 32 : kofs)) >= K;
      p.oob = p.oob || (kt * BKT + kofs) >= K;
    }
    p.base = tl.org + (unsigned)kt * kstep;
    return p;
  }
  __device__ __forceinline__ void issue_j(i32x4 rsrc, const Tile& tl, const Prep& p, int j, unsigned dst) const {
    const unsigned off = (((j & 1) ? p.oob_odd : p.oob) || ((tl.oobmask >> j) & 1)) ? kOob : p.base + rel[j];
    // m0 = LDS byte address of lane 0's 16 bytes; lane l lands at m0 + 16*l.  Written as
    // assembly so that the compiler's wait-count pass does not see an LDS write and put a
    // full vmcnt(0) in front of every following LDS read; completion is waited for by
    // hand (wait_loads in the kernel).  The compiler itself never uses m0 in this file.
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 : : "s"(dst + (unsigned)(wave_base + j * 1024)), "v"(off), "s"(rsrc) : "m0");
  }
  __device__ __forceinline__ void issue(i32x4 rsrc, const Tile& tl, int kt, int K, int kt_lim,
                                        bool valid, unsigned dst) const {
    const Prep p = prep(tl, kt, K, kt_lim, valid);
#pragma unroll
    for (int j = 0; j < NI; ++j) issue_j(rsrc, tl, p, j, dst);
  }
};

// Fragment addresses of one operand inside its stage area: NF blocks of 32 tile rows
// starting at row w0, for lane (lr = lane%32, hb = lane/32).
template <int ROWS, bool KC, int NF, int BKT = BK>
struct FragReader {
  int addr[KC ? 1 : NF];
  int ch[BKT / 16];
  __device__ __forceinline__ void init(int w0) {
    const int lane = threadIdx.x & 63;
    if constexpr (KC) {
      const int lr = lane & 31, hb = lane >> 5, sw = kc_swizzle<BKT>(lr);
      addr[0] = (w0 + lr) * (BKT * 2);
#pragma unroll
      for (int ks = 0; ks < BKT / 16; ++ks) ch[ks] = ((2 * ks + hb) ^ sw) << 4;
    } else {
      const int G = lane >> 4, i = lane & 15, hh = G >> 1, q = i >> 2, g = i & 3;
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        const int c64 = (w0 + 32 * f) >> 5;
        addr[f] = (8 * hh + q) * (ROWS * 2) + ((c64 ^ q) << 6) + 32 * (G & 1) + 8 * g;
      }
#pragma unroll
      for (int ks = 0; ks < BKT / 16; ++ks) ch[ks] = 0;
    }
  }
  // fragment f for k-step ks of the K-tile in operand area `base`
  __device__ __forceinline__ bf16x8 read(const lds_byte* base, int f, int ks) const {
    if constexpr (KC) {
      return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(base + addr[0] + f * 32 * (BKT * 2) + ch[ks]);
    } else {
      const lds_byte* p = base + addr[f] + ks * 16 * (ROWS * 2);
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p + 4 * (ROWS * 2)));
      typedef __attribute__((ext_vector_type(8))) short s16x8;
      const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      return __builtin_bit_cast(bf16x8, v);
    }
  }
};

// Position `tile` of the tile list -> (tile row, tile column).  The list is panel-major: panels
// of 8 tile columns, row-major inside a panel, so 32 consecutive entries form a 4 x 8 patch that
// shares operand panels in one XCD's L2.  Above that, tile rows are taken in super-blocks of
// `row_block` rows (all panels of a super-block before the next super-block), sized on the
// host so that the row operand of a super-block (row_block x 256 rows x K) stays in the
// last-level cache: it is then re-read from there, not from HBM, once per panel (measured on
// the 7B-shaped products: +3 % forward, +4 % input gradient; the board is power-bound and HBM
// reads cost energy).  Both kernels and both launches of a mixed plan use this one order.
__device__ __forceinline__ void tile_coords(int tile, int tiles_m, int tiles_n, int row_block, int* row, int* col) {
  const int per_sb = row_block * tiles_n;
  const int sb = tile / per_sb, rem = tile - sb * per_sb;
  const int rows_sb = min(row_block, tiles_m - sb * row_block);
  const int panel = rem / (rows_sb * 8);
  const int pw = min(8, tiles_n - panel * 8);
  const int in_panel = rem - panel * rows_sb * 8;
  *row = sb * row_block + in_panel / pw;
  *col = panel * 8 + in_panel % pw;
}

// One unit of work: an output tile, or (PIECES_APART) one K-piece of an output tile.
struct WorkItem {
  int m0, n0, kt0, kt_end, split, tl;      // tl: position of the item's coarse tile in this launch's range
  bool valid;
};

// PIECES_APART: the K range is cut into `ksplit` contiguous pieces of `ktiles_per` K-tiles; piece s
// of the launch's t-th tile is accumulated by its own workgroup and stored in fp32 to
// P[s][t][BM][BN]; a second kernel adds the pieces in ascending s.  Which tiles are cut and
// into how many pieces depends on the problem shape only.
//
// A workgroup streams the K-tiles of ALL its work items through one pipeline: a load
// cursor runs AHEAD K-tiles ahead of the compute cursor and crosses item boundaries, so
// the first tiles of the next item are already in LDS while the epilogue of the current one
// runs (the other wave on the SIMD keeps the matrix cores busy meanwhile).
//
// ACT (forward form only): the epilogue also writes an activation of the output to C2, so the
// pass that would read the output back is never launched.  ACT_GELU: C2 = gelu(C), same shape.
// ACT_SWIGLU: C is [gate | up] with gu_f columns each and C2[M, gu_f] = silu(gate) * up; the
// weight tile's columns are gathered so that a wave holds matching gate and up columns
// (DmaLoader GU).  The activation is taken of the bf16 value that is stored to C, as the
// separate pass would.
constexpr int ACT_NONE = 0, ACT_GELU = 1, ACT_SWIGLU = 2, ACT_TAPS = 3;
struct ActArgs {
  int act = ACT_NONE;
  bf16* C2 = nullptr;
  int64_t ldc2 = 0;
  uint32_t c2_bytes = 0;
  int gu_f = 0;
  int row_block = 1 << 20;   // tile rows per super-block of the tile order (set by the launcher)
  uint32_t r_rows = 0, r_magic = 0;   // r_rows > 0: R has that many rows, and row r of C gets row r mod r_rows (a position table)
  // ACT_TAPS: GELU, and C2 is the gathered input [M / 2, 3N] of a three-tap convolution of stride 2 over samples of 2 * r_rows rows
};
// Where row r of the activation goes in that input (24000 x 1280 from 240 k-values: product 59 us and gather 35 -> 82): tap 1 of output r / 2 (even rows), or tap 2 of it and tap 0 of the next one; the last row
// of a sample, which has no next one, clears tap 0 of the sample's first output.  Element offsets of its first column, -1: none.
struct TapRows { int64_t first, second; bool zero; };
// r mod r_rows with r_magic = 2^32 / r_rows + 1: exact as long as r * r_rows < 2^32 (checked by the launcher)
__device__ __forceinline__ int table_row(int r, uint32_t r_rows, uint32_t r_magic) { return r - (int)(__umulhi((uint32_t)r, r_magic) * r_rows); }
__device__ __forceinline__ TapRows tap_rows(int r, int M, int64_t n, uint32_t lo, uint32_t magic) {
  const int t = r >> 1;
  TapRows o = {-1, -1, false};
  if (r < M) {
    o.first = (3 * (int64_t)t + 1 + (r & 1)) * n;
    if (r & 1) {
      o.zero = table_row(t + 1, lo, magic) == 0;
      o.second = 3 * (int64_t)(o.zero ? t + 1 - (int)lo : t + 1) * n;
    }
  }
  return o;
}

// PIECES_CHAINED: one workgroup takes the pieces of its tile one after the other and adds them in registers,
// in the order and with the additions of the second kernel: the same bits as PIECES_APART, no scratch.
constexpr int PIECES_NONE = 0, PIECES_APART = 1, PIECES_CHAINED = 2;
template <int BM, int BN, int NWM, int NWN, bool A_KC, bool B_KC, int PIECES, int ACT = ACT_NONE, int BKT = BK>
__device__ __forceinline__ void gemm_bf16_body(
    const bf16* __restrict__ A, const bf16* __restrict__ B, bf16* __restrict__ C,
    const bf16* __restrict__ bias, const bf16* __restrict__ R, int M, int N, int K,
    int64_t lda, int64_t ldb, int64_t ldc, uint32_t a_bytes, uint32_t b_bytes, uint32_t c_bytes,
    int tiles_m, int tiles_n, int tile_begin, int tile_count, int sub, int ksplit, int ktiles_per,
    float* __restrict__ P, const TileQueueArgs& tq, const ActArgs& aa) {
  constexpr bool SPLITK = PIECES == PIECES_APART, CHAINED = PIECES == PIECES_CHAINED;
  static_assert(ACT == ACT_NONE || (A_KC && !B_KC && PIECES == PIECES_NONE), "activation epilogues exist for the forward form");
  constexpr int NT = 64 * NWM * NWN;
  constexpr int WM = BM / NWM, WN = BN / NWN;   // wave tile
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int AREA_A = BM * BKT * 2;      // bytes of the row operand in a stage
  constexpr int STAGE = AREA_A + BN * BKT * 2;     // bytes per LDS stage
  extern __shared__ __align__(16) unsigned char smem[];

  const __amdgpu_buffer_rsrc_t ra = make_rsrc(A, a_bytes), rb = make_rsrc(B, b_bytes);
  const __amdgpu_buffer_rsrc_t rc = make_rsrc(C, c_bytes);
  const __amdgpu_buffer_rsrc_t rr = make_rsrc(R, !R ? 0u : aa.r_rows ? (uint32_t)(aa.r_rows * ldc * 2) : c_bytes);
  const __amdgpu_buffer_rsrc_t rbias = make_rsrc(bias, bias ? (uint32_t)N * 2u : 0u);

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = (wave / NWN) * WM, wn = (wave % NWN) * WN;
  const int lr = lane & 31, hb = lane >> 5;
  lds_byte* const lds = (lds_byte*)smem;
  const int nk_all = (K + BKT - 1) / BKT;

  // Work order.  The output is cut into coarse tiles of (sub*BM) x (sub*BN), listed
  // panel-major: panels of 8 coarse-tile columns, row-major inside a panel, so 32 consecutive
  // entries form a 4 x 8 patch that shares operand panels.  This launch covers entries
  // [tile_begin, tile_begin + tile_count) of that list, each as sub*sub tiles of BM x BN
  // (sub = 2: the 128x128 kernel finishing the quarter tiles of the 256x256 tiles that did
  // not fill a whole round of the large kernel), once per split piece (split-major).  The
  // flat list of these items is handed out by the work queue (tile_queue.h): a chunk of as
  // many consecutive items as an XCD has resident workgroups goes to the list of one XCD, so
  // the workgroups of an XCD work on one patch at a time and reuse each other's panels in
  // that XCD's L2.
  const int per_split = tile_count * sub * sub;
  auto decode = [&](int item) -> WorkItem {
    WorkItem it;
    it.valid = item >= 0; it.m0 = 0; it.n0 = 0; it.kt0 = 0; it.kt_end = 0; it.split = 0; it.tl = 0;
    if (!it.valid) return it;
    it.split = item / per_split;
    const int fine = item - it.split * per_split;
    const int quad = fine % (sub * sub);
    it.tl = fine / (sub * sub);
    const int tile = tile_begin + it.tl;
    it.kt0 = it.split * ktiles_per;
    it.kt_end = SPLITK ? min(nk_all, it.kt0 + ktiles_per) : nk_all;
    int trow, tcol;
    tile_coords(tile, tiles_m, tiles_n, aa.row_block, &trow, &tcol);
    it.m0 = (trow * sub + quad / sub) * BM;
    it.n0 = (tcol * sub + quad % sub) * BN;
    return it;
  };

  // stage ring: K-tile number t of the stream lives in stage t % NS
  int si = 0;                                   // stage of the compute cursor's K-tile
  auto stg = [&](int ahead) { const int i = si + ahead; return (i >= NS ? i - NS : i) * STAGE; };

  // Drawing items.  Thread 0 talks to the queue and hands the item to the workgroup through
  // four bytes of the LDS stage that is free between two pipeline steps (the kernel's LDS is
  // otherwise full).  A draw is a round trip to memory.  The first item is drawn at the start;
  // the second when the load cursor asks for it (once per workgroup, in mid-pipeline: drawn
  // earlier, a workgroup that started first would take items from workgroups that have not
  // started yet); from then on one item is claimed at the start of every epilogue and resolved
  // at its end, so the round trip hides under the epilogue.  `drawn` holds an item drawn
  // ahead; `lq` the items the load cursor has entered and the compute cursor has not.
  TileQueueCursor qc;
  bool drained = false;
  int drawn = -1;
  bool have_drawn = false;
  // Claiming under the epilogue takes the item after the next, a whole tile before it is needed.
  // That is harmless while the list is long, but near its end a workgroup a few microseconds
  // ahead of the others would take two of the last items and leave another workgroup with
  // none (measured: a launch of exactly two rounds took three).  So an item comes with a
  // flag: `ahead_ok` says that the list it came from (this XCD's own) still held two rounds of
  // work after the claim; without it the next item is drawn when the load cursor asks for it.
  bool ahead_ok = false;
  auto publish = [&](int v) -> int {           // v is thread 0's (item | flag << 30); returns the item to every thread
    volatile int* mail = reinterpret_cast<volatile int*>(smem + stg(AHEAD));
    if (threadIdx.x == 0) *mail = v;
    __syncthreads();
    const int r = __builtin_amdgcn_readfirstlane(*mail);
    __syncthreads();                           // read by all before the stage is filled again
    if (r < 0) { drained = true; ahead_ok = false; return -1; }
    ahead_ok = (r >> 30) != 0;
    return r & 0x3fffffff;
  };
  int home_list = -1;                          // thread 0: the list of the XCD this workgroup runs on
  auto flagged = [&](int item, int left) -> int {
    if (item < 0) return -1;
    return item | ((qc.list == home_list && left >= 2 * tq.chunk) ? (1 << 30) : 0);
  };
  auto draw_sync = [&]() -> int {
    if (drained) return -1;
    if (tq.mode == TQ_ROUNDS) {                // static rounds: every thread computes its item
      const int r = tq_rounds_item(tq, ++qc.round);
      if (r < 0) drained = true;
      return r;
    }
    int v = -1;
    if (threadIdx.x == 0) { int left = 0; const int it = tq_resolve(tq, qc, tq_claim(tq, qc), &left); v = flagged(it, left); }
    return publish(v);
  };
  auto draw_first = [&]() -> int {
    if (tq.mode == TQ_ROUNDS) {
      const int r = tq_first_item(tq, qc);
      if (r < 0) drained = true;
      return r;
    }
    int v = -1;
    if (threadIdx.x == 0) {
      qc.init();
      home_list = qc.list;
      int left = 0;
      const int it = tq_resolve(tq, qc, tq_claim(tq, qc), &left);
      v = flagged(it, left);
    }
    const int r = publish(v);
    if (tq.mode != TQ_QUEUE) drained = true;   // one item per workgroup at most
    return r;
  };
  auto next_drawn = [&]() -> int {             // the next item in draw order
    if (have_drawn) { have_drawn = false; return drawn; }
    return draw_sync();
  };
  int lq0 = -1, lq1 = -1, lq2 = -1, lq3 = -1, lq4 = -1, lq5 = -1, lqn = 0;
  auto lq_push = [&](int v) {
    lq0 = lqn == 0 ? v : lq0; lq1 = lqn == 1 ? v : lq1; lq2 = lqn == 2 ? v : lq2;
    lq3 = lqn == 3 ? v : lq3; lq4 = lqn == 4 ? v : lq4; lq5 = lqn == 5 ? v : lq5;
    ++lqn;
  };
  auto lq_pop = [&]() -> int {
    const int v = lq0;
    lq0 = lq1; lq1 = lq2; lq2 = lq3; lq3 = lq4; lq4 = lq5; lq5 = -1;
    --lqn;
    return v;
  };

  WorkItem cur = decode(draw_first());
  if (!cur.valid) {                // a workgroup that started after the queue ran dry
    if (threadIdx.x == 0) tq_leave(tq);
    return;
  }

  typedef DmaLoader<BM, A_KC, NWM * NWN, false, BKT> LA;
  typedef DmaLoader<BN, B_KC, NWM * NWN, ACT == ACT_SWIGLU, BKT> LB;
  LA la; LB lb;
  la.init(lda); lb.init(ldb, aa.gu_f);
  constexpr int NLOADS = LA::NI + LB::NI;      // requests per lane and K-tile

  // load cursor: the next K-tile to request
  WorkItem lit = cur;
  int lkt = cur.kt0;
  typename LA::Tile lta = la.tile(lda, lit.m0, M);
  typename LB::Tile ltb = lb.tile(ldb, lit.n0, N);
  // buffer descriptors for the direct-to-LDS requests: base, no stride, size in bytes, raw 32-bit format
  auto desc = [](const void* p, uint32_t bytes) {
    i32x4 d;
    d.x = (int)(uint32_t)(uintptr_t)p; d.y = (int)((uint32_t)((uintptr_t)p >> 32) & 0xffffu);
    d.z = (int)bytes; d.w = 0x00020000;
    return d;
  };
  const i32x4 da = desc(A, a_bytes), db = desc(B, b_bytes);
  const unsigned lds0 = (unsigned)(uintptr_t)lds;      // LDS byte address of the dynamic segment
  auto issue = [&](int stage) {
    la.issue(da, lta, lkt, K, lit.kt_end, lit.valid, lds0 + (unsigned)stage);
    lb.issue(db, ltb, lkt, K, lit.kt_end, lit.valid, lds0 + (unsigned)(stage + AREA_A));
  };
  auto load_cursor_next_item = [&]() {
    const int item = next_drawn();
    if (item >= 0) lq_push(item);
    lit = decode(item);
    lkt = lit.kt0;
    lta = la.tile(lda, lit.m0, M);
    ltb = lb.tile(ldb, lit.n0, N);
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // vmcnt(n) alone: lgkmcnt and expcnt fields at "no wait"
  auto wait_loads = [](auto n) { constexpr int N = decltype(n)::value; __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14)); };

  // prologue: the first AHEAD K-tiles of the stream are requested; the first two must have
  // landed before anyone reads
#pragma unroll
  for (int u = 0; u < AHEAD; ++u) {
    issue(u * STAGE);
    if (++lkt >= lit.kt_end && lit.valid) load_cursor_next_item();
  }
  wait_loads(std::integral_constant<int, 2 * NLOADS>{});
  __syncthreads();

  FragReader<BM, A_KC, TM, BKT> fra; FragReader<BN, B_KC, TN, BKT> frb;
  fra.init(wm); frb.init(wn);
  bf16x8 fa0[TM], fb0[TN], fa1[TM], fb1[TN];
  auto frags = [&](bf16x8* fa, bf16x8* fb, int stage, int ks) {
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[i] = fra.read(lds + stage, i, ks);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[j] = frb.read(lds + stage + AREA_A, j, ks);
  };
  frags(fa0, fb0, 0, 0);

  // Epilogue of one work item.  acc[i][j][4g+e] is output (row m0+wm+32i+lr, column
  // n0+wn+32j+8g+4hb+e): a lane holds 4-column pieces of 32 different rows, which would
  // reach memory as 8-byte fragments.  The accumulators therefore pass through a 4 KB
  // per-wave patch of the LDS stage that is free between two pipeline steps (XOR swizzled)
  // and leave row-contiguous.
  // Three variants, chosen by a uniform branch, so that each holds no request it does not
  // need.  The compiler's wait before a use of a loaded value counts every request of the
  // wave in issue order, stores included: a bias or residual request issued between two
  // stores makes the block that uses it wait until all earlier blocks' stores have been
  // acknowledged.
  //   EPI_PLAIN: no bias, no residual - stores only, nothing waits        (finish_rows)
  //   EPI_BIAS:  every bias value is requested before the first store     (finish_rows)
  //   EPI_RES:   residual (and bias, if any: a null bias reads zeros through its empty
  //              descriptor); the requests for block b+1 are issued before block b is stored,
  //              so a wait never covers the newest stores                 (finish_impl)
  // finish_impl moves one 32x32 block at a time in fp32 and adds bias and residual in
  // row-contiguous layout (fp32, one rounding); split-K pieces take the same path and leave
  // as fp32.
  constexpr int EPI_PLAIN = 0, EPI_BIAS = 1, EPI_RES = 2;
  auto finish_impl = [&](const WorkItem& it, int free_stage, auto mode_) {
    constexpr int MODE = decltype(mode_)::value;
    float* patch = reinterpret_cast<float*>(smem + free_stage) + wave * 1024;
    // The lane index passes through an empty asm so that the write-back offsets are computed
    // here, per tile, instead of being kept in registers across the K loop.
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int elr = ln & 31, ehb = ln >> 5;
    // Blocks leave in the order b = i * TN + j (row block i outer, column block j inner):
    // the two 64-byte halves of a 128-byte line of C belong to column blocks j, j+1 of the
    // same rows and are stored back to back, so they meet in the L2 before the line is
    // written out.
    // byte offset in C (and in the residual) of the 8 columns this lane writes back for row
    // half q of block b; rows past M fall outside the descriptor's range
    auto out_off = [&](int b, int q) -> unsigned {
      const int row = it.m0 + wm + 32 * (b / TN) + (ln >> 2) + 16 * q;
      const int col = it.n0 + wn + 32 * (b % TN) + 8 * (ln & 3);
      return (col < N) ? (unsigned)(((int64_t)row * ldc + col) * 2) : kOob;
    };
    auto res_off = [&](int b, int q) -> int {            // the same in R
      if (!aa.r_rows) return (int)out_off(b, q);
      const int row = table_row(it.m0 + wm + 32 * (b / TN) + (ln >> 2) + 16 * q, aa.r_rows, aa.r_magic);
      const int col = it.n0 + wn + 32 * (b % TN) + 8 * (ln & 3);
      return (col < N) ? (int)(unsigned)(((int64_t)row * ldc + col) * 2) : (int)kOob;
    };
    // bias for the 8 columns this lane writes back in column block j (same for every row block)
    auto bias_req = [&](int j) -> u32x4 {
      const int col = it.n0 + wn + 32 * j + 8 * (ln & 3);
      return __builtin_amdgcn_raw_buffer_load_b128(rbias, col < N ? col * 2 : (int)kOob, 0, 0);
    };
    u32x4 rnext[2] = {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}};
    u32x4 braw[MODE == EPI_BIAS ? TN : 1] = {};
    u32x4 bnext = {0u, 0u, 0u, 0u};
    if constexpr (MODE == EPI_BIAS) {
#pragma unroll
      for (int j = 0; j < TN; ++j) braw[j] = bias_req(j);
    }
    if constexpr (MODE == EPI_RES) {
      bnext = bias_req(0);
#pragma unroll
      for (int q = 0; q < 2; ++q) rnext[q] = __builtin_amdgcn_raw_buffer_load_b128(rr, res_off(0, q), 0, 0);
    }
#pragma unroll
    for (int b = 0; b < TM * TN; ++b) {
      const int i = b / TN, j = b % TN;
      const int cb = it.n0 + wn + 32 * j;                 // first column of the block
      const int rb0 = it.m0 + wm + 32 * i;                // first row of the block
      float bvals[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) bvals[e] = 0.f;
      if constexpr (MODE != EPI_PLAIN) {
        const bf16x8 bv = __builtin_bit_cast(bf16x8, MODE == EPI_BIAS ? braw[MODE == EPI_BIAS ? j : 0] : bnext);
#pragma unroll
        for (int e = 0; e < 8; ++e) bvals[e] = (float)bv[e];
      }
      {
        // accumulator layout -> LDS: row lr, column group cg = 2g + hb (4 columns each)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int cg = (2 * g + ehb) ^ ((elr >> 1) & 7);
          float4 v = make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
          *reinterpret_cast<float4*>(patch + elr * 32 + cg * 4) = v;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if constexpr (SPLITK) {
          float* Ps = P + ((int64_t)it.split * tile_count + it.tl) * (BM * BN);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int r = (ln >> 3) + 8 * q, cgl = ln & 7;
            const float4 v = *reinterpret_cast<const float4*>(patch + r * 32 + ((cgl ^ ((r >> 1) & 7)) * 4));
            const int row = rb0 + r, col = cb + 4 * cgl;
            if (row < M && col < N) *reinterpret_cast<float4*>(Ps + (row - it.m0) * BN + (col - it.n0)) = v;
          }
        } else {
          float4 v0[2], v1[2];
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int r = (ln >> 2) + 16 * q, c8 = ln & 3;
            const int sx = (r >> 1) & 7;
            v0[q] = *reinterpret_cast<const float4*>(patch + r * 32 + (((2 * c8) ^ sx) * 4));
            v1[q] = *reinterpret_cast<const float4*>(patch + r * 32 + (((2 * c8 + 1) ^ sx) * 4));
          }
          const u32x4 rcur[2] = {rnext[0], rnext[1]};
          if constexpr (MODE == EPI_RES) {
            if (b + 1 < TM * TN) {
#pragma unroll
              for (int q = 0; q < 2; ++q) rnext[q] = __builtin_amdgcn_raw_buffer_load_b128(rr, res_off(b + 1, q), 0, 0);
              bnext = bias_req((b + 1) % TN);
            }
          }
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const bf16x8 rv = __builtin_bit_cast(bf16x8, rcur[q]);
            const float vals[8] = {v0[q].x, v0[q].y, v0[q].z, v0[q].w, v1[q].x, v1[q].y, v1[q].z, v1[q].w};
            bf16x8 o;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              // one order of additions in every variant (value + bias + residual; the absent
              // terms are exact zeros), so the variant never changes a bit
              float v = vals[e];
              if constexpr (MODE != EPI_PLAIN) v += bvals[e];
              if constexpr (MODE == EPI_RES) v += (float)rv[e];
              o[e] = (bf16)v;
            }
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), rc, (int)out_off(b, q), 0, 0);
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    __syncthreads();               // the patch lives in the stage the next step overwrites
  };
  // Plain and bias variants when the wave tile is 64 columns wide: the two column blocks of
  // a row block are rounded to bf16 in accumulator layout (bias added in fp32 first) and
  // pass through the patch together as 32 rows of 128 bytes, 16-byte chunks XOR-swizzled
  // by (row/2)%8; they leave as whole 128-byte lines, 8 rows per store instruction.
  auto finish_rows = [&](const WorkItem& it, int free_stage, auto mode_) {
    constexpr int MODE = decltype(mode_)::value;
    static_assert(TN % 2 == 0, "row-wide epilogue moves 64-column halves of the wave tile");
    unsigned char* patch = smem + free_stage + wave * 4096;
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int elr = ln & 31, ehb = ln >> 5;
    // bias of the columns this lane holds in accumulator layout: block j, group g -> 4 values
    u32x2 braw[MODE == EPI_BIAS ? TN * 4 : 1] = {};
    if constexpr (MODE == EPI_BIAS) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int col = it.n0 + wn + 32 * j + 8 * g + 4 * ehb;
          braw[4 * j + g] = __builtin_amdgcn_raw_buffer_load_b64(rbias, col < N ? col * 2 : (int)kOob, 0, 0);
        }
    }
    const int wr = elr * 128 + ehb * 8, wsx = (elr >> 1) & 7;
    const int c16 = ln & 7;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int h = 0; h < TN / 2; ++h) {         // 64-column halves of the wave tile
        const int ocol = it.n0 + wn + 64 * h + 8 * c16;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            bf16x4 o;
            bf16x4 bv = {};
            if constexpr (MODE == EPI_BIAS) bv = __builtin_bit_cast(bf16x4, braw[4 * (2 * h + j) + g]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              float v = acc[i][2 * h + j][4 * g + e];
              if constexpr (MODE == EPI_BIAS) v += (float)bv[e];
              o[e] = (bf16)v;
            }
            *reinterpret_cast<bf16x4*>(patch + wr + (((4 * j + g) ^ wsx) << 4)) = o;
          }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        u32x4 v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int r = (ln >> 3) + 8 * q;
          v[q] = *reinterpret_cast<const u32x4*>(patch + r * 128 + ((c16 ^ ((r >> 1) & 7)) << 4));
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = it.m0 + wm + 32 * i + (ln >> 3) + 8 * q;
          const unsigned off = (ocol < N) ? (unsigned)(((int64_t)row * ldc + ocol) * 2) : kOob;
          __builtin_amdgcn_raw_buffer_store_b128(v[q], rc, (int)off, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    __syncthreads();               // the patch lives in the stage the next step overwrites
  };
  // Activation variants (forward form, no residual): every row block passes through the patch
  // twice, first the output itself (bias added in fp32, rounded to bf16) on its way to C, then
  // the activation of those rounded values on its way to C2.  The bias descriptor of a null
  // bias is empty and reads zeros.
  auto finish_act = [&](const WorkItem& it, int free_stage) {
    static_assert(ACT == ACT_NONE || TN == 2, "a wave holds two 32-column blocks");
    constexpr bool GU = ACT == ACT_SWIGLU;
    unsigned char* patch = smem + free_stage + wave * 4096;
    // stages of 64-deep K-tiles have room for a table of erf behind the patches (ErfTable; the same bits): 7 erff to
    // fill it where the tile has 64 values a thread
    constexpr bool TABLE = (ACT == ACT_GELU || ACT == ACT_TAPS) && NWM * NWN * 4096 + ErfTable::kEntries * 4 <= STAGE;
    float* const erf_table = reinterpret_cast<float*>(smem + free_stage + NWM * NWN * 4096);
    if constexpr (TABLE) {
      ErfTable::fill(erf_table, threadIdx.x, NT);
      __syncthreads();
    }
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int elr = ln & 31, ehb = ln >> 5;
    const __amdgpu_buffer_rsrc_t rc2 = make_rsrc(aa.C2, aa.c2_bytes);
    // first column in C of the wave's accumulator block 0 and block 1
    const int zc0 = GU ? (it.n0 >> 1) + (wn >> 1) : it.n0 + wn;
    const int zc1 = GU ? zc0 + aa.gu_f : zc0 + 32;
    u32x2 braw[8];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int col = (j ? zc1 : zc0) + 8 * g + 4 * ehb;
        braw[4 * j + g] = __builtin_amdgcn_raw_buffer_load_b64(rbias, col < N ? col * 2 : (int)kOob, 0, 0);
      }
    const int wr = elr * 128 + ehb * 8, wsx = (elr >> 1) & 7;
    const int c16 = ln & 7;
    // column this lane writes back (16 bytes = 8 columns of patch chunk c16), in C and in C2
    const int zcol = c16 < 4 ? zc0 + 8 * c16 : zc1 + 8 * (c16 - 4);
    const int acol = GU ? (c16 < 4 ? zc0 + 8 * c16 : -1) : zcol;
    const int a_n = GU ? aa.gu_f : N;
    // the value stored to C for accumulator register (i, j, 4g+e)
    auto zval = [&](int i, int j, int g, int e) -> float {
      const bf16x4 bv = __builtin_bit_cast(bf16x4, braw[4 * j + g]);
      return (float)(bf16)(acc[i][j][4 * g + e] + (float)bv[e]);
    };
    auto patch_sync = [&]() {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // patch (32 rows of 128 bytes, chunks XOR-swizzled) -> rows of `rsrc`, 8 rows per instruction
    auto drain = [&](int i, __amdgpu_buffer_rsrc_t rsrc, int64_t ld, int col, int ncols, auto second_) {
      constexpr bool TAPS = decltype(second_)::value && ACT == ACT_TAPS;
      u32x4 v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = (ln >> 3) + 8 * q;
        v[q] = *reinterpret_cast<const u32x4*>(patch + r * 128 + ((c16 ^ ((r >> 1) & 7)) << 4));
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = it.m0 + wm + 32 * i + (ln >> 3) + 8 * q;
        const bool in = col >= 0 && col < ncols;
        if constexpr (TAPS) {
          const TapRows t = tap_rows(row, M, N, aa.r_rows, aa.r_magic);
          __builtin_amdgcn_raw_buffer_store_b128(v[q], rsrc, (int)(in && t.first >= 0 ? (unsigned)((t.first + col) * 2) : kOob), 0, 0);
          __builtin_amdgcn_raw_buffer_store_b128(t.zero ? u32x4{0u, 0u, 0u, 0u} : v[q], rsrc, (int)(in && t.second >= 0 ? (unsigned)((t.second + col) * 2) : kOob), 0, 0);
          continue;
        }
        const unsigned off = in ? (unsigned)(((int64_t)row * ld + col) * 2) : kOob;
        __builtin_amdgcn_raw_buffer_store_b128(v[q], rsrc, (int)off, 0, 0);
      }
    };
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = (bf16)zval(i, j, g, e);
          *reinterpret_cast<bf16x4*>(patch + wr + (((4 * j + g) ^ wsx) << 4)) = o;
        }
      patch_sync();
      drain(i, rc, ldc, zcol, N, std::false_type{});
      patch_sync();
      if constexpr (GU) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = (bf16)swiglu_f(zval(i, 0, g, e), zval(i, 1, g, e));
          *reinterpret_cast<bf16x4*>(patch + wr + ((g ^ wsx) << 4)) = o;
        }
      } else {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (bf16)(TABLE ? ErfTable::gelu(erf_table, zval(i, j, g, e)) : gelu_f(zval(i, j, g, e)));
            *reinterpret_cast<bf16x4*>(patch + wr + (((4 * j + g) ^ wsx) << 4)) = o;
          }
      }
      patch_sync();
      drain(i, rc2, aa.ldc2, acol, a_n, std::true_type{});
      patch_sync();
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    __syncthreads();               // the patch lives in the stage the next step overwrites
  };
  // Only the forward form meets a bias without a residual often enough to hold a variant for
  // it; elsewhere such a call takes EPI_RES, whose empty residual descriptor reads zeros.
  constexpr bool BIAS_VARIANT = A_KC && !B_KC;
  const int epi_mode = SPLITK ? EPI_PLAIN : (R != nullptr) ? EPI_RES
                     : (bias != nullptr) ? (BIAS_VARIANT ? EPI_BIAS : EPI_RES) : EPI_PLAIN;
  auto finish = [&](const WorkItem& it, int free_stage) {
    if constexpr (SPLITK) {
      finish_impl(it, free_stage, std::integral_constant<int, EPI_PLAIN>{});
    } else if constexpr (ACT != ACT_NONE) {
      finish_act(it, free_stage);
    } else {
      if (epi_mode == EPI_RES) { finish_impl(it, free_stage, std::integral_constant<int, EPI_RES>{}); return; }
      if constexpr (BIAS_VARIANT) {
        if (epi_mode == EPI_BIAS) { finish_rows(it, free_stage, std::integral_constant<int, EPI_BIAS>{}); return; }
      }
      finish_rows(it, free_stage, std::integral_constant<int, EPI_PLAIN>{});
    }
  };

  int kt = cur.kt0;
  // One pipeline step, straight-line: the K-tile AHEAD of the compute cursor is requested
  // into the stage that was read last step, the current K-tile is multiplied, and before
  // the barrier every wave waits for its own requests of the K-tile two ahead, so that
  // after the barrier that tile is complete for all waves.
  // Written slot by slot: one MFMA, then at most a fragment read and a request, then a
  // scheduling barrier that keeps the compiler from regrouping them.  A wave that is alone
  // on its SIMD has nobody to cover a clump of requests or a wait for a read it has just
  // issued, so every fragment is read a whole batch of MFMAs before its first use and the
  // requests are spread over the first batch.
  // The barrier is the bare instruction.  What it has to order: (1) requests into the
  // stage read in this step are issued in the next step, after every wave has passed this
  // barrier, and all reads of that stage feed MFMAs that precede the barrier in program
  // order (the scheduling barriers keep them there), so those reads have returned;
  // (2) each wave has waited for its own requests of the K-tile two ahead before it
  // arrives, so after the barrier that tile is complete.
  constexpr int NM = TM * TN, NF = TM + TN;
  auto read_frag = [&](bf16x8* fa, bf16x8* fb, int stage, int ks, int r) {
    // fragment order: weight-side block 0, the TM activation-side blocks, the other weight-side blocks
    if (r == 0) fb[0] = frb.read(lds + stage + AREA_A, 0, ks);
    else if (r <= TM) fa[r - 1] = fra.read(lds + stage, r - 1, ks);
    else fb[r - TM] = frb.read(lds + stage + AREA_A, r - TM, ks);
  };
  auto step = [&]() {
    const int rd = stg(0), nx = stg(1), ldst = stg(AHEAD);
    const typename LA::Prep pa = la.prep(lta, lkt, K, lit.kt_end, lit.valid);
    const typename LB::Prep pb = lb.prep(ltb, lkt, K, lit.kt_end, lit.valid);
    const unsigned dsta = lds0 + (unsigned)ldst, dstb = dsta + AREA_A;
    __builtin_amdgcn_sched_barrier(0);
    constexpr int KS = BKT / 16, LSLOTS = NM * KS / 2;       // k-steps; slots of the first half, which make the requests
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      bf16x8* const fc = (ks & 1) ? fa1 : fa0; bf16x8* const gc = (ks & 1) ? fb1 : fb0;     // fragments of this k-step
      bf16x8* const fn = (ks & 1) ? fa0 : fa1; bf16x8* const gn = (ks & 1) ? fb0 : fb1;     // and of the next (of the next K-tile's first)
#pragma unroll
      for (int q = 0; q < NM; ++q) {
        const int i = q % TM, j = q / TM, slot = ks * NM + q;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gc[j], fc[i], acc[i][j], 0, 0, 0);
#pragma unroll
        for (int r = (q * NF + NM - 1) / NM; r < ((q + 1) * NF + NM - 1) / NM; ++r) read_frag(fn, gn, ks + 1 < KS ? rd : nx, ks + 1 < KS ? ks + 1 : 0, r);
        if (slot < LSLOTS) {
#pragma unroll
          for (int l = slot * NLOADS / LSLOTS; l < (slot + 1) * NLOADS / LSLOTS; ++l) {
            if (l < LA::NI) la.issue_j(da, lta, pa, l, dsta);
            else lb.issue_j(db, ltb, pb, l - LA::NI, dstb);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    wait_loads(std::integral_constant<int, 2 * NLOADS>{});
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    si = si + 1 >= NS ? 0 : si + 1;
    ++lkt; ++kt;
  };
  f32x16 sum[CHAINED ? TM : 1][CHAINED ? TN : 1];     // of the finished pieces of the tile
  int piece_end = CHAINED ? ktiles_per : 0;
  while (true) {
    int n = cur.kt_end - kt;
    if (lit.valid) n = min(n, lit.kt_end - lkt);
    if constexpr (CHAINED) n = min(n, piece_end - kt);
    for (; n > 0; --n) step();
    if (lit.valid && lkt >= lit.kt_end) load_cursor_next_item();
    if constexpr (CHAINED) {
      const bool first = piece_end == ktiles_per, last = kt >= cur.kt_end;
      if (kt == piece_end || last) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            if (!first) acc[i][j] = sum[i][j] + acc[i][j];
            if (!last) { sum[i][j] = acc[i][j]; acc[i][j] = f32x16{}; }
          }
        piece_end = last ? ktiles_per : piece_end + ktiles_per;
      }
    }
    if (kt >= cur.kt_end) {
      // an item is claimed under the epilogue when none is drawn ahead
      const bool claim = tq.mode == TQ_QUEUE && !have_drawn && !drained && ahead_ok;
      unsigned entry = 0;
      if (claim && threadIdx.x == 0) entry = tq_claim(tq, qc);
      finish(cur, stg(NS - 1));
      if (claim) {
        int v = -1;
        if (threadIdx.x == 0) { int left = 0; const int it = tq_resolve(tq, qc, entry, &left); v = flagged(it, left); }
        drawn = publish(v);
        have_drawn = drawn >= 0;
      }
      if (lqn == 0) break;         // the load cursor has found the queue empty
      cur = decode(lq_pop());
      kt = cur.kt0;
    }
  }
  wait_loads(std::integral_constant<int, 0>{});
  if (threadIdx.x == 0) tq_leave(tq);
}

template <int BM, int BN, int NWM, int NWN, bool A_KC, bool B_KC, int PIECES, int ACT = ACT_NONE, int BKT = BK>
__global__ __launch_bounds__(64 * NWM * NWN, 2) void gemm_bf16_kernel(
    const bf16* __restrict__ A, const bf16* __restrict__ B, bf16* __restrict__ C,
    const bf16* __restrict__ bias, const bf16* __restrict__ R, int M, int N, int K,
    int64_t lda, int64_t ldb, int64_t ldc, uint32_t a_bytes, uint32_t b_bytes, uint32_t c_bytes,
    int tiles_m, int tiles_n, int tile_begin, int tile_count, int sub, int ksplit, int ktiles_per,
    float* __restrict__ P, TileQueueArgs tq, ActArgs aa) {
  gemm_bf16_body<BM, BN, NWM, NWN, A_KC, B_KC, PIECES, ACT, BKT>(A, B, C, bias, R, M, N, K, lda, ldb, ldc, a_bytes, b_bytes, c_bytes, tiles_m, tiles_n,
                                                                 tile_begin, tile_count, sub, ksplit, ktiles_per, P, tq, aa);
}

// The input gradient and the weight gradient of a linear layer side by side in one launch (pair_plan): the first
// dg.tq.wgs workgroups walk the tiles of the one, the others those of the other, each as gemm_bf16_kernel would.
// Bound by what its longer product is bound by: the LDS of one CU per tile.  Measured, two launches -> one: two encoder
// layers of 1568 rows, width 768, MLP 3072 (eight pairs) 625 -> 537 us; projector 768 -> 2048 of 1568 rows (one pair)
// 132.7 -> 123.7.
struct PairHalf {
  const bf16 *A, *B;
  bf16* C;
  int M, N, K;
  int64_t lda, ldb, ldc;
  uint32_t a_bytes, b_bytes, c_bytes;
  int tiles_m, tiles_n, ktiles_per;
  TileQueueArgs tq;
  ActArgs aa;
};
template <int PIECES>
__global__ __launch_bounds__(256, 2) void gemm_bf16_pair_kernel(PairHalf dg, PairHalf wg) {
  if ((int)blockIdx.x < dg.tq.wgs)
    gemm_bf16_body<128, 128, 2, 2, true, true, PIECES_NONE, ACT_NONE, 64>(dg.A, dg.B, dg.C, nullptr, nullptr, dg.M, dg.N, dg.K, dg.lda, dg.ldb, dg.ldc, dg.a_bytes,
                                                                         dg.b_bytes, dg.c_bytes, dg.tiles_m, dg.tiles_n, 0, dg.tiles_m * dg.tiles_n, 1, 1, 0,
                                                                         nullptr, dg.tq, dg.aa);
  else
    gemm_bf16_body<128, 128, 2, 2, false, false, PIECES, ACT_NONE, 64>(wg.A, wg.B, wg.C, nullptr, nullptr, wg.M, wg.N, wg.K, wg.lda, wg.ldb, wg.ldc, wg.a_bytes,
                                                                      wg.b_bytes, wg.c_bytes, wg.tiles_m, wg.tiles_n, 0, wg.tiles_m * wg.tiles_n, 1, 1,
                                                                      wg.ktiles_per, nullptr, wg.tq, wg.aa);
}

// ------------------------------------------------------------------ four-wave kernel
// 256x256x64 tiles, four waves of 128x128, v_mfma_f32_16x16x32_bf16, for every form whose
// K-contiguous operands have a contraction of whole K-tiles (K a multiple of 64).  Where the row operand is
// K-contiguous the tile may be 32 * MI rows high, MI = 8, 7, 6 or 5 (launch_mfma_shape says when).
//
// What bounds it: on the whole chip the board's power.  Registers only, random data, the
// 16x16x32 instruction delivers 1830 TFLOP/s and the 32x32x16 one 1760 (it reads and writes twice
// the accumulator bytes per flop); around it the kernel spends as little as it can: a wave tile of
// 128x128 reads 1 LDS byte per 64 flops (two thirds of what 128x64 wave tiles read), a K-tile of 64
// brings whole 128-byte lines, operands go HBM -> LDS without passing registers, 128 matrix instructions
// come with about 135 others per K-tile.
//   LDS: two stages of 64 KB.  The fragments of a K-tile's second half are read under its first 16
//     matrix instructions; after a barrier (slot 24 of 128) the stage is free and the K-tile after the
//     next is requested into it, one request per six matrix instructions: requests made faster than
//     the CU's vector cache takes them (16 cycles each, four waves) hold up the wave that makes
//     them.  The next K-tile has to be there, behind a second barrier, at slot 88, when its first
//     fragments are read.  Measured on 32768 x 4096 x 22016 input gradient / 12000 x 5120 x 1280
//     forward: a request per two slots, one barrier in the middle 4697 / 118 us; per four 4734 / 112;
//     two barriers and one per six 3960 / 112; without any requests the K loop takes 20 % less than
//     the first of these.
//   The stream of K-tiles runs on across output tiles; the epilogue passes through 4 KB per
//     wave behind the stages, so the next tile's first K-tiles land under it.
//   K-contiguous operand: rows of 128 bytes, 16-byte chunks XOR-swizzled by (row/2)%8, a fragment is
//     one ds_read_b128.  K-strided operand: k-rows of 512 bytes as in HBM, 32-byte chunks XOR-swizzled
//     by 2*(k%4) + (k/8)%2, a fragment is two ds_read_b64_tr_b16.  Both touch every bank once.
//   Requests take a constant offset per lane; the K-tile moves the descriptor (base and remaining
//     bytes: scalar instructions), which also bounds it: rows past the end read zeros, columns past
//     the end read the next row's values and only reach outputs that are not stored.
//   The matrix instruction is written in assembly to tie the result to its accumulator: left to
//     itself the compiler copied 400 accumulator registers per K-tile.
// Each output element is accumulated in ascending k: same bits as gemm_bf16_kernel's.
// Measured, whole device, eight-wave kernel (input gradient: a four-wave kernel that staged through
// registers) -> this: forward 32768 x 4096 x 12288 2525 -> 2300 us (1434 TFLOP/s), 8192 x 5632 x 2048
// 149 -> 129; with GELU 12000 x 1280 x 5120 199 -> 151, with SwiGLU 8192 x 2048 x 11264 365 -> 338;
// input gradient 32768 x 4096 x 22016 4433 -> 3960 (1492 TFLOP/s), 9216 x 4096 x 1024 77 -> 70;
// weight gradient 4096 x 32768 x 22016 4268 -> 4000, 2048 x 8192 x 11264 339 -> 331.
struct W4Args {
  const bf16 *A, *B, *bias, *R;
  bf16 *C, *C2;
  int M, N, K;
  int64_t lda, ldb, ldc, ldc2;
  uint32_t a_bytes, b_bytes, c_bytes, c2_bytes;
  int tiles_m, tiles_n, tile_begin, tile_count, row_block, gu_f;
  uint32_t r_rows, r_magic;        // W4_TABLE, W4_TAPS: see ActArgs
};
enum { W4_PLAIN, W4_BIAS, W4_RES, W4_GELU, W4_SWIGLU, W4_TABLE, W4_TAPS };
constexpr int kW4Stage = 2 * 256 * 64 * 2;                         // both operands of a K-tile
constexpr int kW4Pitch = 68;                                       // floats per row of the epilogue's patch: 16 rows of 64
constexpr int kW4Patch = 4 * 16 * kW4Pitch * 4;
constexpr int w4_lds(int epi) { return 2 * kW4Stage + kW4Patch + (epi == W4_GELU || epi == W4_TAPS ? ErfTable::kEntries * 4 : 0); }

// One operand: what a lane requests of a K-tile, and where its fragments are.
template <bool KC, bool GU, int NF = 8>
struct W4Operand {
  unsigned voff[NF];                       // byte offset of request j from the K-tile's first byte
  int frag[KC ? 2 : 8];                    // LDS offsets: KC: of k-half 0 / 1, + 2048 per 16 rows; else of 16 columns each, + 16384 per k-half
  __device__ __forceinline__ void init(int wave, int w0, int64_t ld, int gu_f) {
    const int lane = threadIdx.x & 63, lr = lane & 15, g = lane >> 4;
#pragma unroll
    for (int j = 0; j < NF; ++j) {
      if constexpr (KC) {
        const int r = 8 * NF * wave + 8 * j + (lane >> 3), ch = (lane & 7) ^ ((r >> 1) & 7);
        voff[j] = (unsigned)((int64_t)r * ld * 2 + ch * 16);
      } else {
        const int kr = 16 * wave + 2 * j + (lane >> 5), pos = lane & 31;
        const int c32 = (pos >> 1) ^ (((kr & 3) << 1) | ((kr >> 3) & 1));
        // GU: 16-column group c32 of the tile belongs to the gate half (even) or the up half (odd)
        const int64_t byte = GU ? (c32 >> 1) * 32 + (int64_t)(c32 & 1) * gu_f * 2 : c32 * 32;
        voff[j] = (unsigned)((int64_t)kr * ld * 2 + byte + (pos & 1) * 16);
      }
    }
    if constexpr (KC) {
      const int sw = (lr >> 1) & 7;
      frag[0] = (w0 + lr) * 128 + ((g ^ sw) << 4);
      frag[1] = (w0 + lr) * 128 + (((4 + g) ^ sw) << 4);
    } else {
      const int q = lr >> 2, f = (q << 1) | (g & 1);
#pragma unroll
      for (int i = 0; i < 8; ++i) frag[i] = (8 * g + q) * 512 + (((w0 >> 4) + (i ^ f)) << 5) + 8 * (lr & 3);
    }
  }
  __device__ __forceinline__ u32x4 read(const lds_byte* area, int i, int half) const {
    if constexpr (KC) {
      return *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(area + frag[half] + 2048 * i);
    } else {
      const lds_byte* p = area + frag[i] + 16384 * half;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p + 2048));
      typedef __attribute__((ext_vector_type(8))) short s16x8;
      return __builtin_bit_cast(u32x4, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  }
};

// Where an operand's next K-tile starts and how many bytes of the tensor lie behind that point.
struct W4Cursor {
  uint64_t at;
  uint32_t left;
  __device__ __forceinline__ void set(const void* base, uint64_t off, uint32_t bytes) {
    at = (uint64_t)(uintptr_t)base + off;
    left = off < bytes ? (uint32_t)(bytes - off) : 0u;
  }
  __device__ __forceinline__ void advance(uint32_t step) { at += step; left = left > step ? left - step : 0u; }
  __device__ __forceinline__ i32x4 desc(bool live) const {
    i32x4 d;
    d.x = __builtin_amdgcn_readfirstlane((int)(uint32_t)at); d.y = __builtin_amdgcn_readfirstlane((int)((uint32_t)(at >> 32) & 0xffffu));
    d.z = __builtin_amdgcn_readfirstlane((int)(live ? left : 0u)); d.w = 0x00020000;
    return d;
  }
};

template <bool A_KC, bool B_KC, int EPI, int MI>
__global__ __launch_bounds__(256, 1) void gemm_bf16_w4_kernel(W4Args p, TileQueueArgs tq) {
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  constexpr int OPB = kW4Stage / 2;
  static_assert(MI == 8 || A_KC, "a K-strided row operand fills whole requests with 256 rows only");
  extern __shared__ __align__(16) unsigned char smem[];
  lds_byte* const lds = (lds_byte*)smem;
  const unsigned lds0 = (unsigned)(uintptr_t)lds;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = (wave >> 1) * (16 * MI), wn = (wave & 1) * 128;
  const int nk = (p.K + 63) / 64;              // at least two, the depth of the request stream
  const uint32_t astep = A_KC ? 128u : (uint32_t)(64 * p.lda * 2), bstep = B_KC ? 128u : (uint32_t)(64 * p.ldb * 2);
  W4Operand<A_KC, false, MI> oa;
  W4Operand<B_KC, EPI == W4_SWIGLU> ob;
  oa.init(wave, wm, p.lda, 0);
  ob.init(wave, wn, p.ldb, p.gu_f);

  struct Item { int m0, n0; };
  auto decode = [&](int item) -> Item {
    int trow, tcol;
    tile_coords(p.tile_begin + item, p.tiles_m, p.tiles_n, p.row_block, &trow, &tcol);
    return {trow * (32 * MI), tcol * 256};
  };
  W4Cursor ca, cb;
  auto point = [&](const Item& it) {
    ca.set(p.A, A_KC ? (uint64_t)it.m0 * p.lda * 2 : (uint64_t)it.m0 * 2, p.a_bytes);
    cb.set(p.B, B_KC ? (uint64_t)it.n0 * p.ldb * 2 : (uint64_t)(EPI == W4_SWIGLU ? it.n0 : it.n0 * 2), p.b_bytes);
  };
  const unsigned wdst = lds0 + (unsigned)wave * 8192, adst = lds0 + (unsigned)wave * (MI * 1024);
  auto request = [&](const i32x4& d, unsigned off, unsigned dst) {
    // m0 = LDS address of lane 0's 16 bytes; lane l lands at m0 + 16*l.  Completion is waited for by hand.
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" : : "s"(dst), "v"(off), "s"(d) : "m0");
  };
  auto request_tile = [&](int st) {
    i32x4 da = ca.desc(true), db = cb.desc(true);
    // A memory instruction may read a scalar register that the vector unit wrote (v_readfirstlane) five wait
    // states later at the earliest, and the compiler does not see the requests: both descriptors
    // pass through these five, so that no part of them is formed later.
    asm volatile("s_nop 4" : "+s"(da), "+s"(db));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < MI; ++j) request(da, oa.voff[j], adst + (unsigned)(st * kW4Stage + j * 1024));
#pragma unroll
    for (int j = 0; j < 8; ++j) request(db, ob.voff[j], wdst + (unsigned)(st * kW4Stage + OPB + j * 1024));
    ca.advance(astep);
    cb.advance(bstep);
  };

  __shared__ int mail;
  TileQueueCursor qc;
  int item = tq_first(tq, qc, &mail);
  if (item < 0) { tq_done(tq); return; }
  Item it = decode(item);
  point(it);
  request_tile(0);
  request_tile(1);
  // 256 values of a tile to a thread: seven erff to fill the table instead of 256 (the epilogue of 12000 x 1280 x 5120
  // takes 10 us of 150; with erff in it, four waves a CU, 83 of 239)
  float* const erf_table = reinterpret_cast<float*>(smem + 2 * kW4Stage + kW4Patch);
  if constexpr (EPI == W4_GELU || EPI == W4_TAPS) {
    ErfTable::fill(erf_table, threadIdx.x, 256);
    __syncthreads();
  }
  f32x4 acc[MI][8];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  u32x4 ax[MI], bx[8], ay[MI], by[8];          // fragments of the first and of the second half
  __builtin_amdgcn_s_waitcnt(((MI + 8) & 15) | (7 << 4) | (15 << 8) | (((MI + 8) >> 4) << 14));      // vmcnt: the first K-tile has landed
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    if (i < MI) ax[i] = oa.read(lds, i, 0);
    bx[i] = ob.read(lds + OPB, i, 0);
  }
  int st = 0;
  bool live = true;
  auto mfma = [](f32x4& c, const u32x4& b, const u32x4& a) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(b), "v"(a));
  };
  // The compiler knows nothing of the latency of an assembly instruction: this stands between the
  // matrix instructions and other reads or writes of their registers (more than the 19 wait
  // states that the longest of those dependencies wants).
  auto settle = [] { asm volatile("s_nop 15\n\ts_nop 15"); __builtin_amdgcn_sched_barrier(0); };
  // One K-tile: 128 slots of one matrix instruction, the rest placed between them (see above).
  constexpr int NR = MI + 8;                  // requests of a K-tile, fragments of half of it
  constexpr int kFree = NR + 8, kLanded = 16 * MI - 2 * NR - 8, kRequest = kFree + 1, kEvery = MI == 8 ? 6 : MI - 1;
  constexpr int kBefore = (kLanded - kRequest + kEvery - 1) / kEvery;        // requests made before kLanded
  static_assert(kFree <= 8 * MI && kLanded >= 8 * MI && kRequest + (NR - 1) * kEvery < 16 * MI, "slots of a K-tile");
  auto step = [&]() {
    const lds_byte* const here = lds + st * kW4Stage;
    const lds_byte* const there = lds + (st ^ 1) * kW4Stage;
    // formed here, ahead of the scheduling barrier, and first read kRequest matrix instructions on: far beyond the
    // five wait states that request_tile waits out
    const i32x4 da = ca.desc(live), db = cb.desc(live);
    const unsigned dst = wdst + (unsigned)(st * kW4Stage), dsta = adst + (unsigned)(st * kW4Stage);
    __builtin_amdgcn_sched_barrier(0);
    auto half = [&](auto first) {
      constexpr int t0 = decltype(first)::value;
#pragma unroll
      for (int q = 0; q < 8 * MI; ++q) {
        const int t = t0 + q, i = q % MI, j = q / MI;
        if constexpr (t0 == 0) mfma(acc[i][j], bx[j], ax[i]);
        else mfma(acc[i][j], by[j], ay[i]);
        if (t < MI) ay[t] = oa.read(here, t, 1);
        else if (t < NR) by[t - MI] = ob.read(here + OPB, t - MI, 1);
        if (t == kFree) {
          __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));                                       // lgkmcnt(0)
          __builtin_amdgcn_s_barrier();
        }
        if (t == kLanded) {
          __builtin_amdgcn_s_waitcnt((kBefore & 15) | (7 << 4) | (15 << 8) | ((kBefore >> 4) << 14));             // vmcnt(kBefore)
          __builtin_amdgcn_s_barrier();
        }
        if (t >= kRequest && (t - kRequest) % kEvery == 0 && (t - kRequest) / kEvery < NR) {
          const int r = (t - kRequest) / kEvery;
          if (r < MI) request(da, oa.voff[r], dsta + (unsigned)(r * 1024));
          else request(db, ob.voff[r - MI], dst + (unsigned)(OPB + (r - MI) * 1024));
        }
        if (t >= kLanded && (t - kLanded) % 2 == 0 && t < kLanded + 2 * NR) {
          const int r = (t - kLanded) / 2;
          if (r < MI) ax[r] = oa.read(there, r, 0);
          else bx[r - MI] = ob.read(there + OPB, r - MI, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    half(std::integral_constant<int, 0>{});
    half(std::integral_constant<int, 8 * MI>{});
    ca.advance(astep);
    cb.advance(bstep);
    st ^= 1;
  };
  const __amdgpu_buffer_rsrc_t rc = make_rsrc(p.C, p.c_bytes), rc2 = make_rsrc(p.C2, p.C2 ? p.c2_bytes : 0u);
  const __amdgpu_buffer_rsrc_t rr = make_rsrc(p.R, !p.R ? 0u : EPI == W4_TABLE ? (uint32_t)(p.r_rows * p.ldc * 2) : p.c_bytes), rbias = make_rsrc(p.bias, p.bias ? (uint32_t)p.N * 2u : 0u);
  while (true) {
    settle();
    for (int n = nk - 2; n > 0; --n) step();
    // the last K-tile of this item has been requested: the requests move on to the next item
    const unsigned entry = tq_claim_ahead(tq, qc);
    const int next = tq_next(tq, qc, entry, &mail);
    live = next >= 0;
    const Item nit = decode(live ? next : item);
    point(nit);
    for (int n = 2; n > 0; --n) step();
    settle();
    // Epilogue, 16 rows x 64 columns at a time through the patch, leaving row-contiguous.
    // acc[i][j][e] is output (row m0+wm+16i+lr, column n0+wn+16j+4g+e).
    {
      float* const patch = reinterpret_cast<float*>(smem + 2 * kW4Stage) + wave * (16 * kW4Pitch);
      int ln = lane;
      asm volatile("" : "+v"(ln));           // write-back offsets are formed here, not kept across the K loop
      const int elr = ln & 15, eg = ln >> 4;
      constexpr bool GU = EPI == W4_SWIGLU;
      // a lane writes 8 columns: of rows prow and prow + 8, or (SwiGLU) of gate, up and activation of row prow
      const int prow = GU ? ln >> 2 : ln >> 3, pcol = GU ? 32 * ((ln >> 1) & 1) + 8 * (ln & 1) : 8 * (ln & 7);
      auto out_col = [&](int h) { return GU ? (it.n0 >> 1) + ((wn + 64 * h) >> 1) + (pcol >> 5) * 16 + (pcol & 15) : it.n0 + wn + 64 * h + pcol; };
      const int ncols = GU ? p.gu_f : p.N;
      auto off = [&](int row, int col, int64_t ld, bool ok) -> int { return ok ? (int)(unsigned)(((int64_t)row * ld + col) * 2) : (int)kOob; };
      u32x4 bias_[2] = {}, bias_up[2] = {};
      if constexpr (EPI != W4_PLAIN) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int col = out_col(h);
          bias_[h] = __builtin_amdgcn_raw_buffer_load_b128(rbias, col < ncols ? col * 2 : (int)kOob, 0, 0);
          if constexpr (GU) bias_up[h] = __builtin_amdgcn_raw_buffer_load_b128(rbias, col < ncols ? (col + p.gu_f) * 2 : (int)kOob, 0, 0);
        }
      }
      auto patch_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      };
      // What is added to block b, requested RAHEAD blocks before: one block's stores and its way through the patch take less than the latency of
      // memory (a table of positions comes from the caches).  Forward with a residual, requested in its own block -> three ahead: 32768 x 4096 x 4096
      // 863 -> 822 us, 32768 x 11008 x 4096 2091 -> 2056, 12000 x 5120 x 1280 120.2 -> 117.3, 9216 x 1024 x 1024 24.4 -> 23.8.
      constexpr bool HAS_R = EPI == W4_RES || EPI == W4_TABLE;
      constexpr int RAHEAD = EPI == W4_RES ? 3 : EPI == W4_TABLE ? 1 : 0;
      u32x4 ring[RAHEAD + 1][2] = {};
      auto request_res = [&](int b) {
        const int col = out_col(b & 1);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int row = it.m0 + wm + 16 * (b >> 1) + prow + 8 * q;
          ring[b % (RAHEAD + 1)][q] = __builtin_amdgcn_raw_buffer_load_b128(rr, off(EPI == W4_TABLE ? table_row(row, p.r_rows, p.r_magic) : row, col, p.ldc, col < ncols), 0, 0);
        }
      };
      if constexpr (HAS_R) {
#pragma unroll
        for (int b = 0; b < RAHEAD; ++b) request_res(b);
      }
#pragma unroll
      for (int b = 0; b < 2 * MI; ++b) {
        const int i = b >> 1, h = b & 1, row0 = it.m0 + wm + 16 * i, col = out_col(h);
        const bool ok = col < ncols;
        if constexpr (HAS_R) if (b + RAHEAD < 2 * MI) request_res(b + RAHEAD);
        const u32x4* const res = ring[b % (RAHEAD + 1)];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          f32x4& a = acc[i][4 * h + jj];
          *reinterpret_cast<float4*>(patch + elr * kW4Pitch + 16 * jj + 4 * eg) = make_float4(a[0], a[1], a[2], a[3]);
          a = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        patch_sync();
        auto row8 = [&](int r, int c, float* v) {
          const float4 x = *reinterpret_cast<const float4*>(patch + r * kW4Pitch + c), y = *reinterpret_cast<const float4*>(patch + r * kW4Pitch + c + 4);
          v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w; v[4] = y.x; v[5] = y.y; v[6] = y.z; v[7] = y.w;
        };
        if constexpr (GU) {
          float gv[8], uv[8];
          row8(prow, pcol, gv);
          row8(prow, pcol + 16, uv);
          const bf16x8 bg = __builtin_bit_cast(bf16x8, bias_[h]), bu = __builtin_bit_cast(bf16x8, bias_up[h]);
          bf16x8 og, ou, oc;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            og[e] = (bf16)(gv[e] + (float)bg[e]);
            ou[e] = (bf16)(uv[e] + (float)bu[e]);
            oc[e] = (bf16)swiglu_f((float)og[e], (float)ou[e]);     // of the values as stored
          }
          const int row = row0 + prow;
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, og), rc, off(row, col, p.ldc, ok), 0, 0);
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, ou), rc, off(row, col + p.gu_f, p.ldc, ok), 0, 0);
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, oc), rc2, off(row, col, p.ldc2, ok), 0, 0);
        } else {
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int row = row0 + prow + 8 * q;
            float v[8];
            row8(prow + 8 * q, pcol, v);
            const bf16x8 bv = __builtin_bit_cast(bf16x8, bias_[h]), rv = __builtin_bit_cast(bf16x8, res[q]);
            bf16x8 o;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              float x = v[e];
              if constexpr (EPI != W4_PLAIN) x += (float)bv[e];
              if constexpr (EPI == W4_RES || EPI == W4_TABLE) x += (float)rv[e];
              o[e] = (bf16)x;
            }
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), rc, off(row, col, p.ldc, ok), 0, 0);
            if constexpr (EPI == W4_GELU || EPI == W4_TAPS) {
              bf16x8 a2;
#pragma unroll
              for (int e = 0; e < 8; ++e) a2[e] = (bf16)ErfTable::gelu(erf_table, (float)o[e]);     // of the value as stored
              const u32x4 av = __builtin_bit_cast(u32x4, a2);
              if constexpr (EPI == W4_TAPS) {
                const TapRows t = tap_rows(row, p.M, p.N, p.r_rows, p.r_magic);
                __builtin_amdgcn_raw_buffer_store_b128(av, rc2, ok && t.first >= 0 ? (int)(unsigned)((t.first + col) * 2) : (int)kOob, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b128(t.zero ? u32x4{0u, 0u, 0u, 0u} : av, rc2, ok && t.second >= 0 ? (int)(unsigned)((t.second + col) * 2) : (int)kOob, 0, 0);
              } else {
                __builtin_amdgcn_raw_buffer_store_b128(av, rc2, off(row, col, p.ldc2, ok), 0, 0);
              }
            }
          }
        }
        patch_sync();
      }
    }
    if (!live) break;
    item = next;
    it = nit;
  }
  __builtin_amdgcn_s_waitcnt(0);
  tq_done(tq);
}

// out = bf16( P[0] + P[1] + ... ) in ascending piece order, for the tiles [tile_begin,
// tile_begin + tile_count) of the TE x TE tile list that the split launch covered.  One block
// iteration takes 256 float4 of one tile (1024 / TE rows), so the tile's place is found once per
// iteration.  Four pieces are requested together.
template <int TE>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ P, bf16* __restrict__ C,
                                                            int M, int N, int64_t ldc, int ksplit, int tiles_m,
                                                            int tiles_n, int tile_begin, int tile_count, int row_block) {
  constexpr int ROWS = 1024 / TE, PER = TE / ROWS;      // rows of an iteration, iterations of a tile
  const int64_t piece = (int64_t)tile_count * (TE * TE);
  const int units = tile_count * PER;
  for (int u = blockIdx.x; u < units; u += gridDim.x) {
    const int tl = u / PER;
    int trow, tcol;
    tile_coords(tile_begin + tl, tiles_m, tiles_n, row_block, &trow, &tcol);
    const int r = (u % PER) * ROWS + threadIdx.x / (TE / 4), c = (threadIdx.x % (TE / 4)) * 4;
    const int row = trow * TE + r, col = tcol * TE + c;
    if (row >= M || col >= N) continue;
    const float* src = P + (int64_t)tl * (TE * TE) + r * TE + c;
    float4 a = *reinterpret_cast<const float4*>(src);
    int s = 1;
    for (; s + 4 <= ksplit; s += 4) {
      float4 b[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) b[q] = *reinterpret_cast<const float4*>(src + (s + q) * piece);
#pragma unroll
      for (int q = 0; q < 4; ++q) { a.x += b[q].x; a.y += b[q].y; a.z += b[q].z; a.w += b[q].w; }
    }
    for (; s < ksplit; ++s) {
      const float4 b = *reinterpret_cast<const float4*>(src + s * piece);
      a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
    }
    bf16x4 o;
    o[0] = (bf16)a.x; o[1] = (bf16)a.y; o[2] = (bf16)a.z; o[3] = (bf16)a.w;
    *reinterpret_cast<bf16x4*>(C + (int64_t)row * ldc + col) = o;
  }
}

// One launch of the MFMA kernel over coarse tiles [tile_begin, tile_begin + tile_count) of the
// panel-major list of (sub*BM) x (sub*BN) tiles; tile_count < 0 means all of them.
// kper: k-values of a piece (PIECES), whole K-tiles of 32.
template <int BM, int BN, int NWM, int NWN, bool A_KC, bool B_KC, int PIECES = PIECES_NONE, int ACT = ACT_NONE, int BKT = BK>
mosaic_status launch_mfma(hipStream_t s, int quota, int M, int N, int K, const bf16* A, int64_t lda,
                          const bf16* B, int64_t ldb, bf16* C, int64_t ldc, const bf16* bias, const bf16* R,
                          uint32_t a_bytes, uint32_t b_bytes, uint32_t c_bytes, int ksplit = 1,
                          int kper = 0, float* P = nullptr, int sub = 1, int tile_begin = 0,
                          int tile_count = -1, const ActArgs& aa = ActArgs()) {
  // 128x128 tiles that all get a CU to themselves take 64-deep K-tiles: the five stages then fill
  // the LDS (two workgroups per CU would not fit), K-contiguous operands come in whole 128-byte
  // lines and there are half as many barriers.  Such a tile is bound by its CU's LDS (768 cycles
  // of fragment reads and direct-to-LDS writes per 64 k-values against 512 of matrix work).
  // Measured, 32 -> 64 deep: input gradient 1568 x 3072 x 768 27.8 -> 23.1 us, forward 26.9 -> 22.6,
  // weight gradient 768 x 1568 x 768 15.5 -> 14.1.  With more tiles than CUs two workgroups of
  // 32-deep tiles share a CU and cover each other's waits.  The order of the sum is the same.
  if constexpr (BM == 128 && BKT == BK) {
    const int64_t it = (tile_count < 0 ? ceil_div(M, BM * sub) * ceil_div(N, BN * sub) - tile_begin : tile_count) * sub * sub * (PIECES == PIECES_APART ? ksplit : 1);
    if (it <= tile_queue_sure_cus(quota) && (PIECES == PIECES_NONE || kper % 64 == 0))
      return launch_mfma<BM, BN, NWM, NWN, A_KC, B_KC, PIECES, ACT, 64>(s, quota, M, N, K, A, lda, B, ldb, C, ldc, bias, R, a_bytes, b_bytes, c_bytes,
                                                                      ksplit, kper, P, sub, tile_begin, tile_count, aa);
  }
  constexpr size_t smem = (size_t)NS * (BM + BN) * BKT * 2;
  auto kern = gemm_bf16_kernel<BM, BN, NWM, NWN, A_KC, B_KC, PIECES, ACT, BKT>;
  static std::once_flag attr_once;   // per instantiation; launches come from several host threads
  static hipError_t attr_rc = hipSuccess;
  std::call_once(attr_once, [&] {
    attr_rc = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  });
  MOSAIC_HIP(attr_rc);
  const int tiles_m = (int)ceil_div(M, BM * sub), tiles_n = (int)ceil_div(N, BN * sub);
  if (tile_count < 0) tile_count = tiles_m * tiles_n - tile_begin;
  if (tile_count <= 0) return MOSAIC_OK;
  const int wg_per_cu = (BM == 256 || BKT == 64) ? 1 : 2;
  if constexpr (PIECES != PIECES_APART) ksplit = 1;
  const int64_t items = (int64_t)tile_count * sub * sub * ksplit;
  if (items > INT32_MAX) MOSAIC_FAIL(MOSAIC_EUNSUPPORTED, "too many output tiles");
  TileQueueArgs tq;
  int grid;
  MOSAIC_TRY(tile_queue_plan(s, quota, wg_per_cu, items, 0, false, &tq, &grid));
  ActArgs ka = aa;
  // coarse tile rows are BM * sub rows high; every launch over one product (whole rounds,
  // quarter tiles, split tiles) walks the same tile list
  ka.row_block = row_block_for(K, M, BM * sub);
  kern<<<grid, 64 * NWM * NWN, smem, s>>>(A, B, C, bias, R, M, N, K, lda, ldb, ldc, a_bytes, b_bytes, c_bytes,
                                          tiles_m, tiles_n, tile_begin, tile_count, sub, ksplit, kper / BKT, P, tq, ka);
  MOSAIC_LAUNCH_CHECK();
  if constexpr (PIECES == PIECES_APART) {
    static_assert(BM == BN, "the reduce kernel walks square tiles");
    const int g2 = grid_for(quota, 8, (int64_t)tile_count * (BM * BM / 1024));
    splitk_reduce_kernel<BM><<<g2, 256, 0, s>>>(P, C, M, N, ldc, ksplit, tiles_m, tiles_n, tile_begin, tile_count, ka.row_block);
    MOSAIC_LAUNCH_CHECK();
  }
  return MOSAIC_OK;
}

// The four-wave kernel takes a product when its K-contiguous operands are whole K-tiles long.
template <bool A_KC, bool B_KC> constexpr bool w4_form() { return A_KC || !B_KC; }
template <bool A_KC, bool B_KC> bool w4_takes(int64_t K) { return w4_form<A_KC, B_KC>() && K >= 128 && (!(A_KC || B_KC) || K % 64 == 0); }

template <bool A_KC, bool B_KC, int EPI, int MI = 8>
mosaic_status launch_w4_epi(hipStream_t s, int quota, const W4Args& p) {
  auto kern = gemm_bf16_w4_kernel<A_KC, B_KC, EPI, MI>;
  static std::once_flag attr_once;
  static hipError_t attr_rc = hipSuccess;
  std::call_once(attr_once, [&] {
    attr_rc = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, w4_lds(EPI));
  });
  MOSAIC_HIP(attr_rc);
  TileQueueArgs tq;
  int grid;
  MOSAIC_TRY(tile_queue_plan(s, quota, 1, p.tile_count, 0, false, &tq, &grid));
  kern<<<grid, 256, w4_lds(EPI), s>>>(p, tq);
  MOSAIC_LAUNCH_CHECK();
  return MOSAIC_OK;
}

// Tiles [tile_begin, tile_begin + tile_count) of the 256x256 tile list (tile_count < 0: all from
// tile_begin on).  MI < 8: tiles of 32 * MI rows, the whole list.
template <bool A_KC, bool B_KC, int MI = 8>
mosaic_status launch_w4(hipStream_t s, int quota, int M, int N, int K, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, bf16* C,
                        int64_t ldc, const bf16* bias, const bf16* R, uint32_t a_bytes, uint32_t b_bytes, uint32_t c_bytes, int tile_begin,
                        int tile_count, const ActArgs& aa) {
  W4Args p = {};
  p.A = A; p.B = B; p.C = C; p.bias = bias; p.R = R; p.C2 = aa.C2;
  p.M = M; p.N = N; p.K = K; p.lda = lda; p.ldb = ldb; p.ldc = ldc; p.ldc2 = aa.ldc2;
  p.a_bytes = a_bytes; p.b_bytes = b_bytes; p.c_bytes = c_bytes; p.c2_bytes = aa.c2_bytes; p.gu_f = aa.gu_f; p.r_rows = aa.r_rows; p.r_magic = aa.r_magic;
  p.tiles_m = (int)ceil_div(M, 32 * MI); p.tiles_n = (int)ceil_div(N, 256);
  p.tile_begin = tile_begin;
  p.tile_count = tile_count < 0 ? p.tiles_m * p.tiles_n - tile_begin : tile_count;
  if (p.tile_count <= 0) return MOSAIC_OK;
  p.row_block = row_block_for(K, M, 32 * MI);
  if constexpr (A_KC && !B_KC) {
    if (aa.act == ACT_GELU) return launch_w4_epi<A_KC, B_KC, W4_GELU, MI>(s, quota, p);
    if (aa.act == ACT_TAPS) return launch_w4_epi<A_KC, B_KC, W4_TAPS, MI>(s, quota, p);
    if (aa.act == ACT_SWIGLU) return launch_w4_epi<A_KC, B_KC, W4_SWIGLU, MI>(s, quota, p);
    if (bias && !R) return launch_w4_epi<A_KC, B_KC, W4_BIAS, MI>(s, quota, p);
    if (R && aa.r_rows) return launch_w4_epi<A_KC, B_KC, W4_TABLE, MI>(s, quota, p);
  }
  if (R || bias) return launch_w4_epi<A_KC, B_KC, W4_RES, MI>(s, quota, p);
  return launch_w4_epi<A_KC, B_KC, W4_PLAIN, MI>(s, quota, p);
}

// A/B switches for kernel timing, compiled in only with -DMOSAIC_TUNING (never in the library
// that ships): MOSAIC_GEMM_W4=0 sends the 256x256 tiles back to the eight-wave kernel,
// MOSAIC_GEMM_TILE=256 / 128 / 1 forces the all-256, all-128 or mixed tile plan, 7 / 6 / 5 tiles of
// 224 / 192 / 160 rows (the bits are the same either way); MOSAIC_SPLITK=n forces the piece count of a weight gradient's cut tail
// (0: no cut; the bits differ with n); MOSAIC_PIECES=1 / 2 / 3 forces 256x256 tiles, 128x128 tiles or 128x128 tiles one piece
// after the other where all tiles are cut; MOSAIC_PAIR=0 makes two launches of every linear layer's backward pass.
#ifdef MOSAIC_TUNING
bool w4_enabled() { const char* e = getenv("MOSAIC_GEMM_W4"); return !e || atoi(e) != 0; }
int forced_tile() { const char* e = getenv("MOSAIC_GEMM_TILE"); return e ? atoi(e) : 0; }
int forced_pieces() { const char* e = getenv("MOSAIC_PIECES"); return e ? atoi(e) : 0; }
bool pair_enabled() { const char* e = getenv("MOSAIC_PAIR"); return !e || atoi(e) != 0; }
#else
constexpr bool w4_enabled() { return true; }
constexpr int forced_tile() { return 0; }
constexpr int forced_pieces() { return 0; }
constexpr bool pair_enabled() { return true; }
#endif

// dW[M,N] = A^T B, contraction K over the tokens (gemm_plan.h says in which tiles and pieces)
mosaic_status launch_wgrad(hipStream_t s, int quota, int M, int N, int K, const bf16* A, int64_t lda, const bf16* B, int64_t ldb, bf16* C,
                           int64_t ldc, const bf16* bias, const bf16* R, uint32_t a_bytes, uint32_t b_bytes, uint32_t c_bytes, float* scratch) {
  const int cus = tile_queue_sure_cus(quota);
  const bool w4 = w4_takes<false, false>(K) && w4_enabled();
  WgradPlan p = wgrad_plan(M, N, K, cus, scratch && !bias && !R, w4);
  const int t256 = (int)(ceil_div(M, 256) * ceil_div(N, 256));
  typedef std::integral_constant<int, PIECES_NONE> None;
  typedef std::integral_constant<int, PIECES_APART> Apart;
  typedef std::integral_constant<int, PIECES_CHAINED> Chained;
  auto large8 = [&](auto how, int tile_begin, int tile_count) {
    return launch_mfma<256, 256, 2, 4, false, false, decltype(how)::value>(s, quota, M, N, K, A, lda, B, ldb, C, ldc, bias, R, a_bytes, b_bytes, c_bytes,
                                                                           p.pieces, p.kper, scratch, 1, tile_begin, tile_count);
  };
  auto small = [&](auto how, int sub, int tile_begin, int tile_count) {
    return launch_mfma<128, 128, 2, 2, false, false, decltype(how)::value>(s, quota, M, N, K, A, lda, B, ldb, C, ldc, bias, R, a_bytes, b_bytes, c_bytes,
                                                                           p.pieces, p.kper, scratch, sub, tile_begin, tile_count);
  };
  const bool part = p.pieces > 1 && p.first > 0;
  const int tiles = part ? p.first : t256, head = tiles / cus * cus;
  if (p.way <= kPiecesChained) {
    if (forced_pieces() > 0) p.way = (WgradWay)(forced_pieces() - 1);
  } else {
    if (forced_tile() == 256) p.way = w4 ? kWhole4 : kWhole8;
    if (forced_tile() == 128) p.way = kWholeSmall;
    if (forced_tile() == 1 && head > 0 && head < tiles) p.way = w4 ? kMixed4 : kMixed8;
  }
  auto large4 = [&](int count) {
    return launch_w4<false, false>(s, quota, M, N, K, A, lda, B, ldb, C, ldc, bias, R, a_bytes, b_bytes, c_bytes, 0, count, ActArgs());
  };
  switch (p.way) {
    case kPiecesLarge: return large8(Apart(), 0, -1);
    case kPiecesSmall: return small(Apart(), 1, 0, -1);
    case kPiecesChained: return small(Chained(), 1, 0, -1);
    case kWhole8: MOSAIC_TRY(large8(None(), 0, tiles)); break;
    case kWhole4: MOSAIC_TRY(large4(tiles)); break;
    case kWholeSmall: MOSAIC_TRY(part ? small(None(), 2, 0, tiles) : small(None(), 1, 0, -1)); break;
    default:
      MOSAIC_TRY(p.way == kMixed8 ? large8(None(), 0, head) : large4(head));
      MOSAIC_TRY(small(None(), 2, head, tiles - head));
  }
  return part ? large8(Apart(), tiles, t256 - tiles) : MOSAIC_OK;
}

template <bool A_KC, bool B_KC>
mosaic_status launch_mfma_shape(hipStream_t s, int quota, int M, int N, int K, const bf16* A, int64_t lda,
                                const bf16* B, int64_t ldb, bf16* C, int64_t ldc, const bf16* bias, const bf16* R,
                                uint32_t a_bytes, uint32_t b_bytes, uint32_t c_bytes, const ActArgs& aa = ActArgs()) {
  static_assert(A_KC || B_KC, "launch_wgrad takes the K-strided form");
  const int64_t t256 = ceil_div(M, 256) * ceil_div(N, 256);
  // Tile shape only decides which workgroup computes an element, never its bits.  Large
  // tiles halve LDS traffic per MFMA; small tiles fill the CUs when there are few large
  // ones.  Plans, priced in units of a quarter of a 256x256 tile's time on one CU (eight-wave kernel):
  //   all-256: whole rounds of 256x256 tiles, the last one possibly mostly idle;
  //   all-128: 128x128 tiles, two workgroups per CU;
  //   mixed:   the whole rounds with the large kernel, then the tiles of the partial round
  //            as quarter tiles with the small kernel.
  // rounds are counted with the CUs that are certain to run a workgroup at the same time
  const int launch_quota = quota;
  quota = tile_queue_sure_cus(quota);
  const int64_t t128 = ceil_div(M, 128) * ceil_div(N, 128);
  // share of the board's CUs that a round of `tiles` leaves idle: the others run faster for it
  auto idle = [&](int64_t tiles) { return (double)(quota - tiles) / 256.0; };
  auto cost_small = [&](int64_t tiles) {       // 128x128 tiles on `quota` CUs
    const int64_t full = tiles / (2 * (int64_t)quota), rem = tiles % (2 * (int64_t)quota);
    // a CU shared by two workgroups finishes both in about 2 x 1.35 units (more when the
    // operands need the transposing reads); a workgroup alone takes 1.5 with all CUs at work and 1.05
    // with few (64-deep K-tiles: input gradient 4096 x 4096 x 1024, 256 tiles, 38 us; 1568 x 3072 x 768, 78 tiles, 23)
    constexpr double pen = (A_KC && B_KC) ? 1.3 : 1.45;
    const double alone = A_KC ? 1.5 - 0.45 * idle(rem) : 1.2 * pen;
    return (double)full * 2.0 * pen + (rem == 0 ? 0.0 : rem <= quota ? alone : 2.0 * pen);
  };
  // 256x256 tiles go to the four-wave kernel where it takes the product; a round of it takes
  // about 3.5 units where the eight-wave kernel takes 4 (9216 x 1024 x 3072 forward, 1.7 rounds: 52 us in
  // two rounds of large tiles, 55 as one and quarter tiles).  SwiGLU's epilogue, an exponential and a division per
  // pair of values, is not covered by another wave there: up to 1024 k-values the eight-wave
  // kernel is faster (1568 x 768 x 3072 on 96 CUs 28.6 us, 30.2 with four waves; 9216 x 1024 x 3072 on 64 194 and 203), except in whole
  // rounds that load most of the board (the same on 256 CUs 78 and 71).
  const int64_t whole = t256 / quota, rest = t256 % quota;
  const bool w4 = w4_takes<A_KC, B_KC>(K) && w4_enabled() && !(aa.act == ACT_SWIGLU && K <= 1024 && (whole == 0 || quota < 192));
  const double round256 = w4 ? 3.5 : 4.0;
  auto cost_w4 = [&](int64_t tiles, double round) {
    const int64_t rem = tiles % quota;
    return round * ((double)(tiles / quota) + (rem ? 1.0 - 0.39 * idle(rem) : 0.0));
  };
  // A lone round of 256 rows, which leaves CUs without a tile, is priced in full against the quarter tiles (with the
  // discount that it gets against lower tiles, GELU and SwiGLU products took 1 to 2 % longer over 36 shapes
  // on 8 shares of the CUs).
  const double cost256 = w4 && whole > 0 ? cost_w4(t256, round256) : (double)ceil_div(t256, quota) * round256;
  const double cost128 = cost_small(t128);
  const double cost_mix = (whole > 0 && rest > 0) ? (double)whole * round256 + cost_small(4 * rest) + 0.15 : 1e30;
  // Tiles of 224, 192 or 160 rows: where tiles of 256 leave many CUs without one in the last (or only)
  // round, lower ones fill it.  In the units above a round takes 3.15, 2.8 or 2.57 (3.5 for 256 rows: a
  // lower tile reads its weight-side fragments for fewer instructions), less 0.39 of it times the
  // share of the board that it leaves idle (which also has 8192 x 2048 x 11264, 5.5 rounds of 256 rows, end
  // in half a round of large tiles, 274 us, not in quarter tiles, 284).  SwiGLU's epilogue wants all CUs: with
  // fewer tiles than CUs the quarter tiles keep it.
  // Measured, plan with 256 rows -> this: forward 9216 x 4096 x 1024 (144 tiles -> 232 of 160 rows)
  // 74 -> 63 us, 9216 x 1024 x 1024 25.6 -> 21.9; input gradient 9216 x 1024 x 4096 73 -> 62; with GELU
  // 2048 x 4096 x 4096 (160 rows) 82 -> 63; forward
  // 8192 x 2048 x 3072 (1.5 rounds -> 444 tiles of 224) 93 -> 82; 9216 x 1024 x 4096 (2.25 rounds ->
  // 768 tiles of 192) 73 -> 68; left alone: 12000 x 1280 x 1280, 235 tiles, 34 us, 42 and more in lower ones.
  int mi = 8;
  if constexpr (A_KC) {
    if (w4 && forced_tile() == 0) {
      double best = std::min(std::min(cost_w4(t256, round256), cost128), cost_mix);
      for (int m = 7; m >= 5; --m) {
        const int64_t tiles = ceil_div(M, 32 * m) * ceil_div(N, 256);
        if (aa.act == ACT_SWIGLU && tiles < quota) continue;
        const double c = cost_w4(tiles, m == 7 ? 3.15 : m == 6 ? 2.8 : 2.57);
        if (c < best) { best = c; mi = m; }
      }
    }
    if (forced_tile() >= 5 && forced_tile() <= 7 && w4) mi = forced_tile();
    auto low = [&](auto rows) {
      return launch_w4<A_KC, B_KC, decltype(rows)::value>(s, launch_quota, M, N, K, A, lda, B, ldb, C, ldc, bias, R, a_bytes, b_bytes, c_bytes, 0, -1, aa);
    };
    if (mi == 7) return low(std::integral_constant<int, 7>{});
    if (mi == 6) return low(std::integral_constant<int, 6>{});
    if (mi == 5) return low(std::integral_constant<int, 5>{});
  }
  int plan = cost256 <= cost128 ? (cost256 <= cost_mix ? 256 : 0) : (cost128 <= cost_mix ? 128 : 0);
  if (forced_tile() == 128 || forced_tile() == 256) plan = forced_tile();
  if (forced_tile() == 1 && whole > 0 && rest > 0) plan = 0;
  // one launch of 256x256 tiles (big) or of 128x128 (quarter) tiles over coarse tiles
  // [tile_begin, tile_begin + tile_count) (tile_count < 0: all), with the epilogue `aa` asks for
  auto launch_tiles = [&](auto big_, int sub, int tile_begin, int tile_count) -> mosaic_status {
    constexpr bool BIG = decltype(big_)::value;
    constexpr int TB = BIG ? 256 : 128, WN_ = BIG ? 4 : 2;
    if constexpr (BIG && w4_form<A_KC, B_KC>()) {
      if (w4) return launch_w4<A_KC, B_KC>(s, launch_quota, M, N, K, A, lda, B, ldb, C, ldc, bias, R, a_bytes, b_bytes, c_bytes, tile_begin, tile_count, aa);
    }
    if constexpr (A_KC && !B_KC) {
      if (aa.act == ACT_GELU)
        return launch_mfma<TB, TB, 2, WN_, A_KC, B_KC, PIECES_NONE, ACT_GELU>(s, launch_quota, M, N, K, A, lda, B, ldb, C, ldc, bias, R, a_bytes, b_bytes,
                                                                        c_bytes, 1, 0, nullptr, sub, tile_begin, tile_count, aa);
      if (aa.act == ACT_TAPS)
        return launch_mfma<TB, TB, 2, WN_, A_KC, B_KC, PIECES_NONE, ACT_TAPS>(s, launch_quota, M, N, K, A, lda, B, ldb, C, ldc, bias, R, a_bytes, b_bytes,
                                                                        c_bytes, 1, 0, nullptr, sub, tile_begin, tile_count, aa);
      if (aa.act == ACT_SWIGLU)
        return launch_mfma<TB, TB, 2, WN_, A_KC, B_KC, PIECES_NONE, ACT_SWIGLU>(s, launch_quota, M, N, K, A, lda, B, ldb, C, ldc, bias, R, a_bytes, b_bytes,
                                                                          c_bytes, 1, 0, nullptr, sub, tile_begin, tile_count, aa);
    }
    return launch_mfma<TB, TB, 2, WN_, A_KC, B_KC>(s, launch_quota, M, N, K, A, lda, B, ldb, C, ldc, bias, R, a_bytes, b_bytes, c_bytes, 1, 0,
                                                   nullptr, sub, tile_begin, tile_count, aa);
  };
  if (plan == 256) return launch_tiles(std::true_type{}, 1, 0, -1);
  // Tiles of 64 rows where even those all get a CU of their own: a lone tile is bound by what its CU's vector cache and LDS pass per
  // K-tile (a 128 x 128 tile 0.35 us per 64 k-values, 0.21 of it matrix work), so half a tile to each of twice the CUs is faster however
  // short the contraction.  128 -> 64 rows: forward 1568 x 768 x 768 9.6 -> 8.3 us, 1568 x 3072 x 768 22.8 -> 19.2, with GELU
  // 12.8 -> 10.5 and 25.9 -> 21.4; input gradient 200 x 1024 x 3072 21.4 -> 17.7, on 64 CUs 21.4 -> 17.6.
  // An output on an operand stays with 128 rows, of which there may be only one tile: it then reads everything before it stores.
  if constexpr (A_KC) {
    auto on_operand = [&](const void* out, uint32_t bytes) { return overlap(out, bytes, A, a_bytes) || overlap(out, bytes, B, b_bytes); };
    if (plan == 128 && ceil_div(M, 64) * ceil_div(N, 128) <= quota && !on_operand(C, c_bytes) && !on_operand(aa.C2, aa.c2_bytes)) {
      auto go = [&](auto act) {
        return launch_mfma<64, 128, 2, 2, A_KC, B_KC, PIECES_NONE, decltype(act)::value, 64>(s, launch_quota, M, N, K, A, lda, B, ldb, C, ldc, bias, R, a_bytes, b_bytes,
                                                                                          c_bytes, 1, 0, nullptr, 1, 0, -1, aa);
      };
      if constexpr (!B_KC) {
        if (aa.act == ACT_GELU) return go(std::integral_constant<int, ACT_GELU>{});
      }
      if (aa.act == ACT_NONE) return go(std::integral_constant<int, ACT_NONE>{});
    }
  }
  if (plan == 128) return launch_tiles(std::false_type{}, 1, 0, -1);
  const int head = (int)(whole * quota);
  MOSAIC_TRY(launch_tiles(std::true_type{}, 1, 0, head));
  return launch_tiles(std::false_type{}, 2, head, (int)rest);
}

}  // namespace

// gemm_f32.hip
mosaic_status launch_gemm_f32(hipStream_t s, int quota, int dtype, bool a_kc, bool b_kc, int M, int N, int K, const void* A,
                              int64_t lda, const void* B, int64_t ldb, void* C, int64_t ldc, const void* bias, const void* R);
mosaic_status launch_linear_bwd_f32(hipStream_t s, int quota, int64_t T, int64_t k, int64_t n, const void* X, const void* dY, const void* W,
                                    void* dX, void* dW, bool* taken, int act = -1, const void* Z = nullptr, void* dZ = nullptr, float* sums = nullptr);
mosaic_status launch_layer_fwd_f32(hipStream_t s, int quota, int norm, int act, int64_t T, int64_t k, int64_t n, float eps, const void* X, const void* gamma,
                                   const void* beta, void* U, float* stats, const void* W, const void* bias, void* Z, void* A, bool* taken);

size_t gemm_splitk_scratch_bytes(int64_t M, int64_t N, int64_t K) {
  int first = 0;
  const int sk = splitk_plan(M, N, K, &first);
  const int64_t cut = ceil_div(M, 256) * ceil_div(N, 256) - first;      // whole 256x256 tiles, edge tiles too
  return sk > 1 ? (size_t)sk * (size_t)cut * 65536 * sizeof(float) : 0;
}

// fused != null: a forward-form call that also wants act(C) in C2; *fused says whether the
// launch took care of it
static mosaic_status launch_gemm_impl(hipStream_t s, int quota, int dtype, bool a_kc, bool b_kc, int64_t M, int64_t N,
                          int64_t K, const void* A, int64_t lda, const void* B, int64_t ldb, void* C,
                          int64_t ldc, const void* bias, const void* R, void* splitk_scratch,
                          int64_t b_rows, int act, void* C2, int64_t ldc2, bool* fused, int64_t r_rows = 0, int64_t taps_lo = 0) {
  if (fused) *fused = false;
  if (b_rows < 0 || b_kc) b_rows = K;
  if (M < 0 || N < 0 || K < 0) MOSAIC_FAIL(MOSAIC_EINVAL, "negative GEMM size");
  if (M > INT32_MAX || N > INT32_MAX || K > INT32_MAX) MOSAIC_FAIL(MOSAIC_EUNSUPPORTED, "GEMM dimension too large");
  if (M == 0 || N == 0) return MOSAIC_OK;
  const bool vec_ok = (lda % 8 == 0) && (ldb % 8 == 0) && (K % 8 == 0 || (!a_kc && !b_kc)) &&
                      (a_kc || M % 8 == 0 || lda >= ceil_div(M, 8) * 8) && (b_kc || N % 8 == 0) &&
                      ((uintptr_t)A % 16 == 0) && ((uintptr_t)B % 16 == 0) && ((uintptr_t)C % 16 == 0) &&
                      (ldc % 8 == 0) && (N % 8 == 0) && K > 0 &&
                      (R == nullptr || (uintptr_t)R % 16 == 0) && (bias == nullptr || (uintptr_t)bias % 16 == 0);
  // extents in bytes as seen by the buffer descriptors (dense rows: ld >= logical width)
  const int64_t a_ext = a_kc ? ((M - 1) * lda + K) * 2 : ((K - 1) * lda + std::min(ceil_div(M, 8) * 8, lda)) * 2;
  const int64_t b_ext = b_kc ? ((N - 1) * ldb + K) * 2 : ((b_rows - 1) * ldb + N) * 2;
  const int64_t c_ext = ((M - 1) * ldc + N) * 2;
  const int64_t lim = (int64_t)1 << 31;
  if (dtype == MOSAIC_BF16 && vec_ok && a_ext < lim && b_ext < lim && c_ext < lim) {
    const uint32_t ab = (uint32_t)a_ext, bb = (uint32_t)b_ext, cb = (uint32_t)c_ext;
    const bf16 *a = (const bf16*)A, *b = (const bf16*)B, *bi = (const bf16*)bias, *r = (const bf16*)R;
    bf16* c = (bf16*)C;
    if (a_kc && !b_kc) {
      ActArgs aa;
      if (const int64_t d = std::max(r_rows, taps_lo)) { aa.r_rows = (uint32_t)d; aa.r_magic = (uint32_t)(((uint64_t)1 << 32) / (uint64_t)d + 1); }
      if (fused && C2 && !R && (uintptr_t)C2 % 16 == 0 && ldc2 % 8 == 0) {
        const int64_t n2 = act == MOSAIC_SWIGLU ? N / 2 : N;
        const int64_t c2_ext = taps_lo > 0 ? M / 2 * 3 * N * 2 : ((M - 1) * ldc2 + n2) * 2;
        // gate and up halves must be whole quarter tiles wide: a tile then never straddles the halves
        const bool ok = c2_ext < lim && (act == MOSAIC_GELU || (act == MOSAIC_SWIGLU && N % 256 == 0));
        if (ok) {
          aa.act = taps_lo > 0 ? ACT_TAPS : act == MOSAIC_GELU ? ACT_GELU : ACT_SWIGLU;
          aa.C2 = (bf16*)C2; aa.ldc2 = ldc2; aa.c2_bytes = (uint32_t)c2_ext;
          aa.gu_f = act == MOSAIC_SWIGLU ? (int)(N / 2) : 0;
          *fused = true;
        }
      }
      return launch_mfma_shape<true, false>(s, quota, (int)M, (int)N, (int)K, a, lda, b, ldb, c, ldc, bi, r, ab, bb, cb, aa);
    }
    if (a_kc && b_kc) return launch_mfma_shape<true, true>(s, quota, (int)M, (int)N, (int)K, a, lda, b, ldb, c, ldc, bi, r, ab, bb, cb);
    if (!a_kc && !b_kc) return launch_wgrad(s, quota, (int)M, (int)N, (int)K, a, lda, b, ldb, c, ldc, bi, r, ab, bb, cb, (float*)splitk_scratch);
    return launch_mfma_shape<false, true>(s, quota, (int)M, (int)N, (int)K, a, lda, b, ldb, c, ldc, bi, r, ab, bb, cb);
  }
  if (r_rows > 0) {
    MOSAIC_TRY(launch_gemm_f32(s, quota, dtype, a_kc, b_kc, (int)M, (int)N, (int)b_rows, A, lda, B, ldb, C, ldc, bias, nullptr));
    return launch_add_pos(s, quota, dtype, (int)(M / r_rows), (int)r_rows, (int)N, R, C);
  }
  return launch_gemm_f32(s, quota, dtype, a_kc, b_kc, (int)M, (int)N, (int)b_rows, A, lda, B, ldb, C, ldc, bias, R);
}

mosaic_status launch_gemm(hipStream_t s, int quota, int dtype, bool a_kc, bool b_kc, int64_t M, int64_t N,
                          int64_t K, const void* A, int64_t lda, const void* B, int64_t ldb, void* C,
                          int64_t ldc, const void* bias, const void* R, void* splitk_scratch, int64_t b_rows) {
  return launch_gemm_impl(s, quota, dtype, a_kc, b_kc, M, N, K, A, lda, B, ldb, C, ldc, bias, R, splitk_scratch, b_rows, 0, nullptr, 0, nullptr);
}

mosaic_status launch_embed_fwd(hipStream_t s, int quota, int dtype, int64_t B, int64_t rows, int64_t n, int64_t k, int64_t ldx, const void* X,
                               const void* W, const void* bias, const void* table, void* Y) {
  const int64_t M = B * rows;
  if (rows < 2 || (M + 255) * rows >= (int64_t)1 << 32) {      // not table_row's range (rows of a tile past M too)
    MOSAIC_TRY(launch_gemm_impl(s, quota, dtype, true, false, M, n, ldx, X, ldx, W, n, Y, n, bias, nullptr, nullptr, k, 0, nullptr, 0, nullptr));
    return launch_add_pos(s, quota, dtype, (int)B, (int)rows, (int)n, table, Y);
  }
  return launch_gemm_impl(s, quota, dtype, true, false, M, n, ldx, X, ldx, W, n, Y, n, bias, table, nullptr, k, 0, nullptr, 0, nullptr, rows);
}

mosaic_status launch_linear_act_fwd(hipStream_t s, int quota, int dtype, int act, int64_t T, int64_t k, int64_t n,
                                    const void* X, const void* W, const void* bias, void* Z, void* Aout) {
  if (act != MOSAIC_GELU && act != MOSAIC_SWIGLU && act != MOSAIC_GELU_TANH) MOSAIC_FAIL(MOSAIC_EINVAL, "unknown activation %d", act);
  if (act == MOSAIC_SWIGLU && (n % 2)) MOSAIC_FAIL(MOSAIC_EINVAL, "SwiGLU needs an even output width, got %lld", (long long)n);
  const int64_t na = act == MOSAIC_SWIGLU ? n / 2 : n;
  bool fused = false;
  if (dtype == MOSAIC_F32) {
    MOSAIC_TRY(launch_layer_fwd_f32(s, quota, 0, act, T, k, n, 0.f, X, nullptr, nullptr, nullptr, nullptr, W, bias, Z, Aout, &fused));
    if (fused) return MOSAIC_OK;
  }
  MOSAIC_TRY(launch_gemm_impl(s, quota, dtype, true, false, T, n, k, X, k, W, n, Z, n, bias, nullptr, nullptr, -1, act, Aout, na,
                              act == MOSAIC_GELU_TANH ? nullptr : &fused));
  if (fused || T == 0 || n == 0) return MOSAIC_OK;
  if (act == MOSAIC_SWIGLU) return launch_swiglu_fwd(s, quota, dtype, T, na, Z, Aout);
  if (act == MOSAIC_GELU_TANH) return launch_gelu_tanh_fwd(s, quota, dtype, T * n, Z, Aout);
  return launch_gelu_fwd(s, quota, dtype, T * n, Z, Aout);
}

mosaic_status launch_gelu_taps_fwd(hipStream_t s, int quota, int dtype, int64_t B, int64_t lo, int64_t n, int64_t k, int64_t ldx, const void* X, const void* W,
                                   const void* bias, void* Z, void* A, void* P) {
  const int64_t T = 2 * B * lo;
  const bool in_range = lo >= 2 && (T / 2 + 256) * lo < (int64_t)1 << 32;
  bool fused = false;
  MOSAIC_TRY(launch_gemm_impl(s, quota, dtype, true, false, T, n, ldx, X, ldx, W, n, Z, n, bias, nullptr, nullptr, k, MOSAIC_GELU, P, 3 * n,
                              in_range ? &fused : nullptr, 0, in_range ? lo : 0));
  if (fused || T == 0 || n == 0) return MOSAIC_OK;
  MOSAIC_TRY(launch_gelu_fwd(s, quota, dtype, T * n, Z, A));
  return launch_im2col1d(s, quota, dtype, B, (int)(2 * lo), (int)lo, (int)n, 2, A, P);
}

namespace {
template <int PIECES>
mosaic_status launch_pair(hipStream_t s, const PairHalf& dg, const PairHalf& wg) {
  constexpr size_t smem = (size_t)NS * (128 + 128) * 64 * 2;
  auto kern = gemm_bf16_pair_kernel<PIECES>;
  static std::once_flag attr_once;
  static hipError_t attr_rc = hipSuccess;
  std::call_once(attr_once, [&] {
    attr_rc = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  });
  MOSAIC_HIP(attr_rc);
  kern<<<dg.tq.wgs + wg.tq.wgs, 256, smem, s>>>(dg, wg);
  MOSAIC_LAUNCH_CHECK();
  return MOSAIC_OK;
}
}  // namespace

mosaic_status launch_linear_bwd(hipStream_t s, int quota, int dtype, int64_t T, int64_t k, int64_t n, const void* X, const void* dY,
                                const void* W, void* dX, void* dW, void* splitk_scratch, bool dx_first, int64_t ldx) {
  if (ldx == 0) ldx = k;
  const int64_t es = (int64_t)dtype_size(dtype), xin = ((T - 1) * ldx + k) * es, xb = T * k * es, yb = T * n * es, wb = k * n * es, lim = (int64_t)1 << 31;
  const uintptr_t all = (uintptr_t)X | (uintptr_t)dY | (uintptr_t)W | (uintptr_t)dX | (uintptr_t)dW;
  const bool fits = dtype == MOSAIC_BF16 && T > 0 && k > 0 && n > 0 && T <= INT32_MAX && k <= INT32_MAX && n <= INT32_MAX && k % 8 == 0 && n % 8 == 0 && ldx % 8 == 0 &&
                    all % 16 == 0 && xin < lim && xb < lim && yb < lim && wb < lim;
  // an output that lies on an input, which the order of two launches may allow, keeps them
  const bool apart = !overlap(dX, xb, X, xin) && !overlap(dX, xb, dY, yb) && !overlap(dX, xb, W, wb) && !overlap(dX, xb, dW, wb) &&
                     !overlap(dW, wb, X, xin) && !overlap(dW, wb, dY, yb) && !overlap(dW, wb, W, wb);
  if (dtype == MOSAIC_F32 && T > 0 && k > 0 && n > 0 && ldx == k && apart && pair_enabled()) {
    bool taken;
    MOSAIC_TRY(launch_linear_bwd_f32(s, quota, T, k, n, X, dY, W, dX, dW, &taken));
    if (taken) return MOSAIC_OK;
  }
  if (fits && apart) {
    const int cus = tile_queue_sure_cus(quota);
    const WgradPlan wp = wgrad_plan(k, n, T, cus, splitk_scratch != nullptr, w4_takes<false, false>(T));
    const PairPlan pp = pair_plan(T, k, n, cus, wp);
    if (pp.pair && pair_enabled()) {
      auto half = [&](const void* A, int64_t lda, const void* B, int64_t ldb, void* C, int64_t M, int64_t N, int64_t K, int wg0, int wgs) {
        PairHalf h = {};
        h.A = (const bf16*)A; h.B = (const bf16*)B; h.C = (bf16*)C;
        h.M = (int)M; h.N = (int)N; h.K = (int)K; h.lda = lda; h.ldb = ldb; h.ldc = N;
        h.tiles_m = (int)ceil_div(M, 128); h.tiles_n = (int)ceil_div(N, 128);
        h.tq.n_items = h.tiles_m * h.tiles_n; h.tq.chunk = 1; h.tq.mode = TQ_ROUNDS; h.tq.wg0 = wg0; h.tq.wgs = wgs;
        h.aa.row_block = row_block_for(K, M, 128);
        return h;
      };
      PairHalf dg = half(dY, n, W, n, dX, T, k, n, 0, pp.wgs_d), wg = half(X, ldx, dY, n, dW, k, n, T, pp.wgs_d, pp.wgs_w);
      dg.a_bytes = (uint32_t)yb; dg.b_bytes = (uint32_t)wb; dg.c_bytes = (uint32_t)xb;
      wg.a_bytes = (uint32_t)xin; wg.b_bytes = (uint32_t)yb; wg.c_bytes = (uint32_t)wb;
      if (wp.pieces > 1) { wg.ktiles_per = wp.kper / 64; return launch_pair<PIECES_CHAINED>(s, dg, wg); }
      return launch_pair<PIECES_NONE>(s, dg, wg);
    }
  }
  auto input_grad = [&] { return launch_gemm(s, quota, dtype, true, true, T, k, n, dY, n, W, n, dX, k, nullptr, nullptr); };
  if (dx_first) MOSAIC_TRY(input_grad());
  MOSAIC_TRY(launch_gemm(s, quota, dtype, false, false, k, n, T, X, ldx, dY, n, dW, n, nullptr, nullptr, splitk_scratch));
  return dx_first ? MOSAIC_OK : input_grad();
}

mosaic_status launch_norm_linear_fwd(hipStream_t s, int quota, int dtype, int norm, int act, int64_t T, int64_t h, int64_t n, float eps, const void* X,
                                     const void* gamma, const void* beta, void* U, float* stats, const void* W, const void* bias, void* Z, void* A) {
  if (dtype == MOSAIC_F32) {
    bool taken;
    MOSAIC_TRY(launch_layer_fwd_f32(s, quota, norm, act, T, h, n, eps, X, gamma, beta, U, stats, W, bias, Z, A, &taken));
    if (taken) return MOSAIC_OK;
  }
  MOSAIC_TRY(launch_norm_fwd(s, quota, dtype, norm, T, h, eps, X, gamma, beta, U, stats));
  if (act < 0) return launch_gemm(s, quota, dtype, true, false, T, n, h, U, h, W, n, Z, n, bias, nullptr);
  return launch_linear_act_fwd(s, quota, dtype, act, T, h, n, U, W, bias, Z, A);
}

mosaic_status launch_act_linear_bwd(hipStream_t s, int quota, int dtype, int act, int64_t T, int64_t k, int64_t n, const void* Z, const void* A, const void* dY,
                                    const void* W, void* dA, void* dZ, void* dW, void* splitk_scratch, void* colsum, void* scratch, ColReduceList* later) {
  const int64_t np = ceil_div(T, 8), es = (int64_t)dtype_size(dtype), zb = T * k * es * (act == MOSAIC_SWIGLU ? 2 : 1), wb = k * n * es;
  const bool apart = !overlap(dW, wb, A, T * k * es) && !overlap(dW, wb, dY, T * n * es) && !overlap(dW, wb, W, wb) && !overlap(dW, wb, Z, zb) &&
                     !overlap(dW, wb, dZ, zb) && !overlap(dZ, zb, A, T * k * es) && !overlap(dZ, zb, dY, T * n * es) && !overlap(dZ, zb, W, wb) && !overlap(dZ, zb, Z, zb);
  if (dtype == MOSAIC_F32 && apart && T > 0 && k > 0 && n > 0 && (act == MOSAIC_GELU || act == MOSAIC_SWIGLU) && later && later->n < ColReduceList::kMax &&
      (!colsum || colsum_partition_rows(T) == 8) && pair_enabled()) {
    bool taken;
    MOSAIC_TRY(launch_linear_bwd_f32(s, quota, T, k, n, A, dY, W, dA, dW, &taken, act, Z, dZ, colsum ? (float*)scratch : nullptr));
    if (taken) {
      if (colsum) later->job[later->n++] = {(const float*)scratch, (int)np, k, k, k, INT64_MAX, colsum, nullptr, nullptr};
      return MOSAIC_OK;
    }
  }
  MOSAIC_TRY(launch_linear_bwd(s, quota, dtype, T, k, n, A, dY, W, dA, dW, splitk_scratch, true));
  if (act == MOSAIC_SWIGLU) return launch_swiglu_bwd(s, quota, dtype, T, k, Z, dA, dZ);
  if (act == MOSAIC_GELU_TANH) return launch_gelu_tanh_bwd(s, quota, dtype, T * k, Z, dA, dZ);
  if (colsum) return launch_gelu_bwd_colsum(s, quota, dtype, T, k, Z, dA, dZ, colsum, scratch, later);
  return launch_gelu_bwd(s, quota, dtype, T * k, Z, dA, dZ);
}
