// bf16 GEMMs on the gfx950 matrix cores (v_mfma_f32_32x32x16_bf16, fp32 accumulate).
//
// One kernel template covers the three products of a dense layer.  With C[M x N] = A . B:
//   fprop  z  = x W^T      A = x  [M][K] (k contiguous)   B = W   [N][K] (k contiguous)
//   dgrad  dx = dz W_b     A = dz [M][K] (k contiguous)   B = W_b [K][N] (n contiguous)
//   wgrad  dW = dz^T x     A = dz [K][M] (m contiguous)   B = x   [K][N] (n contiguous)
// An operand whose contraction index is the contiguous one is staged in LDS row by row and
// each lane reads its 8 consecutive k values with one 128-bit LDS read.  An operand whose
// contraction index is the strided one is staged as it lies in memory ([k][row]) and each
// lane gets its 8 k values through two LDS transpose reads.
//
// Two kernels share the tile and epilogue code:
//   gemm_bf16_dma_kernel   16-byte aligned operands whose rows are whole 16-byte chunks: global loads write
//                          LDS directly (global_load_lds_dwordx4), NS stages deep, no staging registers;
//                          LDS is unpadded, bank conflicts are avoided by an XOR swizzle of the 16-byte
//                          chunks, applied on the global side of the copy.
//   gemm_bf16_any_kernel   any extents and alignment: global loads go through registers, three k tiles
//                          ahead, LDS double buffered and padded.
// Workgroup ids are remapped so that the workgroups of one XCD (ids equal mod 8) cover a
// compact 2-D patch of output tiles and share their operand panels in that XCD's L2.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <stdint.h>

#include "device_utils.h"
#include "gemm_mfma.h"
#include "mfma_common.h"
#include "kernels.h"

namespace tp {

namespace {


inline int k_tiles(int K) { return (K + DBK - 1) / DBK; }

// 8 consecutive values from an address of any (2-byte) alignment, those from `valid` on zero and not read
__device__ __forceinline__ uint4 load8(const uint16_t* p, int valid) {
  uint4 v = make_uint4(0, 0, 0, 0);
  if (valid >= 8) {
    __builtin_memcpy(&v, p, 16);
  } else if (valid > 0) {
    uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 7; ++j)
      if (j < valid) w[j >> 1] |= (uint32_t)p[j] << (16 * (j & 1));
    v = make_uint4(w[0], w[1], w[2], w[3]);
  }
  return v;
}

// ---- staging of one operand tile -------------------------------------------------------------
// k-contiguous operand: tile [R rows][BKT k]; memory element (r, k) at base[r*ld + k].
template <int R, int BKT, int NT>
struct RowTile {
  static constexpr int LD = BKT + 8;             // +16 B per row: conflict-free 128-bit reads
  static constexpr int kPerRow = BKT / 8;        // 16-byte chunks per row
  static constexpr int kChunks = R * kPerRow / NT;
  static constexpr int kRowStep = NT / kPerRow;
  static constexpr int kLdsElems = R * LD;
  static_assert(R * kPerRow % NT == 0, "tile does not divide among the threads");

  static __device__ __forceinline__ void load(uint4 (&regs)[kChunks], const uint16_t* __restrict__ base, int ld, int r0,
                                              int rows, int k0, int K) {
    const int k = k0 + (threadIdx.x % kPerRow) * 8;
#pragma unroll
    for (int i = 0; i < kChunks; ++i) {
      const int r = threadIdx.x / kPerRow + kRowStep * i;
      // clamp: rows past the edge are computed but never stored
      regs[i] = load8(base + (size_t)min(r0 + r, rows - 1) * ld + k, K - k);
    }
  }
  static __device__ __forceinline__ void store(const uint4 (&regs)[kChunks], uint16_t* lds) {
    const int c = threadIdx.x % kPerRow;
#pragma unroll
    for (int i = 0; i < kChunks; ++i) {
      const int r = threadIdx.x / kPerRow + kRowStep * i;
      *reinterpret_cast<uint4*>(lds + r * LD + c * 8) = regs[i];
    }
  }
  // operand rows rbase..rbase+31: the lane reads k = kk*16 + 8*(lane/32) .. +7 of row rbase + lane%32
  static __device__ __forceinline__ bf16x8 frag(const uint16_t* lds, int rbase, int kk, int lane) {
    const uint4 v = *reinterpret_cast<const uint4*>(lds + (rbase + (lane & 31)) * LD + kk * 16 + (lane >> 5) * 8);
    return __builtin_bit_cast(bf16x8, v);
  }
};

// k-strided operand: tile [BKT k][R rows]; memory element (r, k) at base[k*ld + r].
// Fragments come from the LDS transpose read (ds_read_b64_tr_b16): within each group of 16
// lanes, lane s supplies the address of 4 consecutive bf16 and receives element s%4 of the
// four lanes 4*j + s/4 (j = 0..3).  With lane s pointing at row k0 + s/4, columns
// c0 + 4*(s%4) .. +3, lane i of the group ends up with rows k0..k0+3 of column c0 + i: four
// consecutive k of its own row/column of the MFMA operand.  Two such reads give the 8 k values.
template <int R, int BKT, int NT>
struct ColTile {
  static constexpr int LD = R + 32;  // row stride = 64 B (mod 256 B): the 4 rows of a transpose read hit distinct banks
  static constexpr int kPerK = R / 8;
  static constexpr int kChunks = BKT * kPerK / NT;
  static constexpr int kLdsElems = BKT * LD;
  static_assert(BKT * kPerK % NT == 0, "tile does not divide among the threads");

  static __device__ __forceinline__ void load(uint4 (&regs)[kChunks], const uint16_t* __restrict__ base, int ld, int r0,
                                              int rows, int k0, int K) {
#pragma unroll
    for (int i = 0; i < kChunks; ++i) {
      const int id = threadIdx.x + NT * i;
      const int r = r0 + (id % kPerK) * 8, k = k0 + id / kPerK;
      regs[i] = load8(base + (size_t)k * ld + r, k < K ? rows - r : 0);
    }
  }
  static __device__ __forceinline__ void store(const uint4 (&regs)[kChunks], uint16_t* lds) {
#pragma unroll
    for (int i = 0; i < kChunks; ++i) {
      const int id = threadIdx.x + NT * i;
      const int c = id % kPerK, k = id / kPerK;
      *reinterpret_cast<uint4*>(lds + k * LD + c * 8) = regs[i];
    }
  }
  static __device__ __forceinline__ bf16x8 frag(const uint16_t* lds, int rbase, int kk, int lane) {
    const int g = lane >> 4, s = lane & 15;
    const int k = kk * 16 + 8 * (g >> 1) + (s >> 2);
    const int c = rbase + 16 * (g & 1) + 4 * (s & 3);
    typedef __attribute__((address_space(3))) shortx4* lds_ptr;
    const uint16_t* p = lds + k * LD + c;
    const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p));
    const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + 4 * LD));
    const shortx8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
  }
};

template <int R, int BKT, int NT, bool COL>
struct TileSel { using type = RowTile<R, BKT, NT>; };
template <int R, int BKT, int NT>
struct TileSel<R, BKT, NT, true> { using type = ColTile<R, BKT, NT>; };


// output of contraction range `split`: only the fp32 weight-gradient product is ever split
template <class E>
__device__ __forceinline__ const E& epi_of_split(const E& e, int) { return e; }
struct EpiWgradSplit {
  float* out; int ldc; size_t split_stride;
  static constexpr bool kSwap = false;
};
__device__ __forceinline__ EpiWgrad epi_of_split(const EpiWgradSplit& e, int split) {
  return EpiWgrad{e.out + (size_t)split * e.split_stride, e.ldc};
}

// ---- any extents and alignment ------------------------------------------------------------------
// Bound by the latency of its loads at the few workgroups it mostly has.  PF: k tiles in flight in registers (with one,
// every k tile cost a memory latency: 0.7 us at 100 x 2000 x 2000).  Against bounds-checked fp32 FMAs: stage of width 2315
// 1039 -> 267 us, 783 491 -> 150 us, of width 70 with 200 classes 1095 -> 216 us.
template <int BM, int BN, int WGM, int WGN, int BKT, int PF, bool A_COL, bool B_COL, class Epi>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_bf16_any_kernel(int M, int N, int K, int per,
                                                                        const uint16_t* __restrict__ A, int lda,
                                                                        const uint16_t* __restrict__ B, int ldb,
                                                                        Epi epi, TileMap map) {
  constexpr int NT = 64 * WGM * WGN;
  using ATile = typename TileSel<BM, BKT, NT, A_COL>::type;
  using BTile = typename TileSel<BN, BKT, NT, B_COL>::type;
  constexpr int WM = BM / WGM, WN = BN / WGN;  // wave tile
  constexpr int TM = WM / 32, TN = WN / 32;
  extern __shared__ __attribute__((aligned(16))) uint16_t lds_raw[];
  auto lds_a = [&](int buf) { return lds_raw + buf * ATile::kLdsElems; };
  auto lds_b = [&](int buf) { return lds_raw + 2 * ATile::kLdsElems + buf * BTile::kLdsElems; };

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = (wave / WGN) * WM, wn = (wave % WGN) * WN;
  int tile_m, tile_n;
  map.get(blockIdx.x, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  auto compute = [&](int buf) {
    const uint16_t* la = lds_a(buf);
    const uint16_t* lb = lds_b(buf);
#pragma unroll
    for (int kk = 0; kk < BKT / 16; ++kk) {
      bf16x8 af[TM], bfr[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) af[i] = ATile::frag(la, wm + i * 32, kk, lane);
#pragma unroll
      for (int j = 0; j < TN; ++j) bfr[j] = BTile::frag(lb, wn + j * 32, kk, lane);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = mma<Epi::kSwap>(af[i], bfr[j], acc[i][j]);
    }
  };

  // k tiles first .. end - 1: the contraction range blockIdx.y, `per` tiles long
  const int first = blockIdx.y * per, end = min(first + per, (K + BKT - 1) / BKT);
  uint4 ra[PF][ATile::kChunks], rb[PF][BTile::kChunks];
#pragma unroll
  for (int u = 0; u < PF; ++u)
    if (first + u < end) {
      ATile::load(ra[u], A, lda, m0, M, (first + u) * BKT, K);
      BTile::load(rb[u], B, ldb, n0, N, (first + u) * BKT, K);
    }
  static_assert(PF % 2 == 0, "LDS buffers alternate with the k tiles of a run");
  for (int kt = first; kt < end; kt += PF) {
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      if (kt + u >= end) break;  // uniform
      ATile::store(ra[u], lds_a(u & 1));
      BTile::store(rb[u], lds_b(u & 1));
      // tile kt + u visible; the other buffer is free once every wave is here, behind its reads of the tile before
      lds_barrier();
      if (kt + u + PF < end) {
        ATile::load(ra[u], A, lda, m0, M, (kt + u + PF) * BKT, K);
        BTile::load(rb[u], B, ldb, n0, N, (kt + u + PF) * BKT, K);
      }
      compute(u & 1);
    }
  }
  store_tiles<TM, TN>(acc, epi_of_split(epi, blockIdx.y), m0 + wm, n0 + wn, M, N, lane);
}

template <int BM, int BN, int WGM, int WGN, bool A_COL, bool B_COL, class Epi>
hipError_t launch_any(hipStream_t s, int M, int N, int K, const uint16_t* A, int lda, const uint16_t* B, int ldb, const Epi& epi,
                      int per) {
  constexpr int NT = 64 * WGM * WGN, PF = 4;
  using ATile = typename TileSel<BM, DBK, NT, A_COL>::type;
  using BTile = typename TileSel<BN, DBK, NT, B_COL>::type;
  constexpr size_t lds_bytes = 2 * (ATile::kLdsElems + BTile::kLdsElems) * sizeof(uint16_t);
  static_assert(lds_bytes <= 64 * 1024, "more LDS than a launch has without asking for it");
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  hipLaunchKernelGGL((gemm_bf16_any_kernel<BM, BN, WGM, WGN, DBK, PF, A_COL, B_COL, Epi>),
                     dim3(tiles_m * tiles_n, (k_tiles(K) + per - 1) / per), dim3(NT), lds_bytes, s, M, N, K, per, A, lda, B, ldb,
                     epi, make_tile_map(tiles_m, tiles_n));
  return hipGetLastError();
}

// a pointer that is the same in every lane, where the compiler would form it in vector registers
__device__ __forceinline__ const uint16_t* in_sgprs(const uint16_t* p) {
  const uint64_t a = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a), hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  return reinterpret_cast<const uint16_t*>((uint64_t)hi << 32 | lo);
}

struct NoInputs {
  template <class Epi>
  __device__ __forceinline__ void load(const Epi&, int, int, int) {}
};
template <int TM, int TN, class Epi, bool ROWS>
struct EpiInputs { using type = NoInputs; };
template <int TM, int TN, class Epi>
struct EpiInputs<TM, TN, Epi, true> { using type = RowInputs<TM, TN, Epi>; };

// LEAN: small wave tiles (one or two 32x32 blocks) have so few MFMAs per k tile that the address and stage
// bookkeeping is a third of the instructions of the loop.  The k loop is then unrolled over the NS stage buffers,
// so that every LDS address is a loop-invariant register plus an immediate and the stage indices are constants;
// the source pointers of the copies advance instead of being recomputed.  The last tiles (no copies left to issue
// in step with them) run through the generic loop.  Worth about 5 % on the 64x64 and 128x64 tiles.
// ROT: the barrier that makes a k tile visible sits one k step early, before the last MFMA group of the tile
// before it, so that the first fragment reads of the new tile run under that group instead of stalling the wave
// (with one wave per SIMD nothing else would cover them).  The fragment reads of the next k step go out one by one
// between the MFMAs of the current one, as the copies do: bunched in front of them, all eight waves queued for the LDS
// at once.  Eight waves split 256x128 as 64x64 (4 fragments for 4 MFMAs; 128x32 takes 5).  The last NS - 1 tiles run
// without copies.  Together, weight gradient 8192 x 2048 over 32768 rows 870 -> 850 us, 6144 x 2048 794 -> 765, input
// gradient 2048 x 4096 x 4096 64.6 -> 62.5.
// TAIL: the contraction is no whole number of k tiles; what the last tile lacks is copied from a block of zeros, for
// both operands.  A kernel of its own, so that whole ones carry no second form of the copies.  Through registers, as in
// the kernel above with one k tile in flight, 100 x 2000 x 2000 took 23 us; a last stage of width 2000 235 -> 192 us a step.
template <int BM, int BN, int WGM, int WGN, int NS, bool A_COL, bool B_COL, class Epi, bool LEAN, bool ROT, bool TAIL>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_bf16_dma_kernel(int M, int N, int K, int per,
                                                                        const uint16_t* __restrict__ A, int lda,
                                                                        const uint16_t* __restrict__ B, int ldb,
                                                                        Epi epi, TileMap map, SideCopy side) {
  constexpr int NW = WGM * WGN;
  using AT = typename DmaSel<BM, NW, A_COL>::type;
  using BT = typename DmaSel<BN, NW, B_COL>::type;
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int kStageBytes = AT::kBytes + BT::kBytes;
  constexpr int kLoads = AT::kPerWave + BT::kPerWave;  // copies one wave issues per stage
  static_assert((NS - 2) * kLoads < 64, "too many copies in flight for vmcnt");
  extern __shared__ __attribute__((aligned(16))) uint16_t lds_raw[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = (wave / WGN) * WM, wn = (wave % WGN) * WN;
  for (size_t i = (size_t)blockIdx.x * (64 * NW) + threadIdx.x; i < side.nvec; i += (size_t)gridDim.x * (64 * NW))
    side.dst[i] = side.src[i];
  int tile_m, tile_n, split = blockIdx.y;
  if (A_COL && gridDim.y > 1) {
    const int at = xcd_position(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y), tile = at % gridDim.x;
    split = at / gridDim.x;
    tile_m = tile / map.tiles_n;
    tile_n = tile % map.tiles_n;
  } else {
    map.get(blockIdx.x, tile_m, tile_n);
    if (!map.inside(tile_m, tile_n)) return;
  }
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const uint32_t lds_base = lds_addr_of(lds_raw);
  // split: range of the contraction this workgroup sums over, `per` k tiles long (the last one may be shorter);
  // each range writes its own output (fp32 partial results that a second kernel adds in a fixed order)
  const int first = split * per;
  const int KT = min(per, (TAIL ? (K + DBK - 1) / DBK : K / DBK) - first);
  const int last_k = K - (first + KT - 1) * DBK;  // k values of the last tile, if it holds fewer than DBK
  A = in_sgprs(A + first * AT::tile_step(lda) + (size_t)m0 * (A_COL ? 1 : lda));
  B = in_sgprs(B + first * BT::tile_step(ldb) + (size_t)n0 * (B_COL ? 1 : ldb));

  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  AT ta;
  BT tb;
  ta.init(lda, 0, M - m0, wave, lane);
  tb.init(ldb, 0, N - n0, wave, lane);
  const size_t step_a = AT::tile_step(lda), step_b = BT::tile_step(ldb);
  constexpr int NM = (DBK / 16) * TM * TN;  // MFMAs of one wave per k tile
  // MFMA after which copy t of the next tile is issued.  With three or more stages a copy has a whole tile of slack
  // and the copies are spread evenly; with two stages the tile they fill is waited for at the next barrier, so
  // they all go out during the first MFMAs and the rest of the tile's arithmetic covers their latency.
  auto copy_slot = [](int t) constexpr { return NS == 2 && kLoads <= NM ? t : (t * NM) / kLoads; };

  // copy number t (0 .. kLoads-1) of k tile `tile` into stage `st`.  Tiles past the end re-read
  // the last tile into a stage nobody reads again, which keeps the number of copies per
  // iteration -- and with it the vmcnt arithmetic -- the same from the first tile to the last.
  auto issue_copy = [&](int t, int tile, int st) {
    const int tc = min(tile, KT - 1);
    const uint32_t dst = lds_base + st * kStageBytes;
    if (TAIL && tc == KT - 1) {  // uniform
      if (t < AT::kPerWave) ta.issue_one_of(last_k, t, dst, A + tc * step_a, wave, lane);
      else tb.issue_one_of(last_k, t - AT::kPerWave, dst + AT::kBytes, B + tc * step_b, wave, lane);
      return;
    }
    if (t < AT::kPerWave) ta.issue_one(t, dst, in_sgprs(A + tc * step_a), wave);
    else tb.issue_one(t - AT::kPerWave, dst + AT::kBytes, in_sgprs(B + tc * step_b), wave);
  };

  // prologue: stages 0 .. NS-2
#pragma unroll
  for (int st = 0; st < NS - 1; ++st)
#pragma unroll
    for (int t = 0; t < kLoads; ++t) issue_copy(t, st, st);

  // rows of the wave tile stored whole, by 4 * TN lanes each
  constexpr bool kRowStores = Epi::kSwap && 64 % (4 * TN) == 0;
  bool whole = false;
  if constexpr (kRowStores) whole = m0 + wm + WM <= M && n0 + wn + WN <= N && (N & 7) == 0 && epi.wide == 2;
  typename EpiInputs<TM, TN, Epi, kRowStores>::type row_inputs;

  int kt0 = 0;
  if constexpr (LEAN) {
    const uint16_t* pa = A + (size_t)(NS - 1) * step_a;  // source of the next tile to copy
    const uint16_t* pb = B + (size_t)(NS - 1) * step_b;
    for (; kt0 + NS <= KT - (NS - 1) - TAIL; kt0 += NS) {  // all copies of whole tiles
#pragma unroll
      for (int u = 0; u < NS; ++u) {  // tile kt0 + u lives in buffer u, tile kt0 + u + NS - 1 goes to buffer (u + NS - 1) % NS
        wait_vmcnt<(NS - 2) * kLoads>();
        lds_barrier();
        const uint16_t* la = lds_raw + u * (kStageBytes / 2);
        const uint16_t* lb = la + AT::kBytes / 2;
        const uint32_t dst = lds_base + ((u + NS - 1) % NS) * kStageBytes;
        // all fragments of the k tile first; fetched one k step ahead the forward products and gradients of 170 layers take the same time
        // (forward 1.002, input gradients 0.999, weight gradients 0.999)
        bf16x8 af[DBK / 16][TM], bfr[DBK / 16][TN];
#pragma unroll
        for (int kk = 0; kk < DBK / 16; ++kk) {
#pragma unroll
          for (int i = 0; i < TM; ++i) af[kk][i] = AT::frag(la, wm + i * 32, kk, lane);
#pragma unroll
          for (int j = 0; j < TN; ++j) bfr[kk][j] = BT::frag(lb, wn + j * 32, kk, lane);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kk = 0; kk < DBK / 16; ++kk) {
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
              acc[i][j] = mma<Epi::kSwap>(af[kk][i], bfr[kk][j], acc[i][j]);
              const int q = (kk * TM + i) * TN + j;  // compile-time after unrolling
#pragma unroll
              for (int t = 0; t < kLoads; ++t)
                if (copy_slot(t) == q) {
                  __builtin_amdgcn_sched_barrier(0);
                  if (t < AT::kPerWave) ta.issue_one(t, dst, pa, wave);
                  else tb.issue_one(t - AT::kPerWave, dst + AT::kBytes, pb, wave);
                  __builtin_amdgcn_sched_barrier(0);
                }
            }
          __builtin_amdgcn_sched_barrier(0);
        }
        pa += step_a;
        pb += step_b;
      }
    }
  }
  int rd = 0;        // stage holding tile kt (kt0 is a multiple of NS)
  int wr = NS - 1;   // stage that receives tile kt + NS - 1
  if constexpr (ROT) {
    static_assert(!LEAN, "the rotated loop has no unrolled form");
    constexpr int KS = DBK / 16;
    static_assert(KS % 2 == 0, "fragment buffers alternate with the k steps");
    // Step s of iteration kt reads the fragments of (tile kt, k step s) and multiplies those of the step before:
    // step 0 multiplies the last k step of tile kt-1 (zeros in the first iteration).
    bf16x8 af[2][TM], bfr[2][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) af[1][i][e] = 0;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 8; ++e) bfr[1][j][e] = 0;
    static_assert(NS <= 3, "the wait below knows of one newer tile in flight");
    // copies: issue those of tile kt + NS - 1
    auto tile = [&](int kt, auto copies) {
      if (NS == 2 || kt + 1 >= KT) wait_vmcnt<0>();
      else wait_vmcnt<(NS - 2) * kLoads>();
      lds_barrier();  // tile kt visible; every wave holds its last fragments of tile kt-1 in registers
      const uint16_t* la = lds_raw + rd * (kStageBytes / 2);
      const uint16_t* lb = la + AT::kBytes / 2;
#pragma unroll
      for (int st = 0; st < KS; ++st) {
        const int nx = st & 1, c = nx ^ 1;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            acc[i][j] = mma<Epi::kSwap>(af[c][i], bfr[c][j], acc[i][j]);
            const int q = i * TN + j;
#pragma unroll
            for (int r = 0; r < TM + TN; ++r)
              if (r * TM * TN / (TM + TN) == q) {
                __builtin_amdgcn_sched_barrier(0);
                if (r < TN) bfr[nx][r] = BT::frag(lb, wn + r * 32, st, lane);
                else af[nx][r - TN] = AT::frag(la, wm + (r - TN) * 32, st, lane);
                __builtin_amdgcn_sched_barrier(0);
              }
            if constexpr (decltype(copies)::value) {
#pragma unroll
              for (int t = 0; t < kLoads; ++t)
                if (copy_slot(t) == st * TM * TN + q) {
                  __builtin_amdgcn_sched_barrier(0);
                  issue_copy(t, kt + NS - 1, wr);
                  __builtin_amdgcn_sched_barrier(0);
                }
            }
          }
        __builtin_amdgcn_sched_barrier(0);
      }
      rd = rd + 1 == NS ? 0 : rd + 1;
      wr = wr + 1 == NS ? 0 : wr + 1;
    };
    for (int kt = 0; kt < KT - (NS - 1); ++kt) tile(kt, std::true_type{});
    for (int kt = max(0, KT - (NS - 1)); kt < KT; ++kt) tile(kt, std::false_type{});
    if (whole) row_inputs.load(epi, m0 + wm, n0 + wn, lane);  // under the last products
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = mma<Epi::kSwap>(af[1][i], bfr[1][j], acc[i][j]);
    kt0 = KT;
  }
  for (int kt = kt0; kt < KT; ++kt) {
    // tile kt has landed once at most the NS-2 newer tiles are still in flight
    wait_vmcnt<(NS - 2) * kLoads>();
    lds_barrier();  // tile kt visible to all waves; everybody is done reading stage `wr`
    const uint16_t* la = lds_raw + rd * (kStageBytes / 2);
    const uint16_t* lb = la + AT::kBytes / 2;
    {
      // Fixed schedule per k step: the LDS reads of step kk+1 go out first, then the MFMAs of
      // step kk with the global->LDS copies of tile kt+NS-1 spread evenly between them, so that
      // the wave never sits in the memory-instruction queue while its matrix core idles.
      bf16x8 af[2][TM], bfr[2][TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) af[0][i] = AT::frag(la, wm + i * 32, 0, lane);
#pragma unroll
      for (int j = 0; j < TN; ++j) bfr[0][j] = BT::frag(lb, wn + j * 32, 0, lane);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kk = 0; kk < DBK / 16; ++kk) {
        const int c = kk & 1, nx = c ^ 1;
        if (kk + 1 < DBK / 16) {
#pragma unroll
          for (int i = 0; i < TM; ++i) af[nx][i] = AT::frag(la, wm + i * 32, kk + 1, lane);
#pragma unroll
          for (int j = 0; j < TN; ++j) bfr[nx][j] = BT::frag(lb, wn + j * 32, kk + 1, lane);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            acc[i][j] = mma<Epi::kSwap>(af[c][i], bfr[c][j], acc[i][j]);
            const int q = (kk * TM + i) * TN + j;  // compile-time after unrolling
#pragma unroll
            for (int t = 0; t < kLoads; ++t)
              if (copy_slot(t) == q) {
                __builtin_amdgcn_sched_barrier(0);
                issue_copy(t, kt + NS - 1, wr);
                __builtin_amdgcn_sched_barrier(0);
              }
          }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    rd = rd + 1 == NS ? 0 : rd + 1;
    wr = wr + 1 == NS ? 0 : wr + 1;
  }
  if constexpr (!ROT) wait_vmcnt<0>();  // the trailing dummy copies must have landed before LDS is reused
  lds_barrier();                        // all waves are done with the last stage
  if constexpr (kRowStores) {
    if (whole) {
      if constexpr (!ROT) row_inputs.load(epi, m0 + wm, n0 + wn, lane);
      // where the whole wave tiles do not fit the LDS together (256x256): one 32-row block of every wave at a time
      constexpr int TB = NW * wave_epilogue_bytes<TM, TN>() <= 160 * 1024 ? TM : 1;
      float* wave_lds = reinterpret_cast<float*>(lds_raw) + wave * (wave_epilogue_bytes<TB, TN>() / 4);
      WaveSums<TM, TN, Epi> sums;
#pragma unroll
      for (int i = 0; i < TM; i += TB)
        store_blocks_coalesced<TB>(acc, i, epi, row_inputs, sums, m0 + wm, n0 + wn, lane, wave_lds);
      sums.store(epi, m0 + wm, n0 + wn, lane);
      return;
    }
  }
  store_tiles<TM, TN>(acc, epi_of_split(epi, split), m0 + wm, n0 + wn, M, N, lane);
}

// ---- few output tiles ---------------------------------------------------------------------------
// Forward products whose 64 x 64 tiles leave most CUs idle: 32 x 32 outputs per workgroup, a quarter of the bytes per CU.  All four
// waves copy, each every fourth k tile into stages of its own.  Workgroups of one column of tiles, which read the same rows
// of W, sit on one XCD.
// CHAIN: the first wave multiplies, all k in ascending order, the bits of every other tile.  Bound by the chain of matrix instructions, about 40 ns each, so the barrier behind which a round of four tiles may be read sits in front
// of the last products of the round before, and a tile's fragments are read under the products of the one before it.
// Otherwise each wave multiplies the tiles it has copied and waits for nobody until the four sums meet in LDS, in a fixed order:
// bound by what a CU fetches from the L2, 80 GB/s.  The sums are no further off fp64 (four shorter chains), but not the bits of the
// other tiles: two steps of a bottleneck net later, through normalisations and ReLUs, outputs were 3 % off the others'.
// us on 64 x 64 tiles, in chains, and in four parts: 64 x 512 x 512 5.9, 4.2, 3.8; 100 x 2000 x 2000 9.8, 8.6, 6.1; 512 x 512
// over 2048 9.8, 8.4, 6.4; 64 x 4096 x 4096 15.2, 13.2, 8.8.
template <bool CHAIN, class Epi>
__global__ __launch_bounds__(256) void gemm_bf16_skinny_kernel(int M, int N, int K, const uint16_t* __restrict__ A, int lda,
                                                               const uint16_t* __restrict__ B, int ldb, Epi epi, int tiles_m, int tiles,
                                                               SideCopy side) {
  constexpr int BM = 32, NS = 3, NW = 4, KK = DBK / 16;
  using T = RowDma<32, 1>;
  constexpr int kStageBytes = 2 * T::kBytes, kCopies = 2 * T::kPerWave, kPitch = 36;
  static_assert(BM * kPitch * 4 <= NS * kStageBytes, "a wave's sums go where its stages were");
  extern __shared__ __attribute__((aligned(16))) uint16_t lds_raw[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < side.nvec; i += (size_t)gridDim.x * 256) side.dst[i] = side.src[i];
  const int at = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (at >= tiles) return;
  const int m0 = at % tiles_m * BM, n0 = at / tiles_m * 32;
  A += (size_t)m0 * lda;
  B += (size_t)n0 * ldb;
  T ta, tb;
  ta.init(lda, 0, M - m0, 0, lane);
  tb.init(ldb, 0, N - n0, 0, lane);
  const int KT = (K + DBK - 1) / DBK, last_k = K - (KT - 1) * DBK;
  const int rounds = (KT + NW - 1 - (CHAIN ? 0 : wave)) / NW;  // otherwise: of this wave, perhaps none
  auto stage = [&](int i, int w) { return (w * NS + i % NS) * kStageBytes; };
  const uint32_t lds_base = lds_addr_of(lds_raw);
  // k tile NW * i + wave into the wave's stage of round i; past the end (CHAIN) the last tile again, which is not used
  auto issue = [&](int i) {
    const int tile = min(NW * i + wave, KT - 1);
    const uint32_t dst = lds_base + stage(i, wave);
    const uint16_t *pa = A + (size_t)tile * DBK, *pb = B + (size_t)tile * DBK;
#pragma unroll
    for (int t = 0; t < T::kPerWave; ++t) {
      if (tile == KT - 1 && last_k < DBK) {
        ta.issue_one_of(last_k, t, dst, pa, 0, lane);
        tb.issue_one_of(last_k, t, dst + T::kBytes, pb, 0, lane);
      } else {
        ta.issue_one(t, dst, pa, 0);
        tb.issue_one(t, dst + T::kBytes, pb, 0);
      }
    }
  };
  floatx16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  bf16x8 fa[2][KK], fb[2][KK];
  auto fetch = [&](int i, int w, int buf) {
    const uint16_t *pa = lds_raw + stage(i, w) / 2, *pb = pa + T::kBytes / 2;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      fa[buf][kk] = T::frag(pa, 0, kk, lane);
      fb[buf][kk] = T::frag(pb, 0, kk, lane);
    }
    if constexpr (CHAIN) __builtin_amdgcn_sched_barrier(0);
  };
  auto multiply = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) acc = mma<Epi::kSwap>(fa[buf][kk], fb[buf][kk], acc);
    if constexpr (CHAIN) __builtin_amdgcn_sched_barrier(0);
  };
  auto wait_for = [&](int i) {  // this wave's tile of round i has landed, that of the next one may be in flight
    if (i + 1 < rounds) wait_vmcnt<kCopies>();
    else wait_vmcnt<0>();
  };
  if (rounds > 0) issue(0);
  if (rounds > 1) issue(1);
  if constexpr (CHAIN) {
    auto arrive = [&](int i) {
      wait_for(i);
      lds_barrier();  // every wave's tile has landed, and all of the round before has been read
      if (i + NS - 1 < rounds) issue(i + NS - 1);
    };
    arrive(0);
    if (wave == 0) {
      fetch(0, 0, 0);
      for (int i = 0; i < rounds; ++i) {
        const int here = KT - NW * i;  // tiles of this round, if fewer than NW
#pragma unroll
        for (int w = 0; w < NW - 1; ++w) {
          fetch(i, w + 1, (w + 1) & 1);
          if (w < here) multiply(w & 1);
        }
        if (i + 1 < rounds) {
          arrive(i + 1);
          fetch(i + 1, 0, 0);
        }
        if (NW - 1 < here) multiply((NW - 1) & 1);
      }
    } else {
      for (int i = 1; i < rounds; ++i) arrive(i);
    }
    lds_barrier();  // the stages are dead
  } else {
    for (int i = 0; i < rounds; ++i) {
      wait_for(i);
      fetch(i, wave, 0);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if (i + NS - 1 < rounds) issue(i + NS - 1);  // into the stage that was read a round ago
      multiply(0);
    }
  }
  // the transposed blocks, row by row, each wave's over its own stages; then every thread takes four columns of a row
  if (!CHAIN || wave == 0) {
    float* mine = reinterpret_cast<float*>(lds_raw + stage(0, wave) / 2) + (lane & 31) * kPitch + 4 * (lane >> 5);
#pragma unroll
    for (int g = 0; g < 4; ++g) *reinterpret_cast<float4*>(mine + 8 * g) = make_float4(acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]);
  }
  lds_barrier();
  const int row = threadIdx.x >> 3, col = (threadIdx.x & 7) * 4;
  auto part = [&](int w) { return *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(lds_raw + stage(0, w) / 2) + row * kPitch + col); };
  float4 v = part(0);
  if constexpr (!CHAIN) {
    const float4 b = part(1), c = part(2), d = part(3);
    v = make_float4((v.x + b.x) + (c.x + d.x), (v.y + b.y) + (c.y + d.y), (v.z + b.z) + (c.z + d.z), (v.w + b.w) + (c.w + d.w));
  }
  if (m0 + row < M && n0 + col < N) epi.quad(m0 + row, n0 + col, min(4, N - n0 - col), v.x, v.y, v.z, v.w);
}

template <bool CHAIN, class Epi>
hipError_t launch_skinny(hipStream_t s, int M, int N, int K, const uint16_t* A, int lda, const uint16_t* B, int ldb, const Epi& epi,
                         SideCopy side) {
  static_assert(Epi::kSwap, "four columns per lane");
  constexpr int lds_bytes = 4 * 3 * 2 * RowDma<32, 1>::kBytes;
  auto kernel = gemm_bf16_skinny_kernel<CHAIN, Epi>;
  static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
  if (attr != hipSuccess) return attr;
  const int tiles_m = (M + 31) / 32, tiles = tiles_m * ((N + 31) / 32);
  hipLaunchKernelGGL(kernel, dim3((tiles + 7) / 8 * 8), dim3(256), lds_bytes, s, M, N, K, A, lda, B, ldb, epi, tiles_m, tiles, side);
  return hipGetLastError();
}

// Where a product takes the kernel above: as long as every tile has a CU of its own.  With two rounds of tiles it is behind the
// 64 x 64 ones (512 x 1024 x 1024 7.6 and 7.4 us, 256 x 2000 x 2000 10.6 and 9.6).  64 x 32 tiles in four parts would be ahead alone
// (512 x 1024 x 1024 6.2, 128 x 4096 x 4096 15.4 -> 12.0) but not beside other kernels, with 147 KB of LDS each: a stage of width 4096,
// micro-batches of 128 on two streams, 332 -> 352 us a step.
inline bool few_tiles(int M, int N) { return (long)((M + 31) / 32) * ((N + 31) / 32) <= 256; }

// Operands the direct-to-LDS kernel takes: 16-byte aligned with rows of whole 16-byte chunks (of at least one, along the
// rows of an operand staged [k][row]), 32-bit byte offsets inside a tile (of at most 384 rows or 64 k values).  Offsets from
// the start of the operand left those of 2 GiB and more to the register-staged kernel: forward, backward and update of
// 262144 x 4096 x 4096 took 46.5 ms there, 21.6 ms here.
inline bool dma_ok(int M, int N, int K, int lda, int ldb, bool a_col, bool b_col) {
  if (((a_col ? M : K) | (b_col ? N : K) | lda | ldb) & 7) return false;
  auto tile_bytes = [](int rows, int ld) { return (size_t)std::min(rows, 384) * ld * 2; };
  return tile_bytes(a_col ? K : M, lda) < (1ull << 31) && tile_bytes(b_col ? K : N, ldb) < (1ull << 31);
}

template <int BM, int BN, int WGM, int WGN, int NS, bool A_COL, bool B_COL, bool LEAN, bool ROT, bool TAIL, class Epi>
hipError_t launch_dma(hipStream_t s, int M, int N, int K, const uint16_t* A, int lda, const uint16_t* B, int ldb,
                      const Epi& epi, SideCopy side, int per) {
  constexpr int NW = WGM * WGN;
  using AT = typename DmaSel<BM, NW, A_COL>::type;
  using BT = typename DmaSel<BN, NW, B_COL>::type;
  constexpr size_t stage_bytes = (size_t)NS * (AT::kBytes + BT::kBytes);
  constexpr size_t epi_whole = (size_t)NW * wave_epilogue_bytes<BM / WGM / 32, BN / WGN / 32>();
  constexpr size_t epi_rows = (size_t)NW * wave_epilogue_bytes<1, BN / WGN / 32>();  // one 32-row block per wave
  constexpr bool epi_lds = Epi::kSwap && 64 % (4 * (BN / WGN / 32)) == 0;
  constexpr size_t epi_bytes = !epi_lds ? 0 : epi_whole <= 160 * 1024 ? epi_whole : epi_rows;  // tiles turned through LDS
  constexpr size_t lds_bytes = stage_bytes > epi_bytes ? stage_bytes : epi_bytes;
  static_assert(lds_bytes <= 160 * 1024, "stages do not fit the LDS of a CU");
  auto kernel = gemm_bf16_dma_kernel<BM, BN, WGM, WGN, NS, A_COL, B_COL, Epi, LEAN, ROT, TAIL>;
  if (lds_bytes > 64 * 1024) {
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (attr != hipSuccess) return attr;
  }
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  const int ranges = (k_tiles(K) + per - 1) / per;
  // Uneven patches save what arrives per k step, so little of a short contraction on the smallest tiles, and of a short weight gradient,
  // which writes fp32: 64 x 64 tiles are 0.99 of the time below 512 values, with one in thirteen 3 % or more behind, 0.986 from there
  // on and 0.94 from 1024 on; weight gradients 1.01 below 1024, up to 1 us of 9 behind, and 0.98 above.
  const bool short_k = K < (A_COL ? 1024 : BM * BN == 64 * 64 ? 512 : 0);
  const TileMap map = ranges > 1 ? TileMap{tiles_m, tiles_n, 0, 0, 0, 0}
                      : short_k  ? make_tile_map(tiles_m, tiles_n)
                                 : make_uneven_tile_map(tiles_m, tiles_n, BM, BN);
  hipLaunchKernelGGL(kernel, dim3(map.grid(), ranges), dim3(64 * NW), lds_bytes, s, M, N, K, per, A,
                     lda, B, ldb, epi, map, side);
  return hipGetLastError();
}

// Tile choice: the tile that needs the least time on 256 CUs, taken as (rounds of 256 workgroups) x (tile area) x (k tiles
// of a range) / (rate the tile sustains relative to the largest one): large tiles move less data per flop, but a last round
// that fills a fraction of the chip costs a whole round -- the 6144 x 2048 weight gradient of a fused QKV projection is 1.5
// rounds of 256x128 tiles, 192 tiles of 256x256 and exactly 256 tiles of 384x128 (51 us against 65 us and 57 us at 2048
// rows).  The 384-wide tiles serve the fp32-output product only (three 32-wide blocks per wave row do not fit the 16-byte
// row stores of the bf16 epilogues) and only shapes they divide.
enum Tile { T256x256, T384x128, T128x384, T256x128, T128x128, T128x64, T64x64 };
struct TileCost {
  Tile t;
  int bm, bn, rate;  // rate in per cent of the 256x256 tile's
  bool wgrad_only;
};
constexpr TileCost kTiles[] = {{T256x256, 256, 256, 100, false}, {T384x128, 384, 128, 88, true},  {T128x384, 128, 384, 88, true},
                               {T256x128, 256, 128, 88, false},  {T128x128, 128, 128, 78, false}, {T128x64, 128, 64, 62, false},
                               {T64x64, 64, 64, 45, false}};

inline long blocks_of(const TileCost& t, int M, int N) { return (long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn); }

Tile pick(int M, int N, bool wgrad) {
  Tile best = T64x64;
  long best_cost = -1;
  for (const TileCost& t : kTiles) {
    if (t.wgrad_only && !(wgrad && M % t.bm == 0 && N % t.bn == 0)) continue;
    const long cost = (blocks_of(t, M, N) + 255) / 256 * t.bm * t.bn * 100 / t.rate;
    if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = t.t; }
  }
  return best;
}

// Tile of a weight gradient and k tiles per range of its contraction (the rows of the mini-batch).  Where the output has too
// few tiles to fill the chip, it is formed over as many ranges as give every CU a workgroup, at least 8 k tiles each (a
// 64 x 64 gradient over the 131072 pixels of 16x16 maps is one tile and 2048 k tiles), and small tiles that fill it
// unsplit give way to ranges of larger ones where that takes less time: a k tile of a 256x256 tile takes 1.66 us (32768
// rows), of the others by their rates, and the ranges cost a launch (3 us) and their fp32 partial sums at 4 TB/s.  Ranges
// are formed on the three square tiles only: the rates of the other four lie between theirs, and each would be two more
// kernels for the partial sums; how they compare is not measured.
// 2048 x 512 and 1536 x 512 over 6400 rows: 64x64 tiles fill the chip but wait for memory (34 us), 128x128 ones over four and
// five ranges do less of it: two decoder blocks of width 512 1.087 -> 1.039 ms; 2048 x 2048 over 32768 rows, 128x128 tiles
// before, 256x256 over four ranges now: decoder block of width 2048 10.52 -> 10.45 ms.
struct WgradPlan { Tile tile; int per; };
WgradPlan wgrad_plan(int M, int N, int K, bool dma) {
  const int kt = k_tiles(M);
  if (!dma) {
    const long blocks = (long)((N + 63) / 64) * ((K + 63) / 64);
    const int ranges = (int)std::min<long>(256 / blocks, kt / 8);
    return {T64x64, ranges > 1 ? (kt + ranges - 1) / ranges : kt};
  }
  auto k_tile_us = [](const TileCost& t) { return 1.66 * t.bm * t.bn / 65536 * 100 / t.rate; };
  WgradPlan best{pick(N, K, true), kt};
  double best_us = -1;
  for (const TileCost& t : kTiles)
    if (t.t == best.tile) best_us = (double)((blocks_of(t, N, K) + 255) / 256) * k_tile_us(t) * kt;
  for (const TileCost& t : kTiles) {
    if (t.t != T256x256 && t.t != T128x128 && t.t != T64x64) continue;
    const int ranges = (int)std::min<long>(256 / blocks_of(t, N, K), kt / 8);
    if (ranges < 2) continue;
    const int per = (kt + ranges - 1) / ranges;
    const double us = k_tile_us(t) * per + 3 + (double)(ranges + 1) * N * K * 4 / 4e6;
    if (us < best_us) { best_us = us; best = {t.t, per}; }
  }
  return best;
}
inline int wgrad_ranges(int M, int N, int K) {
  const int per = wgrad_plan(M, N, K, dma_ok(N, K, M, N, K, true, true)).per;
  return (k_tiles(M) + per - 1) / per;
}

inline bool aligned(int bytes, const void* a, const void* b = nullptr, const void* c = nullptr) {
  return (((uintptr_t)a | (uintptr_t)b | (uintptr_t)c) & (bytes - 1)) == 0;
}

// per: k tiles per contraction range
template <bool A_COL, bool B_COL, bool TAIL, class Epi>
hipError_t run_dma(Tile tile, hipStream_t s, int M, int N, int K, const uint16_t* A, int lda, const uint16_t* B, int ldb,
                   const Epi& e, SideCopy side, int per) {
  switch (tile) {
    case T256x256: return launch_dma<256, 256, 2, 4, 2, A_COL, B_COL, false, true, TAIL>(s, M, N, K, A, lda, B, ldb, e, side, per);
    case T256x128: return launch_dma<256, 128, 4, 2, 3, A_COL, B_COL, false, true, TAIL>(s, M, N, K, A, lda, B, ldb, e, side, per);
    case T384x128:
      if constexpr (A_COL) return launch_dma<384, 128, 4, 2, 2, A_COL, B_COL, false, true, TAIL>(s, M, N, K, A, lda, B, ldb, e, side, per);
      break;
    case T128x384:
      if constexpr (A_COL) return launch_dma<128, 384, 2, 4, 2, A_COL, B_COL, false, true, TAIL>(s, M, N, K, A, lda, B, ldb, e, side, per);
      break;
    case T128x128: return launch_dma<128, 128, 2, 2, 3, A_COL, B_COL, false, true, TAIL>(s, M, N, K, A, lda, B, ldb, e, side, per);
    case T128x64: return launch_dma<128, 64, 2, 2, 4, A_COL, B_COL, true, false, TAIL>(s, M, N, K, A, lda, B, ldb, e, side, per);
    case T64x64: return launch_dma<64, 64, 2, 2, 4, A_COL, B_COL, true, false, TAIL>(s, M, N, K, A, lda, B, ldb, e, side, per);
  }
  return hipErrorInvalidValue;
}

// 64x64 tiles, or 128x64 ones where those still fill the chip half
template <bool A_COL, bool B_COL, class Epi>
hipError_t run_any(hipStream_t s, int M, int N, int K, const uint16_t* A, int lda, const uint16_t* B, int ldb, const Epi& e) {
  const int per = k_tiles(K);
  if ((long)((M + 127) / 128) * ((N + 63) / 64) >= 128)
    return launch_any<128, 64, 2, 2, A_COL, B_COL>(s, M, N, K, A, lda, B, ldb, e, per);
  return launch_any<64, 64, 2, 2, A_COL, B_COL>(s, M, N, K, A, lda, B, ldb, e, per);
}

// dma: the operands suit the direct-to-LDS kernel
template <bool A_COL, bool B_COL, class Epi>
hipError_t run(bool dma, hipStream_t s, int M, int N, int K, const uint16_t* A, int lda, const uint16_t* B, int ldb, const Epi& e,
               SideCopy side = SideCopy{nullptr, nullptr, 0}) {
  const int per = k_tiles(K);
  if (dma && K % DBK) return run_dma<A_COL, B_COL, true>(pick(M, N, A_COL), s, M, N, K, A, lda, B, ldb, e, side, per);
  if (dma) return run_dma<A_COL, B_COL, false>(pick(M, N, A_COL), s, M, N, K, A, lda, B, ldb, e, side, per);
  return run_any<A_COL, B_COL>(s, M, N, K, A, lda, B, ldb, e);
}

}  // namespace

inline int store_width(const void* a, const void* b) { return aligned(16, a, b) ? 2 : aligned(8, a, b) ? 1 : 0; }

hipError_t mfma_fprop(hipStream_t s, int M, int N, int K, const uint16_t* x, const uint16_t* W, const float* bias,
                      int act, uint16_t* d_out, uint16_t* a_out, uint16_t* x_copy, const uint16_t* addend, int spread) {
  const bool fits = dma_ok(M, N, K, K, K, false, false) && aligned(16, W, x_copy);
  if (x_copy && !(fits && aligned(16, x))) {
    const hipError_t err = launch_copy(s, x, x_copy, (size_t)M * K * 2);
    if (err != hipSuccess) return err;
    if (fits) x = x_copy;  // an input that is not aligned: its copy is, and the direct-to-LDS kernel takes that
  }
  const bool dma = fits && aligned(16, x);
  // whole 16-byte units with dma
  const SideCopy side{(const uint4*)x, (uint4*)x_copy, dma && x_copy && x != x_copy ? (size_t)M * K / 8 : 0};
  const int wide = store_width(d_out, a_out);
  // contractions that are no multiple of 8 ran on fp32 FMAs with GELU from erff, and keep it
  if (K % 8) return run_any<false, false>(s, M, N, K, x, K, W, K, EpiFpropExact{bias, d_out, a_out, act, N, nullptr, wide});
  auto product = [&](const auto& e) {
    if (dma && spread == SPREAD_PARTS && few_tiles(M, N)) return launch_skinny<false>(s, M, N, K, x, K, W, K, e, side);
    if (dma && spread == SPREAD_CHAINS && few_tiles(M, N)) return launch_skinny<true>(s, M, N, K, x, K, W, K, e, side);
    return run<false, false>(dma, s, M, N, K, x, K, W, K, e, side);
  };
  if (addend) return product(EpiFpropAdd{bias, d_out, a_out, act, N, addend, wide});
  return product(EpiFprop{bias, d_out, a_out, act, N, nullptr, wide});
}

int mfma_dgrad_sum_rows(int M, int K) {
  const Tile tile = pick(M, K, false);
  for (const TileCost& t : kTiles)
    if (t.t == tile && M % t.bm == 0 && K % t.bn == 0)
      return worthwhile_sum_rows(ELT_BF16, M, tile == T256x256 ? 128 : tile == T64x64 ? 32 : 64);  // rows of a wave tile
  return 0;
}

hipError_t mfma_dgrad(hipStream_t s, int M, int N, int K, const uint16_t* dz, const uint16_t* Wb,
                      const uint16_t* d_prev, uint16_t* out, int relu_mask, float* sums, int* sum_rows) {
  // out[M x K] = dz[M x N] . Wb[N x K]: GEMM (M, K, contraction N)
  const bool dma = dma_ok(M, K, N, N, K, false, true) && aligned(16, dz, Wb);
  EpiDgrad e{d_prev, out, K, relu_mask, store_width(d_prev, out)};
  if (sums) {
    *sum_rows = dma && e.wide == 2 ? mfma_dgrad_sum_rows(M, K) : 0;
    if (*sum_rows) e.sums = sums;
  }
  return run<false, true>(dma, s, M, K, N, dz, N, Wb, K, e);
}

size_t mfma_wgrad_scratch_floats(int M, int N, int K) {
  const int ranges = wgrad_ranges(M, N, K);
  return ranges > 1 ? (size_t)ranges * N * K : 0;
}

hipError_t mfma_wgrad(hipStream_t s, int M, int N, int K, const uint16_t* dz, const uint16_t* x, float* gW, float* partial) {
  // gW[N x K] = dz^T[N x M] . x[M x K]: GEMM (N, K, contraction M)
  const bool fits = dma_ok(N, K, M, N, K, true, true);
  const bool dma = fits && aligned(16, dz, x);
  const WgradPlan plan = wgrad_plan(M, N, K, fits);
  const int per = plan.per, ranges = (k_tiles(M) + per - 1) / per;
  if (!partial || ranges == 1) return run<true, true>(dma, s, N, K, M, dz, N, x, K, EpiWgrad{gW, K});
  const EpiWgradSplit e{partial, K, (size_t)N * K};
  const SideCopy none{nullptr, nullptr, 0};
  auto split = [&](auto tail) {
    constexpr bool T = decltype(tail)::value;
    switch (plan.tile) {
      case T256x256: return launch_dma<256, 256, 2, 4, 2, true, true, false, true, T>(s, N, K, M, dz, N, x, K, e, none, per);
      case T128x128: return launch_dma<128, 128, 2, 2, 3, true, true, false, true, T>(s, N, K, M, dz, N, x, K, e, none, per);
      default: return launch_dma<64, 64, 2, 2, 4, true, true, true, false, T>(s, N, K, M, dz, N, x, K, e, none, per);
    }
  };
  const hipError_t err = !dma        ? launch_any<64, 64, 2, 2, true, true>(s, N, K, M, dz, N, x, K, e, per)
                         : M % DBK ? split(std::true_type{})
                                   : split(std::false_type{});
  if (err != hipSuccess) return err;
  return launch_sum_partials(s, (size_t)N * K, ranges, partial, gW);
}

}  // namespace tp
