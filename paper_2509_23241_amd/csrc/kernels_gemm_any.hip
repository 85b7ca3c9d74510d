// Matrix-core GEMMs for whatever the tuned bf16 kernels do not take: every product of the fp32 mode, dense and
// convolution, and the bf16 convolutions of any kernel size, image size and channel count that is a multiple of 8.
//
// Forward products and input gradients keep the arithmetic of a plain fp32 loop: every output is ONE chain of fused
// multiply-adds over the contraction index in ascending order (v_mfma_f32_16x16x4_f32 adds its four products one after
// the other, lowest k first, rounding each time; tests/test_gpu_gemm_any.py holds dense layers and convolutions to such a
// chain bit for bit).  What feeds a ReLU or a pooling is therefore the same to the last bit whatever tile it was formed
// in, and the same as the bounds-checked FMA kernel of kernels_conv.hip gives.  That is a choice, made so that results
// did not move when these kernels replaced that one; the tuned bf16 kernels sum in the order of their own instructions.  bf16 operands are widened on their way out of LDS.  Weight gradients are sums over thousands of
// rows, whose order is not kept: they may be formed over several row ranges, in bf16 with v_mfma_f32_16x16x32_bf16.
//
// One kernel template; what differs between the products is where the 16-byte chunks of an operand's k tile come from
// (the loaders below).  A k tile is 128 bytes of the contraction index per row: 32 fp32 or 64 bf16 values.  Copies go
// global -> LDS without registers, each lane with an address of its own: positions outside the image and k values past
// the end of the contraction read a block of zeros, rows past the edge repeat the last row (computed, never stored).
// fp32 operands whose rows are no whole 16-byte units are copied word by word (VEC = 1).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "conv.h"
#include "device_utils.h"
#include "gemm_any.h"
#include "kernels.h"
#include "mfma_common.h"

namespace tp {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// ---- LDS stages --------------------------------------------------------------------------------
// k-contiguous operand: [R rows][8 chunks of 16 bytes], chunk c of row r in slot c ^ ((r / 2) % 8): the 16 rows of a
// fragment read fall into different banks.
// k-strided operand: [k][R rows], chunks of a k row XORed by a function of k chosen so that the k rows one fragment
// read touches at once lie in different banks (as far as the row is long enough).
template <class T>
struct Elem;
template <>
struct Elem<float> {
  static constexpr int kChunk = 4;  // values per 16 bytes
};
template <>
struct Elem<uint16_t> {
  static constexpr int kChunk = 8;
};
template <class T>
constexpr int kTileK = 8 * Elem<T>::kChunk;  // k values of one stage

// How a product is summed: Chain = one fp32 chain per output in ascending k, Free = bf16 matrix instructions
struct Chain {};
struct Free {};

template <class T, class Sum, int R>
__device__ __forceinline__ int col_swizzle(int k) {
  constexpr int chunks = R * (int)sizeof(T) / 16;  // per k row
  if constexpr (sizeof(T) == 4) {  // a read: 64 bytes of rows 4 m + g, g = 0 .. 3
    return chunks >= 16 ? 4 * (k & 3) : 4 * ((k >> 1) & 1);
  } else if constexpr (__is_same(Sum, Chain)) {  // 32 bytes of rows 4 m + g
    return chunks >= 16 ? 2 * (k & 3) : chunks >= 8 ? 2 * ((k >> 1) & 1) : 0;
  } else {  // 32 bytes of rows 32 s + 8 g + 0 .. 3; half a wave (two values of g) at a time
    const int hi = 2 * ((k >> 3) & 1);
    return chunks >= 16 ? (4 * (k & 3)) ^ hi : chunks >= 8 ? (4 * ((k >> 1) & 1)) ^ hi : hi;
  }
}

// What one side of the matrix instructions needs for a step of 32 k values.  Lane (i, g) = (lane % 16, lane / 16) holds
//   Chain: k = 4 m + g of row i for m = 0 .. 7 (instruction m covers 4 m .. 4 m + 3);  Free: k = 8 g .. 8 g + 7 of row i.
template <class Sum>
struct Frag;
template <>
struct Frag<Chain> {
  float v[8];
};
template <>
struct Frag<Free> {
  bf16x8 v;
};
template <class T>
constexpr int kSteps = kTileK<T> / 32;

// A fragment is read in kParts<Sum> parts, one LDS instruction (two for a transposed one) each, so that the reads of the
// next step can go out one by one between the matrix instructions of the current one.
template <class Sum>
constexpr int kParts = __is_same(Sum, Chain) ? 8 : 1;

template <class T, class Sum, int R>
__device__ __forceinline__ void row_part(Frag<Sum>& f, const char* lds, int rbase, int step, int lane, int m) {
  const int r = rbase + (lane & 15), g = lane >> 4;
  const char* row = lds + r * 128;
  const int swz = (r >> 1) & 7;
  if constexpr (__is_same(Sum, Free)) {
    f.v = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(row + (((4 * step + g) ^ swz) << 4)));
  } else if constexpr (sizeof(T) == 4) {
    f.v[m] = *reinterpret_cast<const float*>(row + ((m ^ swz) << 4) + 4 * g);
  } else {
    f.v[m] = bf16_to_float(*reinterpret_cast<const uint16_t*>(row + (((4 * step + (m >> 1)) ^ swz) << 4) + 8 * (m & 1) + 2 * g));
  }
}

template <class T, class Sum, int R>
__device__ __forceinline__ void col_part(Frag<Sum>& f, const char* lds, int rbase, int step, int lane, int m) {
  const int i = lane & 15, g = lane >> 4;
  if constexpr (__is_same(Sum, Free)) {
    // ds_read_b64_tr_b16: lane s of a group of 16 points at 4 consecutive values of k row k0 + s/4 and receives rows
    // k0 .. k0+3 of column c0 + s
    const int k = 32 * step + 8 * g + (i >> 2);
    const int col = rbase + 4 * (i & 3);
    typedef __attribute__((address_space(3))) shortx4* lds_ptr;
    const char* lo = lds + k * (R * 2) + ((col >> 3) ^ col_swizzle<T, Sum, R>(k)) * 16 + (col & 7) * 2;
    const char* hi = lo + 4 * (R * 2);  // k + 4: the same swizzle
    const shortx4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(lo));
    const shortx4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(hi));
    f.v = __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
  } else {
    constexpr int C = Elem<T>::kChunk;
    const int r = rbase + i;
    const char* at = lds + g * (R * (int)sizeof(T)) + ((r / C) ^ col_swizzle<T, Sum, R>(g)) * 16 + (r % C) * (int)sizeof(T);
    // k = 32 step + 4 m + g: the swizzle depends on g alone
    f.v[m] = to_float(*reinterpret_cast<const T*>(at + (32 * step + 4 * m) * (R * (int)sizeof(T))));
  }
}

// acc += (A . B^T of part m), transposed: register r of a lane is column 4 (lane / 16) + r of row lane % 16
__device__ __forceinline__ void multiply(const Frag<Chain>& a, const Frag<Chain>& b, int m, floatx4& acc) {
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(b.v[m], a.v[m], acc, 0, 0, 0);
}
__device__ __forceinline__ void multiply(const Frag<Free>& a, const Frag<Free>& b, int, floatx4& acc) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b.v, a.v, acc, 0, 0, 0);
}

// ---- loaders -----------------------------------------------------------------------------------
// Where a lane's piece (one chunk, or one word with VEC = 1) of copy t lies in the stage: row and k of a k-contiguous
// stage, k and row of a k-strided one.
template <class T, int R, int NW, int VEC>
struct RowSpot {
  static constexpr int kPieceBytes = VEC * (int)sizeof(T);
  static constexpr int kPerRow = 128 / kPieceBytes;
  static constexpr int kInstr = R * kPerRow / 64;
  static constexpr int kPerWave = kInstr / NW;
  static_assert(kInstr % NW == 0 && kPerWave > 0, "copies do not divide among the waves");
  static __device__ __forceinline__ void at(int t, int wave, int lane, int& r, int& k) {
    const int flat = 64 * (wave + NW * t) + lane;
    r = flat / kPerRow;
    const int byte = (flat % kPerRow) * kPieceBytes;
    const int chunk = (byte >> 4) ^ ((r >> 1) & 7);
    k = chunk * Elem<T>::kChunk + (byte & 15) / (int)sizeof(T);
  }
};
template <class T, class Sum, int R, int NW, int VEC>
struct ColSpot {
  static constexpr int kPieceBytes = VEC * (int)sizeof(T);
  static constexpr int kPerK = R / VEC;
  static constexpr int kInstr = kTileK<T> * kPerK / 64;
  static constexpr int kPerWave = kInstr / NW;
  static_assert(kInstr % NW == 0 && kPerWave > 0, "copies do not divide among the waves");
  static __device__ __forceinline__ void at(int t, int wave, int lane, int& r, int& k) {
    const int flat = 64 * (wave + NW * t) + lane;
    k = flat / kPerK;
    const int byte = (flat % kPerK) * kPieceBytes;
    const int chunk = (byte >> 4) ^ col_swizzle<T, Sum, R>(k);
    r = chunk * Elem<T>::kChunk + (byte & 15) / (int)sizeof(T);
  }
};

// A matrix as it lies in memory.  Row: element (r, k) at base[r * ld + k];  Col: at base[k * ld + r].
struct DenseDesc {
  const void* base;
  int ld, rows, K;  // K: extent of the contraction; k >= K reads zero
};

template <class T, class Sum, int R, int NW, int VEC>
struct DenseRow {
  using Desc = DenseDesc;
  using Spot = RowSpot<T, R, NW, VEC>;
  static constexpr int kPerWave = Spot::kPerWave;
  const T* p[kPerWave];
  int k[kPerWave], K;
  __device__ __forceinline__ void init(const Desc& d, int r0, int wave, int lane) {
    K = d.K;
#pragma unroll
    for (int t = 0; t < kPerWave; ++t) {
      int r;
      Spot::at(t, wave, lane, r, k[t]);
      p[t] = (const T*)d.base + (size_t)min(r0 + r, d.rows - 1) * d.ld + k[t];
    }
  }
  using Tile = int;
  __device__ __forceinline__ Tile tile(int tile) const { return tile; }
  __device__ __forceinline__ void copy(int t, int tile, uint32_t lds) const {
    const int k0 = tile * kTileK<T>;
    dma_addr<Spot::kPieceBytes>(lds, k0 + k[t] < K ? (const char*)(p[t] + k0) : zero_chunk());
  }
  static __device__ __forceinline__ void part(Frag<Sum>& f, const char* lds, int rbase, int step, int lane, int m) {
    row_part<T, Sum, R>(f, lds, rbase, step, lane, m);
  }
};

template <class T, class Sum, int R, int NW, int VEC>
struct DenseCol {
  using Desc = DenseDesc;
  using Spot = ColSpot<T, Sum, R, NW, VEC>;
  static constexpr int kPerWave = Spot::kPerWave;
  const T* p[kPerWave];
  int k[kPerWave], K, ld;
  __device__ __forceinline__ void init(const Desc& d, int r0, int wave, int lane) {
    K = d.K;
    ld = d.ld;
#pragma unroll
    for (int t = 0; t < kPerWave; ++t) {
      int r;
      Spot::at(t, wave, lane, r, k[t]);
      p[t] = (const T*)d.base + (size_t)k[t] * d.ld + min(r0 + r, d.rows - VEC);
    }
  }
  using Tile = int;
  __device__ __forceinline__ Tile tile(int tile) const { return tile; }
  __device__ __forceinline__ void copy(int t, int tile, uint32_t lds) const {
    const int k0 = tile * kTileK<T>;
    dma_addr<Spot::kPieceBytes>(lds, k0 + k[t] < K ? (const char*)(p[t] + (size_t)k0 * ld) : zero_chunk());
  }
  static __device__ __forceinline__ void part(Frag<Sum>& f, const char* lds, int rbase, int step, int lane, int m) {
    col_part<T, Sum, R>(f, lds, rbase, step, lane, m);
  }
};

// The same for contractions of whole k tiles: a scalar base and 32-bit offsets that stay, so that a copy takes no vector
// instruction (next to fp32 matrix instructions those are not free, see below).  Rows (COL: k values) of a tile
// lie within 4 GiB.
template <class T, class Sum, int R, int NW, bool COL>
struct DenseWhole {
  static constexpr int VEC = Elem<T>::kChunk;
  using Desc = DenseDesc;
  using Row = RowSpot<T, R, NW, VEC>;
  using Col = ColSpot<T, Sum, R, NW, VEC>;
  struct Spot {
    static constexpr int kPieceBytes = 16;
  };
  static constexpr int kPerWave = COL ? Col::kPerWave : Row::kPerWave;
  const T* base;
  size_t step;
  uint32_t off[kPerWave];
  __device__ __forceinline__ void init(const Desc& d, int r0, int wave, int lane) {
    r0 = __builtin_amdgcn_readfirstlane(r0);
    base = (const T*)d.base + (COL ? (size_t)r0 : (size_t)r0 * d.ld);
    step = COL ? (size_t)kTileK<T> * d.ld : (size_t)kTileK<T>;
#pragma unroll
    for (int t = 0; t < kPerWave; ++t) {
      int r, k;
      if constexpr (COL) Col::at(t, wave, lane, r, k);
      else Row::at(t, wave, lane, r, k);
      const uint32_t row = min(r0 + r, d.rows - (COL ? VEC : 1)) - r0;
      off[t] = (COL ? (uint32_t)k * (uint32_t)d.ld + row : row * (uint32_t)d.ld + k) * (uint32_t)sizeof(T);
    }
  }
  using Tile = const T*;
  __device__ __forceinline__ Tile tile(int tile) const { return base + tile * step; }
  __device__ __forceinline__ void copy(int t, Tile tile, uint32_t lds) const { dma16(lds, tile, off[t]); }
  static __device__ __forceinline__ void part(Frag<Sum>& f, const char* lds, int rbase, int step, int lane, int m) {
    if constexpr (COL) col_part<T, Sum, R>(f, lds, rbase, step, lane, m);
    else row_part<T, Sum, R>(f, lds, rbase, step, lane, m);
  }
};

// Quotient and remainder by a divisor known on the host: n * ceil(2^32 / div) >> 32 is exact for every n with
// n * div < 2^32; mul = 0 where that does not cover the range (or div is 1): a division.
struct FastDiv {
  uint32_t mul, div;
  __device__ __forceinline__ void get(int n, int& q, int& r) const {
    q = mul ? (int)__umulhi((uint32_t)n, mul) : n / (int)div;
    r = n - q * (int)div;
  }
};

// Rows are the pixels of a grid [imgs][H][W]; k runs over (tap, channel).  Forward (DX = false): output pixels reading
// the input at S*(h, w) + tap - Pd.  Input gradient (DX = true): input pixels reading dz where (h, w) + Pd - tap is a
// whole output position.
struct GatherRowDesc {
  const void* base;  // [imgs][SH][SW][C]
  int rows, H, W;    // the grid the rows run over
  int SH, SW;        // the grid that is read
  int C, K;          // channels; kernel taps * C
  int S, Pd;
  FastDiv by_c, by_r;
};
template <class T, class Sum, int R, int NW, int VEC, bool DX>
struct GatherRow {
  using Desc = GatherRowDesc;
  using Spot = RowSpot<T, R, NW, VEC>;
  static constexpr int kPerWave = Spot::kPerWave;
  // A lane's copies lie in rows that are NW * 8 (or, word by word, NW * 2) apart, so with the swizzle repeating every 16
  // rows they have one k value (two) between them: the division into tap and channel is done once per tile and value.
  static constexpr int kKinds = VEC == 1 ? 2 : 1;
  static_assert(NW % 4 == 0, "which copies share a k value");
  Desc d;
  const T* image[kPerWave];
  int hw[kPerWave], k[kKinds];
  __device__ __forceinline__ void init(const Desc& desc, int r0, int wave, int lane) {
    d = desc;
#pragma unroll
    for (int t = 0; t < kPerWave; ++t) {
      int r, kt;
      Spot::at(t, wave, lane, r, kt);
      if (t < kKinds) k[t] = kt;
      const int p = min(r0 + r, d.rows - 1);
      const int q = p / d.W, w = p - q * d.W, img = q / d.H, h = q - img * d.H;
      image[t] = (const T*)d.base + (size_t)img * d.SH * d.SW * d.C;
      hw[t] = DX ? (h + d.Pd) << 16 | (w + d.Pd) : (h * d.S) << 16 | (w * d.S);
    }
  }
  struct Tile {
    int kh[kKinds], kw[kKinds], c[kKinds];  // kh: out of every image where the k value is past the end
  };
  __device__ __forceinline__ Tile tile(int tile) const {
    Tile o;
#pragma unroll
    for (int i = 0; i < kKinds; ++i) {
      int tap;
      const int kk = tile * kTileK<T> + k[i];
      d.by_c.get(kk, tap, o.c[i]);
      d.by_r.get(tap, o.kh[i], o.kw[i]);
      if (!DX) {
        o.kh[i] -= d.Pd;
        o.kw[i] -= d.Pd;
      }
      if (kk >= d.K) o.kh[i] = 1 << 20;
    }
    return o;
  }
  __device__ __forceinline__ void copy(int t, const Tile& o, uint32_t lds) const {
    const int i = t % kKinds;
    int sh, sw;
    bool ok = true;
    if (DX) {
      sh = (hw[t] >> 16) - o.kh[i];
      sw = (hw[t] & 0xffff) - o.kw[i];
      if (d.S == 2) {
        ok = !((sh | sw) & 1);
        sh >>= 1;
        sw >>= 1;
      }
    } else {
      sh = (hw[t] >> 16) + o.kh[i];
      sw = (hw[t] & 0xffff) + o.kw[i];
    }
    ok = ok && (unsigned)sh < (unsigned)d.SH && (unsigned)sw < (unsigned)d.SW;
    dma_addr<Spot::kPieceBytes>(lds, ok ? (const char*)(image[t] + (uint32_t)((sh * d.SW + sw) * d.C + o.c[i])) : zero_chunk());
  }
  static __device__ __forceinline__ void part(Frag<Sum>& f, const char* lds, int rbase, int step, int lane, int m) {
    row_part<T, Sum, R>(f, lds, rbase, step, lane, m);
  }
};

// The weights of the input gradient: row n = input channel, k = (tap, output channel), element at
// base[co * taps * Cin + tap * Cin + n].
struct WeightColDesc {
  const void* base;
  int cin, taps, cout;
  FastDiv by_cout;
};
template <class T, class Sum, int R, int NW, int VEC>
struct WeightCol {
  using Desc = WeightColDesc;
  using Spot = ColSpot<T, Sum, R, NW, VEC>;
  static constexpr int kPerWave = Spot::kPerWave;
  Desc d;
  int n[kPerWave], k[kPerWave];
  __device__ __forceinline__ void init(const Desc& desc, int r0, int wave, int lane) {
    d = desc;
#pragma unroll
    for (int t = 0; t < kPerWave; ++t) {
      int r;
      Spot::at(t, wave, lane, r, k[t]);
      n[t] = min(r0 + r, d.cin - VEC);
    }
  }
  using Tile = int;
  __device__ __forceinline__ Tile tile(int tile) const { return tile; }
  __device__ __forceinline__ void copy(int t, int tile, uint32_t lds) const {
    int tap, co;
    d.by_cout.get(tile * kTileK<T> + k[t], tap, co);
    const T* at = (const T*)d.base + ((size_t)co * d.taps + tap) * d.cin + n[t];
    dma_addr<Spot::kPieceBytes>(lds, tap < d.taps ? (const char*)at : zero_chunk());
  }
  static __device__ __forceinline__ void part(Frag<Sum>& f, const char* lds, int rbase, int step, int lane, int m) {
    col_part<T, Sum, R>(f, lds, rbase, step, lane, m);
  }
};

// The input as the weight gradient reads it: row n = (tap, input channel), k = output pixel.
struct GatherColDesc {
  const void* base;  // [imgs][SH][SW][C]
  int SH, SW, C, K;  // K: output pixels
  int S, Pd, N;      // N: taps * C
  FastDiv by_c, by_r, by_w, by_h;  // by_w, by_h: the output grid
};
template <class T, class Sum, int R, int NW, int VEC>
struct GatherCol {
  using Desc = GatherColDesc;
  using Spot = ColSpot<T, Sum, R, NW, VEC>;
  static constexpr int kPerWave = Spot::kPerWave;
  Desc d;
  int c[kPerWave], dh[kPerWave], dw[kPerWave], k[kPerWave];
  __device__ __forceinline__ void init(const Desc& desc, int r0, int wave, int lane) {
    d = desc;
#pragma unroll
    for (int t = 0; t < kPerWave; ++t) {
      int r, tap, kh, kw;
      Spot::at(t, wave, lane, r, k[t]);
      d.by_c.get(min(r0 + r, d.N - VEC), tap, c[t]);
      d.by_r.get(tap, kh, kw);
      dh[t] = kh - d.Pd;
      dw[t] = kw - d.Pd;
    }
  }
  using Tile = int;
  __device__ __forceinline__ Tile tile(int tile) const { return tile; }
  __device__ __forceinline__ void copy(int t, int tile, uint32_t lds) const {
    const int p = tile * kTileK<T> + k[t];
    int q, img, h, w;
    d.by_w.get(p, q, w);
    d.by_h.get(q, img, h);
    const int sh = h * d.S + dh[t], sw = w * d.S + dw[t];
    const bool ok = p < d.K && (unsigned)sh < (unsigned)d.SH && (unsigned)sw < (unsigned)d.SW;
    const T* at = (const T*)d.base + ((size_t)(img * d.SH + sh) * d.SW + sw) * d.C + c[t];
    dma_addr<Spot::kPieceBytes>(lds, ok ? (const char*)at : zero_chunk());
  }
  static __device__ __forceinline__ void part(Frag<Sum>& f, const char* lds, int rbase, int step, int lane, int m) {
    col_part<T, Sum, R>(f, lds, rbase, step, lane, m);
  }
};

// ---- epilogues: four consecutive columns n .. n+3 (count of them inside the matrix) of row m ----
// vec: whole units of four values everywhere.
template <class T>
__device__ __forceinline__ void store4(T* p, const float (&v)[4]) {
  if constexpr (sizeof(T) == 4) *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  else *reinterpret_cast<uint2*>(p) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
}
// finish: the same with what the epilogue reads besides the product (input) in hand, so that a kernel can fetch it early.
template <class T>
struct EpiForward {
  static constexpr int kPartK = 0;
  static constexpr bool kSums = false;
  const float* bias;
  T *d_out, *a_out;
  int act, ldc, vec;
  __device__ __forceinline__ floatx4 input(int, int n, int count) const {
    floatx4 b;
#pragma unroll
    for (int j = 0; j < 4; ++j) b[j] = bias[j < count ? n + j : n];
    return b;
  }
  __device__ __forceinline__ void finish(int m, int n, int count, const floatx4& v, const floatx4& b) const {
    const size_t i = (size_t)m * ldc + n;
    float a[4], d[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float z = v[j] + b[j];
      a[j] = act_forward(z, act);
      d[j] = d_out ? act_derivative(z, act) : 0.f;
    }
    if (vec && count == 4) {
      if (d_out) store4(d_out + i, d);
      store4(a_out + i, a);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (j < count) {
          if (d_out) d_out[i + j] = from_float<T>(d[j]);
          a_out[i + j] = from_float<T>(a[j]);
        }
    }
  }
  __device__ __forceinline__ void quad(int m, int n, int count, const floatx4& v, int) const {
    finish(m, n, count, v, input(m, n, count));
  }
};
template <class T>
struct EpiInputGrad {
  static constexpr int kPartK = 0;
  const T* d_prev;  // saved act'(z) of the layer before, with relu_mask its ReLU output, or null
  T* out;
  int ldc, relu_mask, vec;
  float* sums = nullptr;  // column sums of what is stored, [every 16 rows][ldc], or null
  static constexpr bool kSums = true;
  __device__ __forceinline__ floatx4 input(int m, int n, int count) const {
    const size_t i = (size_t)m * ldc + n;
    floatx4 d;
#pragma unroll
    for (int j = 0; j < 4; ++j) d[j] = d_prev ? to_float(d_prev[j < count ? i + j : i]) : 0.f;
    return d;
  }
  // returns what was stored, zeros in the columns outside
  __device__ __forceinline__ floatx4 finish(int m, int n, int count, const floatx4& v, const floatx4& d) const {
    const size_t i = (size_t)m * ldc + n;
    float o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = !d_prev ? v[j] : relu_mask ? (d[j] > 0.f ? v[j] : 0.f) : v[j] * d[j];
    if (vec && count == 4) {
      store4(out + i, o);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (j < count) out[i + j] = from_float<T>(o[j]);
    }
    floatx4 kept;
#pragma unroll
    for (int j = 0; j < 4; ++j) kept[j] = j < count ? to_float(from_float<T>(o[j])) : 0.f;
    return kept;
  }
  __device__ __forceinline__ floatx4 quad(int m, int n, int count, const floatx4& v, int) const {
    return finish(m, n, count, v, input(m, n, count));
  }
  // the 16 rows m - m % 16 .. of columns n .. n+3: the lanes of a row of 16 have one each (rows outside: zeros)
  __device__ __forceinline__ void store_sums(int m, int n, int M, int N, floatx4 v) const {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = row_sum_ascending(v[j]);
    if (m % 16 == 0 && m < M)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (n + j < N) sums[(size_t)(m / 16) * ldc + n + j] = v[j];
  }
};
// fp32 partial result of contraction range `split`
struct EpiPartial {
  static constexpr int kPartK = 0;
  static constexpr bool kSums = false;
  float* out;
  int ldc, vec;
  size_t split_stride;
  __device__ __forceinline__ void quad(int m, int n, int count, const floatx4& v, int split) const {
    float* p = out + (size_t)split * split_stride + (size_t)m * ldc + n;
    if (vec && count == 4) {
      *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (j < count) p[j] = v[j];
    }
  }
};
// The same for convolutions, whose contraction runs over all pixels of a mini-batch: products of 256 pixels each are added
// up apart and then to one another.  The bounds-checked kernel before cut the pixels into ranges of 256 and up; with
// chains over the fewer and longer ranges of these kernels the gradients were up to 1.5 times further off fp64 (3x3 on 16 images
// of 32 x 32, 64 channels: 2.9e-7 -> 4.4e-7).
struct EpiPartialPixels : EpiPartial {
  static constexpr int kPartK = 256;
};
// ---- the kernel --------------------------------------------------------------------------------
// grid = (output tiles, contraction ranges of `per` k tiles each).  U k tiles are multiplied between two barriers; NS runs of U
// tiles are in LDS.  The fragments of a step are read between the matrix instructions of the step before it, and the
// barrier that opens a run stands before the last step of the run before, so that a wave that has its SIMD to itself
// waits for LDS nowhere.  Unrolled over the stages, since an LDS address formed at run time is a vector instruction, and
// those take their time from fp32 matrix instructions (below).
// Epi::kPartK: k values whose products are summed apart (0: all of them in one chain).
template <class T, class Sum, int BM, int BN, int WGM, int WGN, int NS, int U, class AL, class BL, class Epi>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_any_kernel(int M, int N, int KT, int per, typename AL::Desc ad,
                                                                  typename BL::Desc bd, Epi epi, TileMap map, SideCopy side) {
  constexpr int WM = BM / WGM, WN = BN / WGN, TM = WM / 16, TN = WN / 16, NW = WGM * WGN;
  constexpr int kABytes = BM * 128, kStage = (BM + BN) * 128;
  constexpr int kLoads = AL::kPerWave + BL::kPerWave;
  static_assert((NS - 1) * U * kLoads < 64, "too many copies in flight for vmcnt");
  extern __shared__ __attribute__((aligned(16))) char lds[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = (wave / WGN) * WM, wn = (wave % WGN) * WN;
  const int tiles = map.tiles_m * map.tiles_n;
  if ((int)blockIdx.x >= tiles) {
    // Workgroups behind the tiles copy.  Shared among the tiles' workgroups the copy added its own latency to theirs: 7.0 to
    // 8.4 us for 32 rows of 512 by 512, where a launch of its own takes 2.2 us.
    const size_t step = (size_t)(gridDim.x - tiles) * (64 * NW);
    for (size_t i = (size_t)(blockIdx.x - tiles) * (64 * NW) + threadIdx.x; i < side.nvec; i += step) side.dst[i] = side.src[i];
    return;
  }
  int tile_m, tile_n;
  map.get(blockIdx.x, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int first = blockIdx.y * per, last = min(KT, first + per) - 1;  // k tiles of this range (at least one)
  const uint32_t lds_base = lds_addr_of(lds);

  floatx4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  constexpr int kPart = Epi::kPartK / kTileK<T>;  // k tiles of one part
  static_assert(kPart % U == 0, "a part is whole runs of k tiles");
  floatx4 parts[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) parts[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto end_part = [&] {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        parts[i][j] += acc[i][j];
        acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
  };

  AL a;
  BL b;
  a.init(ad, m0, wave, lane);
  b.init(bd, n0, wave, lane);
  auto copy = [&](int q, const typename AL::Tile& at, const typename BL::Tile& bt, uint32_t dst) {
    if (q < AL::kPerWave) a.copy(q, at, dst + (wave + NW * q) * 64 * AL::Spot::kPieceBytes);
    else b.copy(q - AL::kPerWave, bt, dst + kABytes + (wave + NW * (q - AL::kPerWave)) * 64 * BL::Spot::kPieceBytes);
  };
#pragma unroll
  for (int st = 0; st < NS * U; ++st) {  // all stages; tiles past the end copy the last one again, so that their number is known
    const int t = min(first + st, last);
    const typename AL::Tile at = a.tile(t);
    const typename BL::Tile bt = b.tile(t);
#pragma unroll
    for (int q = 0; q < kLoads; ++q) copy(q, at, bt, lds_base + st * kStage);
  }
  constexpr int kRun = U * kSteps<T>;              // steps of a run
  constexpr int kMfmas = kParts<Sum> * TM * TN;    // matrix instructions of a step
  constexpr int kReads = kParts<Sum> * (TM + TN);  // fragment reads of a step
  static_assert(kRun % 2 == 0, "fragment buffers alternate with the steps");
  Frag<Sum> fa[2][TM], fb[2][TN];
  // read number x of the fragments of step q of the run in stage s
  auto fetch = [&](int s, int q, int x) {
    const char* la = lds + (s * U + q / kSteps<T>) * kStage;
    const int m = x / (TM + TN), r = x % (TM + TN), step = q % kSteps<T>;
    if (r < TM) AL::part(fa[q & 1][r], la, wm + 16 * r, step, lane, m);
    else BL::part(fb[q & 1][r - TM], la + kABytes, wn + 16 * (r - TM), step, lane, m);
  };
  wait_vmcnt<(NS - 1) * U * kLoads>();
  lds_barrier();  // the first run visible to all waves
#pragma unroll
  for (int x = 0; x < kReads; ++x) fetch(0, 0, x);
  // Step q of the run in stage s: its matrix instructions, between them the fragment reads of the next step and copies of the run
  // that replaces the one consumed last, kShare in each of kWindow steps, counted (w) from the one behind a barrier.
  // With two stages that run is waited for at the next barrier, so its copies go out in the first half of the time.
  constexpr int kWindow = NS > 2 ? kRun : __is_same(Sum, Free) ? 1 : (kRun + 1) / 2, kShare = (U * kLoads + kWindow - 1) / kWindow;
  auto copy_slot = [](int c) constexpr { return __is_same(Sum, Free) ? 0 : c * kMfmas / kShare; };
  int fill = last + 1;  // first k tile of that run (past the last: none)
  auto step = [&](int s, int q, int fill_stage, auto filling) {
    const int c0 = (q + 1) % kRun * kShare;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < kParts<Sum>; ++m)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          multiply(fa[q & 1][i], fb[q & 1][j], m, acc[i][j]);
          __builtin_amdgcn_sched_barrier(0);
          const int slot = (m * TM + i) * TN + j;
#pragma unroll
          for (int x = 0; x < kReads; ++x)
            if (x * kMfmas / kReads == slot) fetch(q == kRun - 1 ? (s + 1) % NS : s, (q + 1) % kRun, x);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (decltype(filling)::value) {
#pragma unroll
            for (int c = 0; c < kShare; ++c)
              if (copy_slot(c) == slot && c0 + c < U * kLoads) {
                const int t = min(fill + (c0 + c) / kLoads, last);
                copy((c0 + c) % kLoads, a.tile(t), b.tile(t), lds_base + (fill_stage * U + (c0 + c) / kLoads) * kStage);
              }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
  };
  for (int kt = first; kt <= last; kt += NS * U) {  // unrolled over the stages: their LDS addresses are constants
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int run = kt + s * U;
      if (run > last) break;  // wave uniform, as every condition here
#pragma unroll
      for (int q = 0; q < kRun; ++q) {
        if (U > 1 && run + q / kSteps<T> > last) break;  // a shorter last run
        if (q == kRun - 1) {
          // The last fragments of this run are in registers: its stage is free once every wave is here, and the first
          // fragments of the next run are read under the last matrix instructions of this one.
          // with all copies for NS - 1 runs ahead under way
          if (run == first || run + U * NS - 1 <= last) wait_vmcnt<(NS - 2) * U * kLoads>();
          else wait_vmcnt<0>();
          lds_barrier();
          fill = run + U * NS;
        }
        const int fill_stage = q == kRun - 1 ? s : (s + NS - 1) % NS;
        if ((q + 1) % kRun < kWindow && fill + (q + 1) % kRun * kShare / kLoads <= last) step(s, q, fill_stage, std::true_type{});
        else step(s, q, fill_stage, std::false_type{});
      }
      if constexpr (kPart > 0)
        if ((run + U - first) % kPart == 0) end_part();
    }
  }
  wait_vmcnt<0>();  // the trailing copies land before the LDS is given back
  if constexpr (kPart > 0) end_part();

#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + wm + 16 * i + (lane & 15);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + wn + 16 * j + 4 * (lane >> 4);
      if constexpr (Epi::kSums) {
        floatx4 o = {0.f, 0.f, 0.f, 0.f};
        if (m < M && n < N) o = epi.quad(m, n, min(4, N - n), acc[i][j], blockIdx.y);
        if (epi.sums) epi.store_sums(m, n, M, N, o);
      } else {
        if (m < M && n < N) epi.quad(m, n, min(4, N - n), kPart > 0 ? parts[i][j] : acc[i][j], blockIdx.y);
      }
    }
  }
}

template <class T, class Sum, int BM, int BN, int WGM, int WGN, int NS, int U, class AL, class BL, class Epi>
hipError_t launch_any(hipStream_t s, int M, int N, int KT, int splits, const typename AL::Desc& ad, const typename BL::Desc& bd,
                      const Epi& epi, const SideCopy& side) {
  constexpr size_t lds_bytes = (size_t)NS * U * (BM + BN) * 128;
  static_assert(lds_bytes <= 160 * 1024, "stages do not fit the LDS of a CU");
  auto kernel = gemm_any_kernel<T, Sum, BM, BN, WGM, WGN, NS, U, AL, BL, Epi>;
  if (lds_bytes > 64 * 1024) {
    static hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (attr != hipSuccess) return attr;
  }
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  const int per = (KT + splits - 1) / splits;
  const int ranges = (KT + per - 1) / per;  // every one of them has a tile to sum; ranges == splits by any_splits
  if (ranges != splits) return hipErrorInvalidValue;
  constexpr int kThreads = 64 * WGM * WGN;
  const unsigned copiers = (unsigned)std::min<size_t>((side.nvec + 4 * kThreads - 1) / (4 * kThreads), 64);
  hipLaunchKernelGGL(kernel, dim3(tiles_m * tiles_n + copiers, ranges), dim3(kThreads), lds_bytes, s, M, N, KT, per, ad, bd, epi,
                     make_tile_map(tiles_m, tiles_n), side);
  return hipGetLastError();
}

// ---- dense fp32 products of few tiles ------------------------------------------------------------
// Forward products and input gradients of whole k tiles, with rows of whole 16-byte units: the same chains as above, bit for
// bit.  Bound by the chain itself, one dependent v_mfma_f32_16x16x4_f32 per four k values, 32 cycles each.  fp32 matrix
// instructions run on the vector ALUs: between two of them an LDS read or a scalar instruction costs 1 to 3 cycles, a
// vector instruction 8 and more (timed in a chain of its own).  So a workgroup is ONE wave with a tile of 16 x 16, which waits
// for its own copies and for nobody; the copies take a scalar base and a constant offset per lane, and with the loop
// unrolled over the stages every LDS address is a constant register and an immediate.  No vector instruction is left in the loop:
// 41 cycles per matrix instruction, where four waves of a 32 x 32 tile with a barrier every four k tiles took 80.
// 32 x 512 x 512 7.1 -> 4.9 us, 128 x 1024 x 1024 11.5 -> 7.4, input gradient 128 x 512 x 512 7.3 -> 4.8.
// With two or four tiles per wave, for fewer bytes per product, the same three took 6.8, 10.6, 7.0 and 11.0, 18.2, 11.4 us.
constexpr int kWaveStages = 8;   // 32 KB; twelve of them: 5.2, 7.6, 5.0 us
constexpr int kWaveStage = 4096;  // 16 rows of 32 k values of each operand

// [16 rows][32 k], chunks swizzled as above
struct WaveRow {
  uint32_t off[2];  // bytes from the first row
  int at[8];        // LDS byte of k = 4 m + g of row i
  __device__ __forceinline__ void init(int ld, int r0, int rows, int lane) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int r = 8 * t + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
      off[t] = (uint32_t)(min(r0 + r, rows - 1) - r0) * (uint32_t)ld * 4 + c * 16;
    }
    const int i = lane & 15, g = lane >> 4;
#pragma unroll
    for (int m = 0; m < 8; ++m) at[m] = i * 128 + ((m ^ ((i >> 1) & 7)) << 4) + 4 * g;
  }
  static __device__ __forceinline__ size_t start(int ld, int r0) { return (size_t)r0 * ld; }
  static __device__ __forceinline__ size_t step(int) { return 32; }
  __device__ __forceinline__ float read(const char* stage, int m) const { return *reinterpret_cast<const float*>(stage + at[m]); }
};
// [32 k][16 rows]: the 64 lanes of a read lie side by side
struct WaveCol {
  uint32_t off[2];
  int at;
  __device__ __forceinline__ void init(int ld, int r0, int rows, int lane) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int k = 16 * t + (lane >> 2), c = lane & 3;
      off[t] = ((uint32_t)k * (uint32_t)ld + (uint32_t)(min(r0 + 4 * c, rows - 4) - r0)) * 4;
    }
    at = lane * 4;
  }
  static __device__ __forceinline__ size_t start(int, int r0) { return r0; }
  static __device__ __forceinline__ size_t step(int ld) { return (size_t)32 * ld; }
  __device__ __forceinline__ float read(const char* stage, int m) const {
    return *reinterpret_cast<const float*>(stage + at + m * 256);
  }
};

template <class F, int... U>
__device__ __forceinline__ void for_each_stage(const F& f, std::integer_sequence<int, U...>) {
  (f(std::integral_constant<int, U>{}), ...);
}

template <class AL, class BL, class Epi>
__global__ __launch_bounds__(64) void gemm_f32_wave_kernel(int M, int N, int KT, const float* __restrict__ A, int lda,
                                                           const float* __restrict__ B, int ldb, Epi epi, TileMap map,
                                                           SideCopy side) {
  constexpr int NS = kWaveStages, kCopies = 4;
  static_assert(NS % 2 == 0, "fragment buffers alternate with the stages");
  __shared__ __attribute__((aligned(16))) char lds[NS * kWaveStage];
  const int lane = threadIdx.x;
  const int tiles = map.tiles_m * map.tiles_n;
  if ((int)blockIdx.x >= tiles) {  // workgroups behind the tiles copy, as above
    const size_t step = (size_t)(gridDim.x - tiles) * 64;
    for (size_t i = (size_t)(blockIdx.x - tiles) * 64 + lane; i < side.nvec; i += step) side.dst[i] = side.src[i];
    return;
  }
  int tile_m, tile_n;
  map.get(blockIdx.x, tile_m, tile_n);
  const int m0 = __builtin_amdgcn_readfirstlane(tile_m) * 16, n0 = __builtin_amdgcn_readfirstlane(tile_n) * 16;
  const uint32_t lds_base = lds_addr_of(lds);

  AL a;
  BL b;
  a.init(lda, m0, M, lane);
  b.init(ldb, n0, N, lane);
  // row m, columns n .. n+3 of the output are this lane's; what the epilogue reads there is fetched before the products
  const int m = m0 + (lane & 15), n = n0 + 4 * (lane >> 4);
  const floatx4 input = epi.input(min(m, M - 1), min(n, N - 1), N - min(n, N - 1));
  const float* pa = A + AL::start(lda, m0);  // the next tile to be copied
  const float* pb = B + BL::start(ldb, n0);
  const size_t step_a = AL::step(lda), step_b = BL::step(ldb);
  auto copy = [&](int q, int stage) {
    const uint32_t dst = lds_base + stage * kWaveStage + q * 1024;
    if (q < 2) dma16(dst, pa, a.off[q]);
    else dma16(dst, pb, b.off[q - 2]);
  };

  // Tile t lies in stage (t + skip) % NS, so that the last tile is in the last stage: the end of the loop, with fewer and
  // fewer copies in flight, is unrolled with its waits.
  const int skip = (NS - KT % NS) % NS;
#pragma unroll
  for (int t = 0; t < NS - 1; ++t)
    if (t < KT) {
      const int stage = t + skip >= NS ? t + skip - NS : t + skip;
#pragma unroll
      for (int q = 0; q < kCopies; ++q) copy(q, stage);
      pa += step_a;
      pb += step_b;
    }
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
  float fa[2][8], fb[2][8];
  if (KT >= NS - 1) wait_vmcnt<(NS - 2) * kCopies>();
  else wait_vmcnt<0>();
  auto first = [&](auto buf) {  // the first tile's fragments, into the buffer of its stage
    const char* at = lds + skip * kWaveStage;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      fa[decltype(buf)::value][k] = a.read(at, k);
      fb[decltype(buf)::value][k] = b.read(at + 2048, k);
    }
  };
  if (skip & 1) first(std::integral_constant<int, 1>{});
  else first(std::integral_constant<int, 0>{});
  // The tile in stage u.  Between its instructions the fragments of the next tile are read, and the tile NS - 1 further on is
  // copied to the stage before this one, whose fragments the instructions of the tile before have taken.
  auto tile = [&](auto stage_u, auto copying, auto more) {
    constexpr int u = decltype(stage_u)::value, next = (u + 1) % NS;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[u & 1][k], fa[u & 1][k], acc, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (decltype(more)::value) {
        fa[next & 1][k] = a.read(lds + next * kWaveStage, k);
        fb[next & 1][k] = b.read(lds + next * kWaveStage + 2048, k);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (decltype(copying)::value)
        if (k % 2 == 0) {
          copy(k / 2, (u + NS - 1) % NS);
          __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (decltype(copying)::value) {
      pa += step_a;
      pb += step_b;
    }
  };
  auto all_stages = [&](int t0, auto last) {  // tile t0 in stage 0; tiles below zero are left out
    for_each_stage([&](auto stage_u) {
      constexpr int u = decltype(stage_u)::value;
      if (t0 + u < 0) return;
      if constexpr (!decltype(last)::value || u == 0) {
        wait_vmcnt<(NS - 3) * kCopies>();  // the next tile has landed
        tile(stage_u, std::true_type{}, std::true_type{});
      } else if constexpr (u < NS - 1) {
        wait_vmcnt<(NS - 2 - u) * kCopies>();
        tile(stage_u, std::false_type{}, std::true_type{});
      } else {
        tile(stage_u, std::false_type{}, std::false_type{});
      }
    }, std::make_integer_sequence<int, NS>{});
  };
  int t0 = -skip;
  for (; t0 + NS < KT; t0 += NS) all_stages(t0, std::false_type{});
  all_stages(t0, std::true_type{});
  if constexpr (Epi::kSums) {
    floatx4 o = {0.f, 0.f, 0.f, 0.f};
    if (m < M && n < N) o = epi.finish(m, n, min(4, N - n), acc, input);
    if (epi.sums) epi.store_sums(m, n, M, N, o);
  } else {
    if (m < M && n < N) epi.finish(m, n, min(4, N - n), acc, input);
  }
}

template <class AL, class BL, class Epi>
hipError_t launch_wave(hipStream_t s, int M, int N, int K, const float* A, int lda, const float* B, int ldb, const Epi& epi,
                       const SideCopy& side = SideCopy{nullptr, nullptr, 0}) {
  const int tiles_m = (M + 15) / 16, tiles_n = (N + 15) / 16;
  const unsigned copiers = (unsigned)std::min<size_t>((side.nvec + 255) / 256, 256);
  hipLaunchKernelGGL((gemm_f32_wave_kernel<AL, BL, Epi>), dim3(tiles_m * tiles_n + copiers), dim3(64), 0, s, M, N, K / 32, A, lda, B,
                     ldb, epi, make_tile_map(tiles_m, tiles_n), side);
  return hipGetLastError();
}
// Up to one wave per SIMD.  With 1024 tiles, 512 x 512 x 1024, 7.9 us against 8.5 in tiles of 32 x 32; with 2048 the waves share
// the SIMDs and the L2s serve twice the bytes, 19.2 against 12.3.  ld: rows' 32-bit offsets.
inline bool wave_ok(int M, int N, int K, int ld) {
  return K % 32 == 0 && ld < (1 << 24) && (long)((M + 15) / 16) * ((N + 15) / 16) <= 1024;
}

// The tiles, and the time of one k tile on a CU with one workgroup (t1) and two (t2), in ns; 128 x 128 leaves room
// for one.  Chains in fp32 are bound by the matrix cores and by what vector instructions take from them: addresses of LDS and
// copies that are constants or scalars (DenseWhole, the loop unrolled over the stages) brought dense products of 512 x 1024 x
// 1024 from 18.1 to 12.5 us, 1024^3 from 28.0 to 20.5, 2048^3 from 158 to 128 (134 TFLOP/s); gathered 3x3 ones on 16 images of
// 32 x 32, 64 channels, from 18.5 to 16.7, bf16 on 44 images of 48 x 48, 48 channels, from 80 to 72 (a third of that on bf16 matrix
// instructions, which do not keep the order of the sum).  32 x 32, 64 x 64 and 128 x 128 tiles: 512 x 1024 x 1024 12.3 / 20.2 / 67,
// 1024^3 21.1 / 20.7 / 67, 2048 x 4096 x 1024 156 / 138 / 135 us.
// s1, s2: the same for products that may be cut into ranges, as timed before that: how many ranges a weight gradient is summed over,
// and with it its rounding, stays what it was.
enum class Tile { k32, k64, k128 };
struct TileCost {
  Tile t;
  int edge, t1, t2;
  int s1, s2;  // the same for products that may be cut into ranges
};
template <class T, class Sum>
struct Tiles;
template <>
struct Tiles<float, Chain> {
  static constexpr TileCost cost[] = {
      {Tile::k32, 32, 180, 300, 270, 480}, {Tile::k64, 64, 560, 1050, 850, 1300}, {Tile::k128, 128, 2150, 4150, 2450, 4900}};
};
template <>
struct Tiles<uint16_t, Chain> {
  static constexpr TileCost cost[] = {{Tile::k32, 32, 660, 930, 0, 0}, {Tile::k64, 64, 1770, 2900, 0, 0}};
};
template <>
struct Tiles<uint16_t, Free> {
  static constexpr TileCost cost[] = {
      {Tile::k32, 32, 0, 0, 200, 300}, {Tile::k64, 64, 0, 0, 350, 550}, {Tile::k128, 128, 0, 0, 800, 1600}};
};

// Contraction ranges of a product whose output has too few tiles for the chip (weight gradients): as many as give every
// CU a workgroup, each at least 8 k tiles long, and none of them empty.
inline int any_splits(long blocks, int KT) {
  const long s = std::min<long>(256 / std::max<long>(blocks, 1), KT / 8);
  if (s <= 1) return 1;
  const int per = (int)((KT + s - 1) / s);
  return (KT + per - 1) / per;
}

inline long blocks_of(int edge, int M, int N) { return (long)((M + edge - 1) / edge) * ((N + edge - 1) / edge); }

// The tile with the least time for all its workgroups on 256 CUs.  split: the contraction may be cut into ranges, so that
// a long one fills the chip with large tiles too; `ranges` receives their number.
template <class T, class Sum>
Tile pick_tile(int M, int N, int KT, bool split, int* ranges) {
  Tile best = Tile::k32;
  double best_cost = -1;
  for (const TileCost& c : Tiles<T, Sum>::cost) {
    const long blocks = blocks_of(c.edge, M, N);
    const int r = split ? any_splits(blocks, KT) : 1;
    const long all = blocks * r, rest = all % 512;
    const int t1 = split ? c.s1 : c.t1, t2 = split ? c.s2 : c.t2;
    const double cost = ((double)(all / 512) * t2 + (rest == 0 ? 0 : rest <= 256 ? t1 : t2)) * ((KT + r - 1) / r);
    if (best_cost < 0 || cost < best_cost) {
      best_cost = cost;
      best = c.t;
      *ranges = r;
    }
  }
  return best;
}

inline bool aligned16(const void* a, const void* b = nullptr, const void* c = nullptr) {
  return (((uintptr_t)a | (uintptr_t)b | (uintptr_t)c) & 15) == 0;
}
// a divisor of numbers up to `limit`
inline FastDiv fast_div(int d, long limit) {
  return FastDiv{d == 1 || limit * d >= (1l << 32) ? 0u : (uint32_t)(((1ull << 32) + d - 1) / d), (uint32_t)d};
}

// Loader class templates with the element type, kind of sum and vector width filled in per product
template <class T, class Sum, int VEC> struct FpropDense {
  template <int R, int NW> using A = DenseRow<T, Sum, R, NW, VEC>;
  template <int R, int NW> using B = DenseRow<T, Sum, R, NW, VEC>;
};
template <class T, class Sum, int VEC> struct DgradDense {
  template <int R, int NW> using A = DenseRow<T, Sum, R, NW, VEC>;
  template <int R, int NW> using B = DenseCol<T, Sum, R, NW, VEC>;
};
template <class T, class Sum, int VEC> struct WgradDense {
  template <int R, int NW> using A = DenseCol<T, Sum, R, NW, VEC>;
  template <int R, int NW> using B = DenseCol<T, Sum, R, NW, VEC>;
};
template <class T, class Sum, int> struct FpropDenseWhole {
  template <int R, int NW> using A = DenseWhole<T, Sum, R, NW, false>;
  template <int R, int NW> using B = DenseWhole<T, Sum, R, NW, false>;
};
template <class T, class Sum, int> struct DgradDenseWhole {
  template <int R, int NW> using A = DenseWhole<T, Sum, R, NW, false>;
  template <int R, int NW> using B = DenseWhole<T, Sum, R, NW, true>;
};
template <class T, class Sum, int> struct WgradDenseWhole {
  template <int R, int NW> using A = DenseWhole<T, Sum, R, NW, true>;
  template <int R, int NW> using B = DenseWhole<T, Sum, R, NW, true>;
};
template <class T, class Sum, int VEC> struct FpropConv {
  template <int R, int NW> using A = GatherRow<T, Sum, R, NW, VEC, false>;
  template <int R, int NW> using B = DenseRow<T, Sum, R, NW, VEC>;
};
template <class T, class Sum, int VEC> struct DgradConv {
  template <int R, int NW> using A = GatherRow<T, Sum, R, NW, VEC, true>;
  template <int R, int NW> using B = WeightCol<T, Sum, R, NW, VEC>;
};
template <class T, class Sum, int VEC> struct WgradConv {
  template <int R, int NW> using A = DenseCol<T, Sum, R, NW, VEC>;
  template <int R, int NW> using B = GatherCol<T, Sum, R, NW, VEC>;
};

template <class T, class Sum, template <class, class, int> class Product, int VEC, class AD, class BD, class Epi>
hipError_t run(hipStream_t s, int M, int N, int K, const AD& ad, const BD& bd, const Epi& epi, bool split = false,
               const SideCopy& side = SideCopy{nullptr, nullptr, 0}) {
  using P = Product<T, Sum, VEC>;
  const int KT = (K + kTileK<T> - 1) / kTileK<T>;
  int ranges = 1;
#define TP_ANY(E, WGM, WGN, NS, U)                                                                                           \
  launch_any<T, Sum, E, E, WGM, WGN, NS, U, typename P::template A<E, WGM * WGN>, typename P::template B<E, WGM * WGN>>( \
      s, M, N, KT, ranges, ad, bd, epi, side)
  switch (pick_tile<T, Sum>(M, N, KT, split, &ranges)) {
    case Tile::k128:
      if constexpr (sizeof(T) == 4) return TP_ANY(128, 4, 2, 2, 2);
      else if constexpr (__is_same(Sum, Free)) return TP_ANY(128, 4, 2, 3, 1);
      [[fallthrough]];  // not among those tiles
    case Tile::k64: return TP_ANY(64, 4, 2, 2, 2);
    default:
      // with more workgroups than CUs, four of them on a CU at 32 KB each instead of two at 64 KB
      if (blocks_of(32, M, N) * ranges <= 256) return TP_ANY(32, 2, 2, 2, 4);
      return TP_ANY(32, 2, 2, 2, 2);
  }
#undef TP_ANY
}
template <class T, class Sum>
int ranges_of(int M, int N, int K) {
  int ranges = 1;
  pick_tile<T, Sum>(M, N, (K + kTileK<T> - 1) / kTileK<T>, true, &ranges);
  return ranges;
}

// whole k tiles of fp32 operands with rows of `ld` values, 128 rows of which (32 k values, each a row) lie within 2 GiB
inline bool whole_tiles(int K, int ld) { return K % kTileK<float> == 0 && ld < (1 << 22); }

}  // namespace

// ---- dense, fp32 -------------------------------------------------------------------------------
hipError_t f32_fprop(hipStream_t s, int M, int N, int K, const float* x, const float* W, const float* bias, int act, float* d_out,
                     float* a_out, float* x_copy) {
  SideCopy side{nullptr, nullptr, 0};
  if (x_copy) {
    // Behind the tiles the copy is hidden where one stream runs everything: a step of four micro-batches and two layers takes
    // 7 us less than with launches of its own at every size from 16 KB to 1 MB (32 x 512: 103 and 110 us; pipeline of
    // 256-512-512-10, batches of 32: 1140 and 1268 us).  On two forward streams it also takes slots from products of the other
    // one: from process to process 4 us more to 17 us less at 64 KB, 17 us more to 3 us less at 512 KB.  The line lies at
    // 256 KB, in between.
    if (aligned16(x, x_copy) && (size_t)M * K % 4 == 0 && (size_t)M * K <= 65536) {
      side = SideCopy{(const uint4*)x, (uint4*)x_copy, (size_t)M * K / 4};
    } else {
      const hipError_t e = launch_copy(s, x, x_copy, (size_t)M * K * 4);
      if (e != hipSuccess) return e;
    }
  }
  const DenseDesc a{x, K, M, K}, b{W, K, N, K};
  const EpiForward<float> e{bias, d_out, a_out, act, N, N % 4 == 0 && aligned16(d_out, a_out)};
  if (aligned16(x, W) && wave_ok(M, N, K, K))
    return launch_wave<WaveRow, WaveRow>(s, M, N, K, x, K, W, K, e, side);
  if (whole_tiles(K, K) && aligned16(x, W)) return run<float, Chain, FpropDenseWhole, 4>(s, M, N, K, a, b, e, false, side);
  if (K % 4 == 0 && aligned16(x, W)) return run<float, Chain, FpropDense, 4>(s, M, N, K, a, b, e, false, side);
  return run<float, Chain, FpropDense, 1>(s, M, N, K, a, b, e, false, side);
}

hipError_t f32_dgrad(hipStream_t s, int M, int N, int K, const float* dz, const float* Wb, const float* d_prev, float* out,
                     int relu_mask, float* sums) {
  // out[M x K] = dz[M x N] . Wb[N x K]: contraction over N
  const DenseDesc a{dz, N, M, N}, b{Wb, K, K, N};
  const EpiInputGrad<float> e{d_prev, out, K, relu_mask, K % 4 == 0 && aligned16(out), sums};
  if (K % 4 == 0 && aligned16(dz, Wb) && wave_ok(M, K, N, std::max(N, K)))
    return launch_wave<WaveRow, WaveCol>(s, M, K, N, dz, N, Wb, K, e);
  if (whole_tiles(N, std::max(N, K)) && K % 4 == 0 && aligned16(dz, Wb)) return run<float, Chain, DgradDenseWhole, 4>(s, M, K, N, a, b, e);
  if (N % 4 == 0 && K % 4 == 0 && aligned16(dz, Wb)) return run<float, Chain, DgradDense, 4>(s, M, K, N, a, b, e);
  return run<float, Chain, DgradDense, 1>(s, M, K, N, a, b, e);
}

int f32_wgrad_splits(int M, int N, int K) { return ranges_of<float, Chain>(N, K, M); }

hipError_t f32_wgrad(hipStream_t s, int M, int N, int K, const float* dz, const float* x, float* gW, float* partial) {
  // gW[N x K] = dz^T[N x M] . x[M x K]: contraction over M
  const bool split = partial != nullptr;
  const int splits = split ? f32_wgrad_splits(M, N, K) : 1;
  const DenseDesc a{dz, N, N, M}, b{x, K, K, M};
  float* out = splits > 1 ? partial : gW;
  const EpiPartial e{out, K, K % 4 == 0 && aligned16(out), (size_t)N * K};
  const bool chunks = N % 4 == 0 && K % 4 == 0 && aligned16(dz, x);
  const hipError_t err = chunks && whole_tiles(M, std::max(N, K)) ? run<float, Chain, WgradDenseWhole, 4>(s, N, K, M, a, b, e, split)
                         : chunks                                ? run<float, Chain, WgradDense, 4>(s, N, K, M, a, b, e, split)
                                                                 : run<float, Chain, WgradDense, 1>(s, N, K, M, a, b, e, split);
  if (err != hipSuccess || splits == 1) return err;
  return launch_sum_partials(s, (size_t)N * K, splits, partial, gW);
}

// ---- convolutions ------------------------------------------------------------------------------
bool conv_any_supported(int elt, int imgs, int H, int W, int ksize, int stride, int cin, int cout) {
  const long taps = (long)ksize * ksize, pin = (long)imgs * H * W;
  // image edges fit 15 bits; pixel numbers, k values and offsets inside an image 31
  return H + ksize < 32768 && W + ksize < 32768 && pin < (1l << 30) && taps * std::max(cin, cout) < (1l << 30) &&
         (long)H * W * std::max(cin, cout) < (1l << 31) &&
         (elt == ELT_F32 || (cin % 8 == 0 && cout % 8 == 0));
}

hipError_t conv_any_fprop(hipStream_t s, int elt, int imgs, int H, int W, int ksize, int stride, int cin, int cout, const void* x,
                          const void* wgt, const float* bias, int act, void* d_out, void* a_out) {
  const int Ho = H / stride, Wo = W / stride, P = imgs * Ho * Wo, K = ksize * ksize * cin;
  const GatherRowDesc a{x, P, Ho, Wo, H, W, cin, K, stride, (ksize - 1) / 2, fast_div(cin, K + 64), fast_div(ksize, K + 64)};
  const DenseDesc b{wgt, K, cout, K};
  const bool vec = aligned16(x, wgt);
  if (elt == ELT_BF16) {
    if (!vec) return hipErrorNotSupported;
    return run<uint16_t, Chain, FpropConv, 8>(s, P, cout, K, a, b, EpiForward<uint16_t>{bias, (uint16_t*)d_out, (uint16_t*)a_out, act, cout, aligned16(d_out, a_out)});
  }
  const EpiForward<float> e{bias, (float*)d_out, (float*)a_out, act, cout, cout % 4 == 0 && aligned16(d_out, a_out)};
  if (cin % 4 == 0 && vec) return run<float, Chain, FpropConv, 4>(s, P, cout, K, a, b, e);
  return run<float, Chain, FpropConv, 1>(s, P, cout, K, a, b, e);
}

hipError_t conv_any_dgrad(hipStream_t s, int elt, int imgs, int H, int W, int ksize, int stride, int cin, int cout, const void* dz,
                          const void* wb, const void* d_prev, void* out, int relu_mask, float* sums) {
  const int taps = ksize * ksize, P = imgs * H * W, K = taps * cout;
  const GatherRowDesc a{dz, P, H, W, H / stride, W / stride, cout, K, stride, (ksize - 1) / 2, fast_div(cout, K + 64), fast_div(ksize, K + 64)};
  const WeightColDesc b{wb, cin, taps, cout, fast_div(cout, K + 64)};
  const bool vec = aligned16(dz, wb);
  if (elt == ELT_BF16) {
    if (!vec) return hipErrorNotSupported;
    return run<uint16_t, Chain, DgradConv, 8>(s, P, cin, K, a, b, EpiInputGrad<uint16_t>{(const uint16_t*)d_prev, (uint16_t*)out, cin, relu_mask, aligned16(out), sums});
  }
  const EpiInputGrad<float> e{(const float*)d_prev, (float*)out, cin, relu_mask, cin % 4 == 0 && aligned16(out), sums};
  if (cin % 4 == 0 && cout % 4 == 0 && vec) return run<float, Chain, DgradConv, 4>(s, P, cin, K, a, b, e);
  return run<float, Chain, DgradConv, 1>(s, P, cin, K, a, b, e);
}

int conv_any_wgrad_splits(int elt, int pixels, int cin, int cout, int ksize) {
  const int N = ksize * ksize * cin;
  return elt == ELT_BF16 ? ranges_of<uint16_t, Free>(cout, N, pixels) : ranges_of<float, Chain>(cout, N, pixels);
}

hipError_t conv_any_wgrad(hipStream_t s, int elt, int imgs, int H, int W, int ksize, int stride, int cin, int cout, const void* dz,
                          const void* x, float* gW, float* partial) {
  const int Ho = H / stride, Wo = W / stride, P = imgs * Ho * Wo, N = ksize * ksize * cin;
  const int splits = conv_any_wgrad_splits(elt, P, cin, cout, ksize);
  const DenseDesc a{dz, cout, cout, P};
  const GatherColDesc b{x, H, W, cin, P, stride, (ksize - 1) / 2, N, fast_div(cin, N), fast_div(ksize, N), fast_div(Wo, P + 64), fast_div(Ho, P + 64)};
  float* out = splits > 1 ? partial : gW;
  const EpiPartialPixels e{{out, N, N % 4 == 0 && aligned16(out), (size_t)cout * N}};
  const bool vec = aligned16(dz, x);
  hipError_t err;
  if (elt == ELT_BF16) {
    if (!vec) return hipErrorNotSupported;
    err = run<uint16_t, Free, WgradConv, 8>(s, cout, N, P, a, b, e, true);
  } else if (cin % 4 == 0 && cout % 4 == 0 && vec) {
    err = run<float, Chain, WgradConv, 4>(s, cout, N, P, a, b, e, true);
  } else {
    err = run<float, Chain, WgradConv, 1>(s, cout, N, P, a, b, e, true);
  }
  if (err != hipSuccess || splits == 1) return err;
  return launch_sum_partials(s, (size_t)cout * N, splits, partial, gW);
}

}  // namespace tp
