// Launch interface of the convolution, pooling and subsampling kernels (ksize x ksize with ksize 1, 3, 5 or 7,
// stride 1 or 2, pad (ksize-1)/2; 2x2 max pool; every second pixel; global average).  H, W are the INPUT image
// (even for stride 2); with stride s the output image is (H/s) x (W/s).  elt: 0 = fp32, 1 = bf16.  Activations are
// NHWC, [imgs*H*W x C] row-major; weights [Cout][ksize][ksize][Cin].  The matrix-core kernels take ksize 3 only.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

namespace tp {

// the geometries the kernels take; the launchers return hipErrorInvalidValue for any other
bool conv_geometry_supported(int ksize, int stride, int pad);

// a = act(conv(x, W) + bias), d = act'(.) (d_out may be null).  Outputs [imgs*(H/stride)*(W/stride) x cout].
// zeros: device block of >= 128 zero bytes, 16-byte aligned (what padding positions read); the
// matrix-core kernels need it, null sends everything to the generic kernels.
hipError_t launch_conv_fprop(hipStream_t s, int elt, int imgs, int H, int W, int ksize, int stride, int cin, int cout,
                             const void* x, const void* wgt, const float* bias, int act, void* d_out, void* a_out,
                             const void* zeros);

// out = (transposed convolution of dz with W_b) (.) d_prev;  dz:[imgs*H*W x cout], out:[imgs*H*W x cin].
// relu_mask = 1: d_prev holds the previous layer's ReLU output and the factor is (output > 0).
hipError_t launch_conv_dgrad(hipStream_t s, int elt, int imgs, int H, int W, int ksize, int stride, int cin, int cout,
                             const void* dz, const void* wb, const void* d_prev, void* out, const void* zeros,
                             int relu_mask = 0, float* sums = nullptr, int* sum_rows = nullptr);
// sums: room for conv_dgrad_sum_rows(...) rows of cin floats.  *sum_rows receives how many rows of partial column sums of `out`
// were left there (so many, or 0: tensors that are not 16-byte aligned, zeros missing).
int conv_dgrad_sum_rows(int elt, int imgs, int H, int W, int ksize, int stride, int cin, int cout);

// gW[cout][ksize][ksize][cin] (fp32) = sum over pixels of dz (x) shifted x.
// partial: scratch of conv_wgrad_scratch_floats(output pixels of the mini-batch, cin, cout, ksize) floats.
hipError_t launch_conv_wgrad(hipStream_t s, int elt, int imgs, int H, int W, int ksize, int stride, int cin, int cout,
                             const void* dz, const void* x, float* gW, float* partial, const void* zeros);
// nine_taps: as if image tiles took all nine taps per workgroup at every size, three times the ranges of filter rows.
size_t conv_wgrad_scratch_floats(int pixels, int cin, int cout, int ksize, bool nine_taps = false);

// y[imgs x H/2 x W/2 x C] = 2x2/2 max pooling of x[imgs x H x W x C];  backward recomputes the
// position of the (first) maximum from the saved input x.
hipError_t launch_maxpool_fwd(hipStream_t s, int elt, int imgs, int H, int W, int C, const void* x, void* y);
// d_prev (may be null; only where maxpool_bwd_fuses_activation says so and all pointers are 16-byte aligned): the
// gradient also passes the activation in front of the pooling, dx (.)= d_prev (saved act'), or (relu_mask) the
// factor (d_prev > 0) of a saved ReLU output -- with the bits of the two separate kernels.
hipError_t launch_maxpool_bwd(hipStream_t s, int elt, int imgs, int H, int W, int C, const void* x, const void* dy,
                              void* dx, const void* d_prev = nullptr, int relu_mask = 0, float* sums = nullptr,
                              int* sum_rows = nullptr);
// the same for the gradient max pooling hands on
int maxpool_sum_rows(int elt, int imgs, int H, int W, int C);
bool maxpool_bwd_fuses_activation(int elt, int C);

// y[imgs x H/2 x W/2 x C] = x at the even pixel positions; backward: the gradient at those positions, zero elsewhere.
// C * element size must be a multiple of 16 bytes.
hipError_t launch_subsample_fwd(hipStream_t s, int elt, int imgs, int H, int W, int C, const void* x, void* y);
hipError_t launch_subsample_bwd(hipStream_t s, int elt, int imgs, int H, int W, int C, const void* dy, void* dx);

// y[imgs x C] = mean over the positions of x[imgs x positions x C]; backward: dx = dy / positions at every position.
hipError_t launch_avgpool_fwd(hipStream_t s, int elt, int imgs, int positions, int C, const void* x, void* y);
hipError_t launch_avgpool_bwd(hipStream_t s, int elt, int imgs, int positions, int C, const void* dy, void* dx);

// bf16 matrix-core versions (kernels_conv_mfma.hip) and the shapes they take
bool conv_mfma_supported(int imgs, int H, int W, int stride, int cin, int cout);
int conv_mfma_wgrad_max_splits(int pixels, int cin, int cout, bool nine_taps);
// How the 3x3 weight gradient of image tiles (stride 1) is split: pixel ranges, the products of `apart` tiles of a range summed apart, and
// all nine taps per workgroup or the three of a filter row (`rows`).
// The faster of the two by these estimates in ns, fitted to 28 layers of 64 to 1024 channels: nine taps 11 us + 1.8 per tile + 1.1 for
// every time sums are put aside, rows 9.6 + 0.69 per tile and 0.55 for every time, 22 ns per partial result of 64 x 64 channels.  Nine taps and
// rows, with the launch that adds up, us: 128 images of 16 x 16, 384 channels 92 and 108, 512 channels 144 and 194 (one row range for 192
// CUs), 640 channels 246 and 378 (two rounds); 256 of 32 x 32, 64 channels, 37.3 and 36.9; 16 of 64 x 64 26.1 and 21.3; 16 of 16 x 16,
// 512 channels, 38.1 and 36.5; 4 of them 24.5 and 19.8.
// A sum's squared error, in steps of 16 pixels, counts 8 per tile of a nine-tap chain, 4 of a row's, one for every chain, two for the
// meeting of a row's halves, a tenth for every range.  Rows only where that is less than in nine-tap chains over all tiles, and with fewer
// than two tiles per nine-tap workgroup only with a single one of their own (6 images of 16 x 16, 192 -> 320 channels: off fp64 by 6.9e-8
// with nine taps, 7.3e-8 by rows); nine taps only in chains that bring it down to that of rows by eights, since over all tiles of
// a workgroup they are far off (128 images of 16 x 16, 448 channels, 4.1e-7 and 1.4e-7).
constexpr int kWgradPixels = 128;  // of a tile
struct PatchWgradPlan {
  bool rows;
  int splits, apart;
};
inline PatchWgradPlan patch_wgrad_plan(long px_tiles, int cin, int cout) {
  const long blocks = std::max(1l, (long)(cin / 64) * (cout / 64));
  auto over = [](long a, long b) { return (a + b - 1) / b; };
  auto ranges = [&](long workgroups) { return std::max(1l, std::min(px_tiles, 256 / workgroups)); };
  const long nine = ranges(blocks), rows = ranges(3 * blocks), nine_tiles = over(px_tiles, nine), row_tiles = over(px_tiles, rows);
  int row_apart = (int)std::min(row_tiles, 8l), nine_apart = (int)std::min(nine_tiles, 64l);
  while (row_apart > 0 && (10 * (4 * row_apart + over(row_tiles, row_apart) + 2) + rows) * nine >= 80 * px_tiles + nine * nine) --row_apart;
  if (px_tiles < 2 * nine && row_tiles > 1) row_apart = 0;
  const long most = 10 * (34 + over(row_tiles, 8)) + rows;
  while (nine_apart > 0 && 10 * (8 * nine_apart + over(nine_tiles, nine_apart) + 1) + nine > most) --nine_apart;
  const long nine_ns = 11000 + 1800 * nine_tiles + (nine_apart ? 1100 * ((nine_tiles - 1) / nine_apart) : 0) + 22 * blocks * nine;
  const long row_round = 690 * row_tiles + (row_apart ? 550 * ((row_tiles - 1) / row_apart) : 0);
  const long row_ns = 9600 + row_round * over(3 * blocks * rows, 256) + 22 * blocks * rows;
  if (row_apart && (!nine_apart || row_ns < nine_ns)) return {true, (int)rows, row_apart};
  return {false, (int)nine, nine_apart ? nine_apart : (int)nine_tiles};
}
hipError_t conv_mfma_fprop(hipStream_t s, int imgs, int H, int W, int stride, int cin, int cout, const uint16_t* x,
                           const uint16_t* wgt, const float* bias, int act, uint16_t* d_out, uint16_t* a_out,
                           const uint16_t* zeros);
hipError_t conv_mfma_dgrad(hipStream_t s, int imgs, int H, int W, int stride, int cin, int cout, const uint16_t* dz,
                           const uint16_t* wb, const uint16_t* d_prev, uint16_t* out, const uint16_t* zeros, int relu_mask = 0,
                           float* sums = nullptr, int* sum_rows = nullptr);
int conv_mfma_dgrad_sum_rows(int imgs, int H, int W, int stride, int cin, int cout);
hipError_t conv_mfma_wgrad(hipStream_t s, int imgs, int H, int W, int stride, int cin, int cout, const uint16_t* dz,
                           const uint16_t* x, float* gW, float* partial, const uint16_t* zeros);

// First layer of an image net (cin <= 8, bf16) on a zero-padded [pixel][8 channels] copy x8 of its input.
bool conv_c8_supported(int imgs, int H, int W, int cin, int cout);
hipError_t conv_c8_pad(hipStream_t s, size_t pixels, int cin, const uint16_t* x, uint16_t* x8);
hipError_t conv_c8_fprop(hipStream_t s, int imgs, int H, int W, int cin, int cout, const uint16_t* x8, const uint16_t* wgt,
                         const float* bias, int act, uint16_t* d_out, uint16_t* a_out, const uint16_t* zeros);
hipError_t conv_c8_wgrad(hipStream_t s, int imgs, int H, int W, int cin, int cout, const uint16_t* dz, const uint16_t* x8,
                         float* gW, float* partial, const uint16_t* zeros);

// The 7x7 stride-2 pad-3 first layer (cin <= 8, bf16) on the same padded copy; H, W: the input image.
bool conv_stem_supported(int imgs, int H, int W, int cin, int cout);
int conv_stem_wgrad_splits(int out_pixels, int cout);
hipError_t conv_stem_fprop(hipStream_t s, int imgs, int H, int W, int cin, int cout, const uint16_t* x8, const uint16_t* wgt,
                           const float* bias, int act, uint16_t* d_out, uint16_t* a_out, const uint16_t* zeros);
hipError_t conv_stem_wgrad(hipStream_t s, int imgs, int H, int W, int cin, int cout, const uint16_t* dz, const uint16_t* x8,
                           float* gW, float* partial, const uint16_t* zeros);

}  // namespace tp
