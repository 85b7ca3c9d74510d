// Matrix-core products outside the tuned bf16 kernels' shapes: the fp32 mode's dense layers and convolutions, and bf16
// convolutions of any geometry whose channel counts are multiples of 8 (kernels_gemm_any.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace tp {

// fp32 dense layers, any shape and alignment; arguments as launch_fprop, launch_dgrad and launch_wgrad.
hipError_t f32_fprop(hipStream_t s, int M, int N, int K, const float* x, const float* W, const float* bias, int act, float* d_out,
                     float* a_out, float* x_copy);
hipError_t f32_dgrad(hipStream_t s, int M, int N, int K, const float* dz, const float* Wb, const float* d_prev, float* out,
                     int relu_mask, float* sums = nullptr);  // sums: column sums of every 16 rows of `out`, [(M + 15) / 16][K]
// partial: scratch of f32_wgrad_splits(M, N, K) * N * K floats where that is more than one range, or null
hipError_t f32_wgrad(hipStream_t s, int M, int N, int K, const float* dz, const float* x, float* gW, float* partial);
int f32_wgrad_splits(int M, int N, int K);

// Convolutions; arguments as the launchers of conv.h.  bf16 tensors must be 16-byte aligned (hipErrorNotSupported, with
// nothing launched, otherwise).
bool conv_any_supported(int elt, int imgs, int H, int W, int ksize, int stride, int cin, int cout);
hipError_t conv_any_fprop(hipStream_t s, int elt, int imgs, int H, int W, int ksize, int stride, int cin, int cout, const void* x,
                          const void* wgt, const float* bias, int act, void* d_out, void* a_out);
hipError_t conv_any_dgrad(hipStream_t s, int elt, int imgs, int H, int W, int ksize, int stride, int cin, int cout, const void* dz,
                          const void* wb, const void* d_prev, void* out, int relu_mask, float* sums = nullptr);
hipError_t conv_any_wgrad(hipStream_t s, int elt, int imgs, int H, int W, int ksize, int stride, int cin, int cout, const void* dz,
                          const void* x, float* gW, float* partial);
int conv_any_wgrad_splits(int elt, int pixels, int cin, int cout, int ksize);

}  // namespace tp
