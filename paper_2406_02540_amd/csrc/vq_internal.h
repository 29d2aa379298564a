// Internal launch interface between the C-ABI front end (vq_api.hip) and the
// gfx950 kernels.  Every launcher enqueues on `stream` and returns the HIP
// error of the launch; arguments were validated by the caller.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace vq {

// A kernel of one argument.  (An argument costs the host 0.04 us, the <<<>>> stub 0.15 us beyond the 2.1 that a launch
// takes; small layers are host-bound.)
template <class Args>
inline hipError_t enqueue(void (*kernel)(Args), dim3 grid, dim3 block, hipStream_t stream, const Args& a) {
    void* args[] = {const_cast<Args*>(&a)};
    const hipError_t e = hipLaunchKernel((const void*)kernel, grid, block, args, 0, stream);
    if (e != hipSuccess) (void)hipGetLastError();   // (reported here, not once more by the next call)
    return e;
}

hipError_t launch_quantize_per_token(const void* x_f16, const float* chan_mul, int8_t* xq,
                                     float* x_scale, int M, int K, hipStream_t stream);

// Its part for rows of whole chunks (vq_fused.hip): K % 8 == 0, K <= 8192, 16-byte aligned.
hipError_t launch_plain_quantize(const void* x_f16, const float* chan_mul, int8_t* xq, float* x_scale, int M, int K,
                                 hipStream_t stream);

// What runs in front of the quantizer, and its operands (those that it does not have stay null).
enum Producer { kGeluErf = 0, kGeluTanh = 1, kLayerNorm = 2, kResidual = 3, kHadamard = 4, kPlain = 5 };
struct ProducerArgs {
    int producer;
    const void* x;            // fp16 [M,K]
    const float* chan_mul;    // Eq. 3's factor [K], or null
    const void* y;            // residual: the branch output, fp16 [M,K]
    void* r;                  // residual: the sum, fp16 [M,K]
    const float* mod_a;       // LayerNorm: scale [B,K]; residual: gate [B,K]; or null
    const float* mod_b;       // LayerNorm: shift [B,K]; or null
    int tokens_per_sample;    // >= 1
    float eps;
};

// The quantizer behind its producer (vq_fused.hip; kPlain goes to launch_quantize_per_token):
// K % 8 == 0, K <= 8192 (Hadamard: K % 128 == 0).
hipError_t launch_producer_quantize(const ProducerArgs& p, int8_t* xq, float* x_scale, int M, int K, hipStream_t stream);
hipError_t launch_rotate_weight(const float* w, const float* chan_s, float* w_rot, int N, int K,
                                hipStream_t stream);                  // K % 128 == 0, K <= 8192

// Calibration of Eq. 3's mask: column absmax of fp16 (is_f32 = 0) or fp32 rows, and the mask itself.
hipError_t launch_channel_absmax(const void* a, int is_f32, float* amax, int R, int K, int accumulate,
                                 hipStream_t stream);
hipError_t launch_balance_mask(const float* amax_x, const float* amax_w, float alpha, float* s, float* chan_mul,
                               int K, hipStream_t stream);

hipError_t launch_quantize_static(const void* x_f16, const float* chan_mul, float inv_scale, int8_t* xq,
                                  int M, int K, hipStream_t stream);

hipError_t launch_quantize_weight(const float* w, const float* chan_s, int w_bits, void* wq_out,
                                  float* w_scale, int N, int K, hipStream_t stream);

// w_bits 8: w is int8 [N,K]; 4: w is packed nibbles [N,K/2]; 16: the fp16 comparison layer, xq and w
// are fp16 [M,K] and [N,K], x_scale and w_scale are not read, acc_out must be null.  num_cus: compute units of
// the device the stream belongs to (the kernel is persistent, one workgroup per CU).
hipError_t launch_gemm(const int8_t* xq, const float* x_scale, const void* w, int w_bits,
                       const float* w_scale, const void* bias_f16, void* y_f16, int32_t* acc_out,
                       int M, int N, int K, int num_cus, hipStream_t stream);

// The kernel that launch_gemm takes: tiles of tokens x channels, and the number of wavefronts that divide K (0:
// the workgroup shares the tile; with 256 tokens it is the persistent kernel).
struct GemmChoice { int tile_t, tile_c, waves; };
GemmChoice choose_gemm(int w_bits, int M, int N, int K, int num_cus);

// A layer of few tokens in one launch (vq_linear_small.hip): quantizer, with its producer, and GEMM.
// small_layer: whether it is the faster way for these sizes.
bool small_layer(int producer, int M, int N, int K, int num_cus);
hipError_t launch_linear_small(const ProducerArgs& p, const void* w, int w_bits, const float* w_scale, const void* bias_f16,
                               void* y_f16, int M, int N, int K, hipStream_t stream);

}  // namespace vq

// For the tests, which name the kernels that they mean to reach: choose_gemm, and how the persistent kernel
// writes its rows (Out, vq_gemm_common.h).  Not a part of vq.h.
extern "C" void vq_internal_gemm_choice(int w_bits, int M, int N, int K, int num_cus, int choice[3]);
extern "C" int vq_internal_gemm_out(int N, const void* y, const void* acc_out);
