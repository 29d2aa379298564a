// The quantizers fused behind their producers (kernel template and its description:
// vq_fused_kernel.h): the entry points, the plain, LayerNorm, residual and Hadamard kernels (the GELU
// ones are compiled in vq_fused_gelu.hip), and the offline weight rotation.
#include "vq_fused_kernel.h"

namespace vq {
namespace {

// Weight side of the rotation, offline.  A block of 128 channels is 16 lanes; lane p holds its values
// 4p .. 4p+3 and 64+4p .. 64+4p+3, so that every load and store covers whole cache lines, and the
// stages run in the order of the channel's bits: two in registers, four across lanes, the last one
// in registers; no LDS memory and no barrier.  Memory-bound (8 bytes per element).
// 4608 x 1152: 7.65 us (12.0 with a 64-bit division in front of the loads, 8.3 without it and with two blocks
// per thread, 9.1 with four; 14.7-16.4 with eight consecutive values per lane, that is half of every line per load).
constexpr int kRotateWidth = kQuantThreads / 16;   // blocks of 128 per workgroup
__global__ __launch_bounds__(kQuantThreads) void rotate_weight_blocks(const float4v* w,
                                                                      const float4v* __restrict__ chan_s,
                                                                      float4v* out, long blocks, int K128) {
    const int blk = threadIdx.x >> 4, sub = threadIdx.x & 15;
    const long at = (long)blockIdx.x * kRotateWidth + blk;
    if (at >= blocks) return;   // (groups of 16 lanes are wholly in or out)
    float t[1][8];              // (w and out may be one buffer: a thread writes what it read)
    const float4v lo = w[32 * at + sub], hi = w[32 * at + 16 + sub];
    float4v slo, shi;
    if (chan_s) {
        // the block's place in its row, from remainders that stay small (K128 <= 64)
        const unsigned col = ((blockIdx.x % (unsigned)K128) * (unsigned)kRotateWidth + (unsigned)blk) % (unsigned)K128;
        slo = chan_s[32 * col + sub];
        shi = chan_s[32 * col + 16 + sub];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) t[0][j] = lo[j], t[0][4 + j] = hi[j];
    if (chan_s) {
#pragma unroll
        for (int j = 0; j < 4; ++j) t[0][j] = t[0][j] * slo[j], t[0][4 + j] = t[0][4 + j] * shi[j];
    }
    hadamard_register_stages<0, 2>(t);
    hadamard_lane_stage<1>(t, sub);
    hadamard_lane_stage<2>(t, sub);
    hadamard_lane_stage<4>(t, sub);
    hadamard_lane_stage<8>(t, sub);
    hadamard_register_stages<2, 3>(t);
    const float scale = hadamard_sign(sub) * kHadamardScale;
    float4v olo, ohi;
#pragma unroll
    for (int j = 0; j < 4; ++j) olo[j] = t[0][j] * scale, ohi[j] = t[0][4 + j] * scale;
    out[32 * at + sub] = olo;
    out[32 * at + 16 + sub] = ohi;
}

}  // namespace

hipError_t launch_producer_other(int producer, const FusedArgs& a, hipStream_t stream) {
    switch (producer) {
        case kLayerNorm: return launch_producer<kLayerNorm>(a, stream);
        case kResidual: return launch_producer<kResidual>(a, stream);
        case kPlain: return launch_producer<kPlain>(a, stream);
        default: return launch_producer<kHadamard>(a, stream);
    }
}

hipError_t launch_producer_quantize(const ProducerArgs& p, int8_t* xq, float* x_scale, int M, int K, hipStream_t stream) {
    if (p.producer == kPlain) return launch_quantize_per_token(p.x, p.chan_mul, xq, x_scale, M, K, stream);
    const FusedArgs a = fused_args(p, xq, x_scale, M, K);
    if (p.producer == kGeluErf || p.producer == kGeluTanh) return launch_producer_gelu(p.producer, a, stream);
    return launch_producer_other(p.producer, a, stream);
}

hipError_t launch_plain_quantize(const void* x_f16, const float* chan_mul, int8_t* xq, float* x_scale, int M, int K,
                                 hipStream_t stream) {
    ProducerArgs p{};
    p.producer = kPlain;
    p.x = x_f16;
    p.chan_mul = chan_mul;
    p.tokens_per_sample = 1;
    return launch_producer_other(kPlain, fused_args(p, xq, x_scale, M, K), stream);
}

hipError_t launch_rotate_weight(const float* w, const float* chan_s, float* w_rot, int N, int K,
                                hipStream_t stream) {
    // HIP takes less than 2^32 threads: from 2^35 elements on several launches, of whole rows (chan_s begins with each)
    constexpr long most = ((1l << 32) / kQuantThreads - 1) * kRotateWidth;
    const long rows = min((long)N, most / (K / 128));
    for (long n = 0; n < N; n += rows) {
        const long blocks = min(rows, N - n) * (K / 128), at = n * (K / 4);
        hipLaunchKernelGGL(rotate_weight_blocks, dim3((unsigned)((blocks + kRotateWidth - 1) / kRotateWidth)), dim3(kQuantThreads), 0,
                           stream, (const float4v*)w + at, (const float4v*)chan_s, (float4v*)w_rot + at, blocks, K / 128);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace vq
