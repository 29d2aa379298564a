// The quantizers fused behind their producers (kernel template and its description:
// vq_fused_kernel.h): the entry points, the plain, LayerNorm, residual and Hadamard kernels (the GELU
// ones are compiled in vq_fused_gelu.hip), and the offline weight rotation.
#include "vq_fused_kernel.h"

namespace vq {
namespace {

// Weight side of the rotation, offline.  A block of 128 channels is 16 lanes; lane p holds its values
// 4p .. 4p+3 and 64+4p .. 64+4p+3, so that every load and store covers whole cache lines, and the
// stages run in the order of the channel's bits: two in registers, four across lanes, the last one
// in registers; no LDS memory and no barrier.  Memory-bound (8 bytes per element); a thread takes
// kRotateBlocks blocks a workgroup's width apart, asked for first.
// 4608 x 1152: 12.0-12.9 us (21.4 as a workgroup per row with the stages in LDS and a barrier after
// each; 14.7-16.4 with eight consecutive values per lane, that is half of every line per load).
constexpr int kRotateBlocks = 2, kRotateWidth = kQuantThreads / 16;   // blocks of 128 per workgroup and step
__global__ __launch_bounds__(kQuantThreads) void rotate_weight_blocks(const float4v* w,
                                                                      const float4v* __restrict__ chan_s,
                                                                      float4v* out, long blocks, int K128) {
    const long first = (long)blockIdx.x * (kRotateWidth * kRotateBlocks);
    const int blk = threadIdx.x >> 4, sub = threadIdx.x & 15;
    const int col0 = (int)(first % K128);   // block of its row that this workgroup begins with
    float t[kRotateBlocks][8];              // (w and out may be one buffer: a thread writes what it read)
#pragma unroll
    for (int i = 0; i < kRotateBlocks; ++i) {
        const long at = first + i * kRotateWidth + blk;
        float4v lo{}, hi{};
        if (at < blocks) {   // (groups of 16 lanes are wholly in or out)
            lo = w[32 * at + sub];
            hi = w[32 * at + 16 + sub];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) t[i][j] = lo[j], t[i][4 + j] = hi[j];
    }
    if (chan_s) {
#pragma unroll
        for (int i = 0; i < kRotateBlocks; ++i) {
            const int col = (col0 + i * kRotateWidth + blk) % K128;
            const float4v lo = chan_s[32 * col + sub], hi = chan_s[32 * col + 16 + sub];
#pragma unroll
            for (int j = 0; j < 4; ++j) t[i][j] = t[i][j] * lo[j], t[i][4 + j] = t[i][4 + j] * hi[j];
        }
    }
    hadamard_register_stages<0, 2>(t);
    hadamard_lane_stage<1>(t, sub);
    hadamard_lane_stage<2>(t, sub);
    hadamard_lane_stage<4>(t, sub);
    hadamard_lane_stage<8>(t, sub);
    hadamard_register_stages<2, 3>(t);
    const float scale = hadamard_sign(sub) * kHadamardScale;
#pragma unroll
    for (int i = 0; i < kRotateBlocks; ++i) {
        const long at = first + i * kRotateWidth + blk;
        if (at >= blocks) continue;
        float4v lo, hi;
#pragma unroll
        for (int j = 0; j < 4; ++j) lo[j] = t[i][j] * scale, hi[j] = t[i][4 + j] * scale;
        out[32 * at + sub] = lo;
        out[32 * at + 16 + sub] = hi;
    }
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
    const long blocks = (long)N * (K / 128), per_wg = kRotateWidth * kRotateBlocks;
    hipLaunchKernelGGL(rotate_weight_blocks, dim3((unsigned)((blocks + per_wg - 1) / per_wg)), dim3(kQuantThreads), 0,
                       stream, (const float4v*)w, (const float4v*)chan_s, (float4v*)w_rot, blocks, K / 128);
    return hipGetLastError();
}

}  // namespace vq
