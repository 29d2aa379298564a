// The layer of few tokens in one launch (vq_linear_small.h): the rule and the entry.
#include "vq_linear_small.h"

namespace vq {

// Every workgroup has a CU to itself, so the line is drawn at their number; with more of them some would wait for
// a second round of everything.  Rows above 1152 channels end at 256 x 1152 tiles x K.  In captured graphs of 24 layers of 1
// to 300 tokens, K 256 to 1536 and 32 to 4608 channels, 300 to 500 problems each, one launch takes of the two launches' time
// (mean, 98th percentile), with every layer's weights in L2, in the memory-side cache and in memory,
//   plain         0.78, 0.84    0.86, 0.98    0.84, 0.96
//   GELU tanh     0.82, 0.91    0.91, 1.10    0.87, 1.02
//   GELU erf      0.73, 0.93    0.82, 1.07    0.80, 1.00
//   residual      0.80, 0.93    0.90, 1.10    0.85, 1.03
//   Hadamard      0.84, 0.93    0.94, 1.11    0.90, 1.02.
// The slower ones are rows above 1280 channels behind a producer, with weights in the memory-side cache (1.00, 1.13; in L2
// 0.89, 0.95, in memory 0.95, 1.06): a line of 96, 128 or 160 x 1152 for those rows gave up more in the other two states than
// it won there.  Called one by one such layers took 6.5 us where two launches had taken 8.0: a launch is 2.1 us of the host's time.
bool small_layer(int producer, int M, int N, int K, int num_cus) {
    if (producer == kLayerNorm || K > kSmallNch * kSmallLanes * 8) return false;
    const long tiles = (((long)M + kSmallTokens - 1) / kSmallTokens) * (((long)N + kSmallChannels - 1) / kSmallChannels);
    return tiles <= num_cus && tiles * K <= 256l * 1152;
}

hipError_t launch_linear_small(const ProducerArgs& p, const void* w, int w_bits, const float* w_scale, const void* bias_f16,
                               void* y_f16, int M, int N, int K, hipStream_t stream) {
    SmallArgs a{};
    a.t.w = w;
    a.t.w_scale = w_scale;
    a.t.bias = (const _Float16*)bias_f16;
    a.t.y = (_Float16*)y_f16;
    a.t.M = M;
    a.t.N = N;
    a.t.K = K;
    a.f = fused_args(p, nullptr, nullptr, M, K);
    switch (p.producer) {
        case kPlain: return launch_small_producer<kPlain>(a, w_bits, stream);
        case kGeluErf: return launch_small_producer<kGeluErf>(a, w_bits, stream);
        case kGeluTanh: return launch_small_producer<kGeluTanh>(a, w_bits, stream);
        case kResidual: return launch_small_producer<kResidual>(a, w_bits, stream);
        case kHadamard: return launch_small_producer<kHadamard>(a, w_bits, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace vq
