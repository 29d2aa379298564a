// The layer of few tokens in one launch (vq_linear_small.h): the rule and the entry.
#include "vq_linear_small.h"

namespace vq {

// Every workgroup has a CU to itself, so the line is drawn at their number; with more of them some would wait for
// a second round of everything.  Beyond 256 x 1152 tiles x K (rows above 1152 channels) the residual layer, which also
// reads the branch and writes the sum, is no faster.  Over 31000 problems of 1 to 256 tokens, K 256 to 1536 and 32 to
// 4608 channels, in captured graphs, one launch takes of the two launches' time (mean, 98th percentile; in the last
// quarter before the line)
//   plain 0.75, 0.90; 0.81, 0.94    GELU 0.79, 0.95; 0.89, 1.00    residual 0.80, 1.01; 0.90, 1.05    Hadamard 0.82, 0.98;
//   0.89, 1.03,
// and beside that one launch less is 2.8 us less of the host's time.
bool small_layer(int producer, int M, int N, int K, int num_cus) {
    if (producer == kLayerNorm || K > kSmallNch * kSmallLanes * 8) return false;
    const long tiles = (long)((M + kSmallTokens - 1) / kSmallTokens) * ((N + kSmallChannels - 1) / kSmallChannels);
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
