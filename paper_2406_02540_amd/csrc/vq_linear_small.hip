// The layer of few tokens in one launch (vq_linear_small.h): the rule and the entry.
#include "vq_linear_small.h"

namespace vq {

// The one launch costs what every workgroup's quantizer and the weights that are read again by every
// eight tokens add up to, so the line is drawn at tiles x K.  Over 1100 problems of 1 to 256 tokens, K 256
// to 1152 and 128 to 4608 channels, in captured graphs, one launch is faster by (mean; above half of the
// line; worst)
//   plain     23 %; 11 %; -2 %   with tiles x K up to 256 x 1152,
//   GELU      18 %; 10 %; -2 %   and
//   Hadamard  13 %;  8 %; -3 %    up to 160 x 1152,
//   residual  16 %; 11 %; -6 %    up to 96 x 1152 (it also reads the branch and writes the sum),
// and beside that one launch less is 2 us less of the host's time.  Beyond num_cus workgroups some wait.
bool small_layer(int producer, int M, int N, int K, int num_cus) {
    if (producer == kLayerNorm || K > kSmallNch * kSmallLanes * 8) return false;
    const long tiles = (long)((M + kSmallWaves - 1) / kSmallWaves) * ((N + SmallTile::kC - 1) / SmallTile::kC);
    const int line = producer == kPlain ? 256 : producer == kResidual ? 96 : 160;
    return tiles <= num_cus && tiles * K <= (long)line * 1152;
}

hipError_t launch_linear_small(const ProducerArgs& p, const void* w, int w_bits, const float* w_scale, const void* bias_f16,
                               void* y_f16, int M, int N, int K, hipStream_t stream) {
    TileArgs t{};
    t.w = w;
    t.w_scale = w_scale;
    t.bias = (const _Float16*)bias_f16;
    t.y = (_Float16*)y_f16;
    t.M = M;
    t.N = N;
    t.K = K;
    const FusedArgs f = fused_args(p, nullptr, nullptr, M, K);
    switch (p.producer) {
        case kPlain: return launch_small_producer<kPlain>(t, f, w_bits, stream);
        case kGeluErf: return launch_small_producer<kGeluErf>(t, f, w_bits, stream);
        case kGeluTanh: return launch_small_producer<kGeluTanh>(t, f, w_bits, stream);
        case kResidual: return launch_small_producer<kResidual>(t, f, w_bits, stream);
        case kHadamard: return launch_small_producer<kHadamard>(t, f, w_bits, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace vq
