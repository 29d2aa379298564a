// The int8 (and packed 4-bit, and fp16 comparison) GEMM with the dequantization epilogue:
// the 256 x 256 workgroup tile of the kernel template in vq_gemm_kernel.h, and the choice
// between it, the 256 x 192 tile (vq_gemm_192.hip) and the smaller tiles of
// vq_gemm_tiles.hip for a given problem.
#include "vq_gemm_kernel.h"

namespace vq {

namespace {
typedef TileShape<2, 4, 4> Tile256;  // 2 x 4 wavefronts of 128 tokens x 64 channels

// How long a launch takes, in microseconds: `base`, plus for every time a CU is filled with
// `per_cu` workgroups fixed + stage * (stages of 128 bytes of K), plus the same of a last filling
// with one workgroup only.  Fitted by least squares over 720 random problems (1 to 12000 tokens, 32
// to 4608 channels, K 256 to 4608, 8- and 4-bit weights), each timed with every tile in captured
// graphs: mean error 6 to 11 %.  On another 22000 problems of the same ranges (M to 32768), with the kernels
// as they are, the tile chosen by it is on average 0.4 % slower than the best one of each problem.
struct TileCost {
    int tile_t, tile_c, per_cu;
    double base, fixed, stage, fixed_one, stage_one;
};
constexpr TileCost kTileCosts[] = {
    {32, 32, 2, 2.08, 2.01, 0.194, 1.50, 0.147},
    {64, 64, 2, 2.24, 2.69, 0.376, 1.49, 0.213},
    {128, 64, 2, 2.31, 3.69, 0.566, 1.76, 0.321},
    {128, 128, 1, 0.0, 4.90, 0.413, 0.0, 0.0},
    {128, 256, 1, 0.0, 5.40, 0.692, 0.0, 0.0},
    {256, 192, 1, 0.0, 5.91, 0.966, 0.0, 0.0},
    {256, 256, 1, 0.0, 7.16, 1.000, 0.0, 0.0},
};

// Workgroups of the busiest CU: every XCD takes an equal run of tiles.
long tiles_per_cu(int M, int N, int tile_t, int tile_c, int num_cus) {
    const long tiles = (long)((M + tile_t - 1) / tile_t) * ((N + tile_c - 1) / tile_c);
    const long per_xcd = (tiles + kXcds - 1) / kXcds;
    const int cus_per_xcd = num_cus >= kXcds ? num_cus / kXcds : 1;
    return (per_xcd + cus_per_xcd - 1) / cus_per_xcd;
}

double launch_cost(const TileCost& c, int M, int N, int K, int num_cus) {
    const long rounds = tiles_per_cu(M, N, c.tile_t, c.tile_c, num_cus);
    const long nk = (K + kTileK - 1) / kTileK;
    double t = c.base + (double)(rounds / c.per_cu) * (c.fixed + c.stage * (double)nk);
    if (rounds % c.per_cu) t += c.fixed_one + c.stage_one * (double)nk;
    return t;
}
}  // namespace

hipError_t launch_gemm(const int8_t* xq, const float* x_scale, const void* w, int w_bits,
                       const float* w_scale, const void* bias_f16, void* y_f16, int32_t* acc_out,
                       int M, int N, int K, int num_cus, hipStream_t stream) {
    const TileCost* best = nullptr;
    double best_cost = 0.0;
    for (const TileCost& c : kTileCosts) {
        if (w_bits == 16 && c.tile_t != 256) continue;  // (the fp16 layer has the persistent kernel only)
        // fp16: rounds of tiles, the narrower tile (a sixth more operand bytes per multiply-add) only where it saves some
        const double cost = w_bits == 16 ? (double)tiles_per_cu(M, N, 256, c.tile_c, num_cus) * c.tile_c * (c.tile_c == 192 ? 1.05 : 1.0)
                                         : launch_cost(c, M, N, K, num_cus);
        if (!best || cost <= best_cost) {
            best = &c;
            best_cost = cost;
        }
    }
    if (best->tile_t != 256)
        return launch_gemm_tiles(best->tile_t, best->tile_c, xq, x_scale, w, w_bits, w_scale, bias_f16, y_f16, acc_out, M, N,
                                 K, stream);
    GemmArgs a;
    a.xq = xq;
    a.x_scale = x_scale;
    a.w = w;
    a.w_scale = w_scale;
    a.bias = (const _Float16*)bias_f16;
    a.y = (_Float16*)y_f16;
    a.acc_out = acc_out;
    a.M = M;
    a.N = N;
    a.K = K;
    a.tiles_t = a.tiles_c = a.tiles = a.tiles_per_xcd = a.slots = 0;  // (set for the chosen tile)
    if (best->tile_c == 192) return launch_gemm_192(a, w_bits, num_cus, stream);
    return launch_gemm_shape<Tile256>(a, w_bits, num_cus, stream);
}

}  // namespace vq
