// The int8 (and packed 4-bit, and fp16 comparison) GEMM with the dequantization epilogue:
// the 256 x 256 workgroup tile of the kernel template in vq_gemm_kernel.h, and the choice
// between it, the 256 x 192 tile (vq_gemm_192.hip) and the smaller tiles of vq_gemm_tiles.hip and
// vq_gemm_split.hip for a given problem.
#include "vq_gemm_kernel.h"

namespace vq {

namespace {
typedef TileShape<2, 4, 4> Tile256;  // 2 x 4 wavefronts of 128 tokens x 64 channels

// How long a launch takes, in microseconds.  Tiles that all wavefronts of a workgroup share: `base`, plus for
// every time a CU is filled with `per_cu` workgroups fixed + stage * (stages of 128 bytes of K), plus the
// same of a last filling with one workgroup only; widen is what 4-bit weights add to a stage.
// Both tables fitted by least squares over 20000 random problems (1 to 32768 tokens, 32 to 4608 channels, K 256
// to 4608, 8- and 4-bit weights), each timed with every tile in captured graphs, where the tile was within
// 15 % of the best: error 6 to 9 %.  Over those problems the tile chosen is on average 0.2 % (above 1e9
// multiply-adds) and 0.7 % (below 6e9) slower than the best one.
struct TileCost {
    int tile_t, tile_c, per_cu;
    double base, fixed, stage, widen, fixed_one, stage_one, widen_one;
};
constexpr TileCost kTileCosts[] = {
    {64, 64, 2, 2.210, 1.940, 0.361, 0.067, 1.068, 0.215, 0.065},
    {128, 64, 2, 2.671, 3.085, 0.516, 0.018, 1.419, 0.339, 0.023},
    {128, 128, 1, 1.710, 4.068, 0.471, 0.011, 0.0, 0.0, 0.0},
    {128, 256, 1, 2.127, 4.866, 0.778, 0.079, 0.0, 0.0, 0.0},
    {256, 192, 1, 2.571, 4.325, 1.131, 0.0, 0.0, 0.0, 0.0},
    {256, 256, 1, 2.177, 5.544, 1.325, 0.0, 0.0, 0.0, 0.0},
};
// Tiles whose K the `waves` wavefronts of a workgroup divide: `base`, plus for every workgroup of a CU `fixed`
// and, per line of K, `line` and `load` for every 8 KiB that it loads, plus `turn` for every line that a
// wavefront takes in each filling.
struct SplitCost {
    int tile_t, tile_c, waves, per_cu;
    double base, fixed, load, turn, line;
};
constexpr SplitCost kSplitCosts[] = {
    {32, 32, 8, 2, 2.6057, 0.4853, 0.0430, 0.0, 0.0268},
    {64, 32, 4, 3, 2.6815, 0.3912, 0.0646, 0.1748, 0.0119},
    {32, 32, 3, 4, 2.6742, 0.1803, 0.0448, 0.1433, 0.0166},
    {64, 64, 8, 1, 0.7061, 3.1354, 0.0908, 0.0, 0.0123},
    {32, 32, 6, 3, 2.6642, 0.3712, 0.0372, 0.0, 0.0346},
};

// Workgroups of the busiest CU: every XCD takes an equal run of tiles.
long tiles_per_cu(int M, int N, int tile_t, int tile_c, int num_cus) {
    const long tiles = (((long)M + tile_t - 1) / tile_t) * (((long)N + tile_c - 1) / tile_c);
    const long per_xcd = (tiles + kXcds - 1) / kXcds;
    const int cus_per_xcd = num_cus >= kXcds ? num_cus / kXcds : 1;
    return (per_xcd + cus_per_xcd - 1) / cus_per_xcd;
}

double launch_cost(const TileCost& c, int w_bits, int M, int N, int K, int num_cus) {
    const long rounds = tiles_per_cu(M, N, c.tile_t, c.tile_c, num_cus);
    const double nk = (double)((K + kTileK - 1) / kTileK), wide = w_bits == 4 ? 1.0 : 0.0;
    double t = c.base + (double)(rounds / c.per_cu) * (c.fixed + (c.stage + wide * c.widen) * nk);
    if (rounds % c.per_cu) t += c.fixed_one + (c.stage_one + wide * c.widen_one) * nk;
    return t;
}

double launch_cost(const SplitCost& c, int w_bits, int M, int N, int K, int num_cus) {
    const long rounds = tiles_per_cu(M, N, c.tile_t, c.tile_c, num_cus), nl = (K + kTileK - 1) / kTileK;
    const double loaded = ((M < c.tile_t ? M : c.tile_t) + c.tile_c * w_bits / 8.0) / 64.0;   // (rows past M are not loaded)
    return c.base + (double)rounds * (c.fixed + (double)nl * (c.line + c.load * loaded)) +
           (double)((rounds + c.per_cu - 1) / c.per_cu * ((nl + c.waves - 1) / c.waves)) * c.turn;
}
}  // namespace

// The cheapest of the tiles that one launch takes.  (The persistent kernel's grid does not grow with the problem.)
GemmChoice choose_gemm(int w_bits, int M, int N, int K, int num_cus) {
    GemmChoice best{0, 0, 0};
    double best_cost = 0.0;
    for (const TileCost& c : kTileCosts) {
        if (c.tile_t != 256 && (w_bits == 16 || !tiles_launchable(M, N, c.tile_t, c.tile_c, kSharedTileThreads)))
            continue;  // (the fp16 layer has the persistent kernel only)
        // fp16: rounds of tiles, the narrower tile (a sixth more operand bytes per multiply-add) only where it saves some
        const double cost = w_bits == 16 ? (double)tiles_per_cu(M, N, 256, c.tile_c, num_cus) * c.tile_c * (c.tile_c == 192 ? 1.05 : 1.0)
                                         : launch_cost(c, w_bits, M, N, K, num_cus);
        if (!best.tile_t || cost <= best_cost) {
            best = {c.tile_t, c.tile_c, 0};
            best_cost = cost;
        }
    }
    if (w_bits != 16)
        for (const SplitCost& c : kSplitCosts) {
            if (!tiles_launchable(M, N, c.tile_t, c.tile_c, 64 * c.waves)) continue;
            const double cost = launch_cost(c, w_bits, M, N, K, num_cus);
            if (cost < best_cost) {
                best = {c.tile_t, c.tile_c, c.waves};
                best_cost = cost;
            }
        }
    return best;
}

hipError_t launch_gemm(const int8_t* xq, const float* x_scale, const void* w, int w_bits,
                       const float* w_scale, const void* bias_f16, void* y_f16, int32_t* acc_out,
                       int M, int N, int K, int num_cus, hipStream_t stream) {
    const GemmChoice c = choose_gemm(w_bits, M, N, K, num_cus);
    if (c.waves || c.tile_t != 256) {
        TileArgs t{};
        t.xq = xq;
        t.x_scale = x_scale;
        t.w = w;
        t.w_scale = w_scale;
        t.bias = (const _Float16*)bias_f16;
        t.y = (_Float16*)y_f16;
        t.acc_out = acc_out;
        t.M = M;
        t.N = N;
        t.K = K;
        if (c.waves) return launch_gemm_split(c.tile_t, c.tile_c, c.waves, t, w_bits, stream);
        return launch_gemm_tiles(c.tile_t, c.tile_c, t, w_bits, stream);
    }
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
    if (c.tile_c == 192) return launch_gemm_192(a, w_bits, num_cus, stream);
    return launch_gemm_shape<Tile256>(a, w_bits, num_cus, stream);
}

}  // namespace vq

extern "C" void vq_internal_gemm_choice(int w_bits, int M, int N, int K, int num_cus, int choice[3]) {
    const vq::GemmChoice c = vq::choose_gemm(w_bits, M, N, K, num_cus);
    choice[0] = c.tile_t;
    choice[1] = c.tile_c;
    choice[2] = c.waves;
}

extern "C" int vq_internal_gemm_out(int N, const void* y, const void* acc_out) { return vq::rows_out(N, y, acc_out); }
