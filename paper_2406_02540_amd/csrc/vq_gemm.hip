// The int8 (and packed 4-bit, and fp16 comparison) GEMM with the dequantization epilogue:
// the 256 x 256 workgroup tile of the kernel template in vq_gemm_kernel.h, and the choice
// between it, the 256 x 192 tile (vq_gemm_192.hip) and the smaller tiles of vq_gemm_tiles.hip and
// vq_gemm_split.hip for a given problem.
#include "vq_gemm_kernel.h"

namespace vq {

namespace {
typedef TileShape<2, 4, 8, true> Tile256;  // 2 x 4 wavefronts of 128 tokens x 64 channels

// How long a launch takes, in microseconds: `base`; for every MB that moves once, of activations, outputs and weights,
// and for every MB of operands that all the tiles together ask for (Traffic); and what the busiest CU spends on its
// workgroups.  Where all wavefronts share the tile that is, for every time the CU is filled with `per_cu` workgroups, fixed +
// stage * (stages of 128 bytes of K), plus the same of a last filling with one workgroup only; widen is what 4-bit weights
// add to a stage.  Where the `waves` wavefronts divide K it is `fixed` for every workgroup and, for every line of K, `line` and
// `load` for every 8 KiB of it; and in every filling `fill` and `turn` for each line that a wavefront takes.
//
// Fitted to 14000 random problems (1 to 65536 tokens, 8 to 16384 channels, K 16 to 8192, most within 32768, 4608 and 256 to
// 4608; 8- and 4-bit weights), each timed with every tile in captured graphs: by least squares where a tile was within 25 % of
// the best, then by descent on what the tile chosen costs over the best one.  The kernels were those before outputs left from
// the registers, which made 128 x 256 15 % faster on average, 128 x 128 8 %, 128 x 64 with 8-bit weights 4 %, the persistent tiles
// 4 to 8 % (and 3 to 10 % again since, in blocks of 16x16x64), the others 1 % at most.  19580 other problems between those two
// changes, the chosen one timed in each: over the best one on average (98th percentile) 0.7 % (6 %) below 1e8 multiply-adds, 0.8 %
// (8 %) to 1e9, 0.9 % (8 %) to 6e9 and 0.1 % (3 %) above; with many tokens and few channels (8 to 400) 1.4 % (11 %).  With the
// kernels as they are, 1300 problems that take 128 x 128 or larger: 0.2 % (4 %) with 8-bit weights, 0.1 % (2 %) with 4-bit,
// nothing with fp16 operands; 256 x 256 is taken in 3 of 162 where 256 x 192 is 3 to 5 % faster (29853 x 1120 -> 1160 68.7 us and
// 65.5).
// Without the bytes, and fitted to problems few of which had few channels, the rule took 2.2 % (17 %) there: 17964 x 3744 -> 88
// 29.8 us in tiles of 32 x 32, 20.3 in 128 x 128.
struct Traffic { double x, y, w, l2; };
struct TileCost {
    int tile_t, tile_c, per_cu;
    double base, fixed, stage, widen, fixed_one, stage_one, widen_one;
    Traffic mb;
};
constexpr TileCost kTileCosts[] = {
    {32, 32, 2, 1.42, 1.47, 0.172, 0.0256, 0.71, 0.184, 0.0641, {0.0332, 0.0347, 0.0573, 0}},
    {64, 64, 2, 1.67, 2.01, 0.346, 0.0715, 0.801, 0.21, 0.0902, {0.027, 0.00705, 0.0277, 0}},
    {128, 64, 2, 2.25, 1.55, 0.566, 0.0288, 1.24, 0.24, 0.058, {0.0359, 0.0842, 0, 0.00432}},
    {128, 128, 1, 0.00486, 4.46, 0.308, 0.0528, 0, 0, 0, {0.027, 0.00585, 0, 0.0261}},
    {128, 256, 1, 0.226, 4.08, 0.548, 0.146, 0, 0, 0, {0.00305, 0.112, 0, 0.029}},
    {256, 192, 1, 1.75, 4.2, 0.721, 0.0922, 0, 0, 0, {0, 0.031, 0.14, 0.0366}},
    {256, 256, 1, 2.81, 2.96, 1.07, 0.0625, 0, 0, 0, {0, 0.108, 0.133, 0.0238}},
};
struct SplitCost {
    int tile_t, tile_c, waves, per_cu;
    double base, fixed, line, load, fill, turn;
    Traffic mb;
};
constexpr SplitCost kSplitCosts[] = {
    {32, 32, 3, 4, 2.03, 0.165, 0.00313, 0.00566, 0.00119, 0.267, {0.0345, 0.0123, 0.00271, 0.0223}},
    {32, 32, 6, 3, 1.83, 0.361, 0.0523, 0.0113, 0.274, 0, {0.0287, 0.0341, 0.00143, 0.0125}},
    {32, 32, 8, 2, 1.66, 0.586, 0.0218, 0.0189, 0.658, 0, {0.0227, 0.00199, 0, 0.0135}},
    {64, 32, 4, 3, 2.36, 0.00171, 0.035, 0.0401, 0.516, 0.0839, {0.0689, 0.262, 0, 0.00146}},
    {64, 64, 8, 1, 0.928, 2.44, 0.0467, 0.0338, 0, 0, {0.06, 0.188, 0.0218, 0.0144}},
};

// What of a problem the costs depend on.
struct Problem {
    int w_bits, M, N, K, cus_per_xcd;
    long lines;                    // of K
    bool small;                    // a launch of any tiles is below 2^32 threads
    double x_mb, y_mb, w_mb;
    Problem(int w_bits, int M, int N, int K, int num_cus)
        : w_bits(w_bits), M(M), N(N), K(K), cus_per_xcd(num_cus >= kXcds ? num_cus / kXcds : 1), lines((K + kTileK - 1) / kTileK),
          small((M / 32 + 1l) * (N / 32 + 1l) < (1l << 22)),
          x_mb((double)M * K * 1e-6), y_mb((double)M * N * 2e-6), w_mb((double)N * K * w_bits * 0.125e-6) {}
    long tiles(int t, int c) const { return (long)(((unsigned)M + t - 1) / t) * (((unsigned)N + c - 1) / c); }
    // Workgroups of the busiest CU: every XCD takes an equal run of tiles.
    long per_cu(long tiles) const { return ((tiles + kXcds - 1) / kXcds + cus_per_xcd - 1) / cus_per_xcd; }
    // bytes of a tile's operands per byte of K (rows past M not counted)
    double rows(int t, int c) const { return (M < t ? M : t) + c * w_bits * 0.125; }
    double traffic(const Traffic& mb, long tiles, double rows) const {
        return x_mb * mb.x + y_mb * mb.y + w_mb * mb.w + (double)tiles * rows * (double)lines * (kTileK * 1e-6) * mb.l2;
    }
};

double launch_cost(const TileCost& c, const Problem& p) {
    const long tiles = p.tiles(c.tile_t, c.tile_c), rounds = p.per_cu(tiles);
    const double nk = (double)p.lines, wide = p.w_bits == 4 ? 1.0 : 0.0;
    double t = c.base + (double)(rounds / c.per_cu) * (c.fixed + (c.stage + wide * c.widen) * nk);
    if (rounds % c.per_cu) t += c.fixed_one + (c.stage_one + wide * c.widen_one) * nk;
    return t + p.traffic(c.mb, tiles, p.rows(c.tile_t, c.tile_c));
}

double launch_cost(const SplitCost& c, const Problem& p) {
    const long tiles = p.tiles(c.tile_t, c.tile_c), rounds = p.per_cu(tiles);
    const double rows = p.rows(c.tile_t, c.tile_c);
    return c.base + (double)rounds * (c.fixed + (double)p.lines * (c.line + c.load * rows * (1.0 / 64.0))) +
           (double)((rounds + c.per_cu - 1) / c.per_cu) * (c.fill + c.turn * (double)((p.lines + c.waves - 1) / c.waves)) +
           p.traffic(c.mb, tiles, rows);
}

// The cheapest of the tiles that one launch takes.  (The persistent kernel's grid does not grow with the problem.)
GemmChoice cheapest_tile(int w_bits, int M, int N, int K, int num_cus) {
    const Problem p(w_bits, M, N, K, num_cus);
    GemmChoice best{0, 0, 0};
    double best_cost = 0.0;
#pragma unroll   // (the sizes are constants then: 0.07 us of host time, 0.13 with divisions by variables)
    for (const TileCost& c : kTileCosts) {
        if (c.tile_t != 256 && w_bits == 16) continue;  // (the fp16 layer has the persistent kernel only)
        if (c.tile_t != 256 && !p.small && !tiles_launchable(M, N, c.tile_t, c.tile_c, shared_tile_threads(c.tile_t))) continue;
        // fp16: rounds of tiles, the narrower tile (a sixth more operand bytes per multiply-add) only where it saves some
        const double cost = w_bits == 16 ? (double)p.per_cu(p.tiles(256, c.tile_c)) * c.tile_c * (c.tile_c == 192 ? 1.05 : 1.0)
                                         : launch_cost(c, p);
        if (!best.tile_t || cost <= best_cost) {
            best = {c.tile_t, c.tile_c, 0};
            best_cost = cost;
        }
    }
    if (w_bits != 16) {
#pragma unroll
        for (const SplitCost& c : kSplitCosts) {
            if (!p.small && !tiles_launchable(M, N, c.tile_t, c.tile_c, 64 * c.waves)) continue;
            const double cost = launch_cost(c, p);
            if (cost < best_cost) {
                best = {c.tile_t, c.tile_c, c.waves};
                best_cost = cost;
            }
        }
    }
    return best;
}

// Tiles of 48 x 48 in the place of one of 64 x 64 or 64 x 32, where they leave every CU one at most: such a launch waits for the
// CU's load path, and with 160 to 256 of them a CU asks for three quarters of the bytes of 64 x 64, of which there are 144.
// us, without / with: 240 x 4096 -> 2304 9.24 / 7.27 (4-bit weights 8.19 / 6.76), 1514 x 4000 -> 366 11.2 / 8.55, 128 x 4448 ->
// 3896 with 4-bit weights 9.86 / 8.0.  Over 1160 random problems, time with over time without: 0.83 where the 64 x 64 tile's
// wavefronts divide K (none above 0.95), 0.87 of 64 x 32's where K is 2048 at least and the tiles are a hundred (none above 0.97;
// below, up to 1.04 of it), 0.94 of the shared 64 x 64 tile's from twelve lines of K on (up to 1.13; 1.01 at ten and eleven, 1.07
// at nine, where the second turn is one wavefront's, 1.06 below).  The tiles of 32 x 32 stay: 1.11, 1.19 and 1.17 of three, six
// and eight wavefronts', 1.26 of the shared one's (0.91 in the 18 of 360 with three or eight where K is 1600 at least and the tiles
// of 48 x 48 are 170).
inline bool tiles_of_48(const GemmChoice& c, int M, int N, int K, int num_cus) {
    if (c.tile_t != 64) return false;
    const long tiles = (((long)M + 47) / 48) * (((long)N + 47) / 48);
    if ((tiles + kXcds - 1) / kXcds > (num_cus >= kXcds ? num_cus / kXcds : 1)) return false;
    if (c.tile_c == 64) return c.waves == 8 || K > 11 * kLine;
    return K >= 2048 && tiles >= 100;
}
}  // namespace

GemmChoice choose_gemm(int w_bits, int M, int N, int K, int num_cus) {
    const GemmChoice c = cheapest_tile(w_bits, M, N, K, num_cus);
    return w_bits != 16 && tiles_of_48(c, M, N, K, num_cus) ? GemmChoice{48, 48, 8} : c;
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
