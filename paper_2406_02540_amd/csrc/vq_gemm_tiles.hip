// The one-tile-per-workgroup GEMM kernel (vq_gemm_tiles_kernel.h) in its five tile sizes, for
// problems that the persistent kernel's tiles of 256 tokens would not fill the chip with.
#include "vq_gemm_tiles_kernel.h"

namespace vq {

namespace {
// Four wavefronts of 32 x 32 that split K four ways (32 x 32), eight that split it two ways (64 x
// 64, 128 x 64, 128 x 128), eight of 64 x 64 (128 x 256).  The first three leave room for a second
// workgroup on the CU; the ring is as deep as the LDS allows.
typedef OneTile<1, 1, 1, 1, 4, 8, 2> Tile32x32;
typedef OneTile<2, 2, 1, 1, 2, 4, 2> Tile64x64;
typedef OneTile<2, 2, 2, 1, 2, 3, 2> Tile128x64;
typedef OneTile<2, 2, 2, 2, 2, 4, 1> Tile128x128;
typedef OneTile<2, 4, 2, 2, 1, 3, 1> Tile128x256;

template <class S>
hipError_t launch_bits(const TileArgs& a, int w_bits, hipStream_t stream) {
    return w_bits == 8 ? launch_tile_shape<S, RowsOfCodes, 8>(a, {}, stream) : launch_tile_shape<S, RowsOfCodes, 4>(a, {}, stream);
}
}  // namespace

hipError_t launch_gemm_tiles(int tile_t, int tile_c, const int8_t* xq, const float* x_scale, const void* w, int w_bits,
                             const float* w_scale, const void* bias_f16, void* y_f16, int32_t* acc_out,
                             int M, int N, int K, hipStream_t stream) {
    TileArgs a;
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
    a.tiles_t = a.tiles_c = a.tiles = a.tiles_per_xcd = 0;  // (set for the chosen tile)
    a.div_band = a.div_last = 0;
    if (tile_t == 32 && tile_c == 32) return launch_bits<Tile32x32>(a, w_bits, stream);
    if (tile_t == 64 && tile_c == 64) return launch_bits<Tile64x64>(a, w_bits, stream);
    if (tile_t == 128 && tile_c == 64) return launch_bits<Tile128x64>(a, w_bits, stream);
    if (tile_t == 128 && tile_c == 128) return launch_bits<Tile128x128>(a, w_bits, stream);
    if (tile_t == 128 && tile_c == 256) return launch_bits<Tile128x256>(a, w_bits, stream);
    return hipErrorInvalidValue;
}

}  // namespace vq
