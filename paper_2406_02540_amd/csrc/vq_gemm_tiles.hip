// The one-tile-per-workgroup GEMM kernel (vq_gemm_tiles_kernel.h) in its five tile sizes, for
// problems that the persistent kernel's tiles of 256 tokens would not fill the chip with.
#include "vq_gemm_tiles_kernel.h"

namespace vq {

namespace {
// Four wavefronts of 32 x 32 that split the K steps four ways (32 x 32); eight that split them two ways, of 32 x 32 (64 x 64),
// 32 x 64 (128 x 64) or 64 x 64 (128 x 128); and eight of 64 x 64 that share them (128 x 256).  The first three leave room
// for a second workgroup on the CU; the ring is as deep as the LDS allows.  Where a wavefront has two blocks of channels its
// outputs leave from the registers.  128 x 64 with 4-bit weights has wavefronts of 64 x 32: of 32 x 64 each would widen
// twice as many weights (2048 x 1152 -> 1152 9.4 us, 9.8 so; with 8-bit weights 9.3 and 8.6).
// 32 x 32 is for few lines of K, of which the tiles whose wavefronts divide K leave some without work: at K to 128 it is the
// best one, by 4 to 5 %, for four problems in ten, at K to 512 for one in fifteen.
typedef OneTile<1, 1, 1, 1, 4, 8, 2> Tile32x32;
typedef OneTile<2, 2, 1, 1, 2, 4, 2> Tile64x64;
typedef OneTile<4, 1, 1, 2, 2, 3, 2> Tile128x64;
typedef OneTile<2, 2, 2, 1, 2, 3, 2> Tile128x64W4;
typedef OneTile<2, 2, 2, 2, 2, 4, 1> Tile128x128;
typedef OneTile<2, 4, 2, 2, 1, 3, 1> Tile128x256;

template <class S>
hipError_t launch_bits(const TileArgs& a, int w_bits, hipStream_t stream) {
    return w_bits == 8 ? launch_tile_shape<S, 8>(a, stream) : launch_tile_shape<S, 4>(a, stream);
}
}  // namespace

hipError_t launch_gemm_tiles(int tile_t, int tile_c, const TileArgs& a, int w_bits, hipStream_t stream) {
    if (tile_t == 32 && tile_c == 32) return launch_bits<Tile32x32>(a, w_bits, stream);
    if (tile_t == 64 && tile_c == 64) return launch_bits<Tile64x64>(a, w_bits, stream);
    if (tile_t == 128 && tile_c == 64)
        return w_bits == 8 ? launch_tile_shape<Tile128x64, 8>(a, stream) : launch_tile_shape<Tile128x64W4, 4>(a, stream);
    if (tile_t == 128 && tile_c == 128) return launch_bits<Tile128x128>(a, w_bits, stream);
    if (tile_t == 128 && tile_c == 256) return launch_bits<Tile128x256>(a, w_bits, stream);
    return hipErrorInvalidValue;
}

}  // namespace vq
