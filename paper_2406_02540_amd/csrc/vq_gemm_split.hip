// The GEMM kernel whose wavefronts divide K (vq_gemm_split.h) in its tile sizes, for problems of few or
// small tiles.
#include "vq_gemm_split.h"

namespace vq {

namespace {
// (as many workgroups to a CU as their LDS lets in)
typedef SplitTile<1, 1, 3, 4> Split32Waves3;
typedef SplitTile<1, 1, 6, 3> Split32Waves6;
typedef SplitTile<1, 1, 8, 2> Split32Waves8;
typedef SplitTile<2, 1, 4, 3> Split64x32;
typedef SplitTile<2, 2, 8, 1> Split64x64;
typedef SplitTile<3, 3, 8, 1, 16> Split48x48;

template <class S>
hipError_t launch_bits(const TileArgs& a, int w_bits, hipStream_t stream) {
    return w_bits == 8 ? launch_split_tile<S, 8>(a, stream) : launch_split_tile<S, 4>(a, stream);
}
}  // namespace

hipError_t launch_gemm_split(int tile_t, int tile_c, int waves, const TileArgs& a, int w_bits, hipStream_t stream) {
    if (tile_t == 32 && tile_c == 32 && waves == 3) return launch_bits<Split32Waves3>(a, w_bits, stream);
    if (tile_t == 32 && tile_c == 32 && waves == 6) return launch_bits<Split32Waves6>(a, w_bits, stream);
    if (tile_t == 32 && tile_c == 32 && waves == 8) return launch_bits<Split32Waves8>(a, w_bits, stream);
    if (tile_t == 64 && tile_c == 32 && waves == 4) return launch_bits<Split64x32>(a, w_bits, stream);
    if (tile_t == 64 && tile_c == 64 && waves == 8) return launch_bits<Split64x64>(a, w_bits, stream);
    if (tile_t == 48 && tile_c == 48 && waves == 8) return launch_bits<Split48x48>(a, w_bits, stream);
    return hipErrorInvalidValue;
}

}  // namespace vq
