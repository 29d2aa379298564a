// The 256 x 192 workgroup tile of the GEMM kernel template (vq_gemm_kernel.h): 4 x 3
// wavefronts of 64 tokens x 64 channels, three per SIMD.  For channel counts that tiles of
// 256 channels cover badly: a DiT hidden size of 1152 is 6 x 192 but 4.5 x 256.
// With 4-bit weights that tile is another kernel's, vq_gemm_192w4.hip.
#include "vq_gemm_kernel.h"

namespace vq {

namespace {
typedef TileShape<4, 3, 4, false> Tile192;
typedef TileShape<4, 3, 4, false, 2> Tile192TwoStages;
}

// Two stages of activations in LDS where K is no more than four: the way to a third is as long as what it hides.  Time with two
// over that with three, 420 random problems, mean by stages of K, 8-bit weights: 0.96 at one, 0.98 at two and three, 0.99 at four,
// 1.00 at five, 1.01 at six to eight, 1.07 from 17 on; fp16 operands 0.94, 0.97, 0.97, 0.97, 0.98 at five (up to 1.03), 1.00 at
// eight to ten, 1.06 from 20 on.  us, three / two: 8355 x 96 -> 1152 7.36 / 6.92, 14459 x 112 -> 4608 33.4 / 32.3, 2671 x 384 ->
// 3456 9.5 / 9.2, fp16 331 x 96 -> 3456 6.59 / 6.32; 8192 x 4608 -> 1152 40.5 / 42.7.
hipError_t launch_gemm_192(const GemmArgs& a, int w_bits, int num_cus, hipStream_t stream) {
    if (w_bits == 4) return launch_gemm_192w4(a, num_cus, stream);
    if ((w_bits == 16 ? 2l : 1l) * a.K <= 4 * kTileK) return launch_gemm_shape<Tile192TwoStages>(a, w_bits, num_cus, stream);
    return launch_gemm_shape<Tile192>(a, w_bits, num_cus, stream);
}

}  // namespace vq
