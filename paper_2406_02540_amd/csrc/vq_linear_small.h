// A layer of few tokens in one launch: the one-tile-per-workgroup GEMM (vq_gemm_tiles_kernel.h) whose
// workgroups quantize their tokens themselves (vq_fused_kernel.h), straight into the LDS operand
// layout.  ViDiT-Q Sec. 5.1 integrates the quantizer into the operation in front of it; this
// integrates both into the GEMM.
//
// Two launches of such a layer are two latencies (2.4 us for the quantizer, 3.9 for the GEMM) around
// less than a microsecond of work each.  In one launch every workgroup of the same tokens quantizes
// them again while its first seven stages of weights are on their way: eight tokens, one per
// wavefront, so that this takes a wavefront 300 to 450 vector instructions (with 32 tokens per
// workgroup, 16 lanes each, it took longer than the launch that it saves: 32 x 1152 -> 1152 9.6 us when
// two launches were 7.5).  The matrix cores work on blocks a quarter full.
// One launch against two in a captured graph, us: 1 x 1152 -> 1152 5.1 / 6.3 (4-bit weights 5.8 / 6.9),
// 8 x 1152 -> 4608 6.3 / 6.7, 32 x 1152 -> 1152 5.5 / 6.7, 64 x 512 -> 320 4.3 / 5.2; at one token GELU
// 5.6 / 6.9, Hadamard 5.9 / 7.2, residual 5.9 / 7.4.
//
// LayerNorm is not among them: its sums keep the order of the stand-alone kernel's lanes (32 for 1152
// channels), and sixteen tokens of two passes each per workgroup were 5 to 15 % slower than two launches.
#pragma once
#include "vq_fused_kernel.h"
#include "vq_gemm_tiles_kernel.h"

namespace vq {
namespace {

constexpr int kSmallWaves = 8;

// Codes and scales of a wavefront's tokens into the workgroup's LDS: 128-byte stage blocks of [ROWS][128],
// 16-byte pieces XOR-ed by (row/2)%8, as the ring's loads would have laid them out.
template <int ROWS>
struct RowsInLds {
    int8_t* x;
    float* x_scale;
    int row0;   // the wavefront's first token within the tile
    __device__ __forceinline__ void scale(int token, float s) const { x_scale[row0 + token] = s; }
    __device__ __forceinline__ void codes(int token, int chunk, bool exists, int2v o) const {
        if (!exists) return;
        const int row = row0 + token;
        *(int2v*)(x + (chunk >> 4) * (ROWS * kStageK) + row * kStageK + ((((chunk >> 1) & 7) ^ ((row >> 1) & 7)) << 4) +
                  (chunk & 1) * 8) = o;
    }
};

// A wavefront takes 64 / LANES tokens of at most NCH chunks per lane.
template <int PRODUCER, int NCH, int LANES>
struct Quantizes {
    typedef FusedArgs Args;
    static constexpr bool kQuantizes = true;
    static constexpr int kRows = kSmallWaves * (kWave / LANES);
    static constexpr int kMaxK = NCH * LANES * 8;
    static constexpr int kXBytes = kRows * ((kMaxK + kStageK - 1) / kStageK) * kStageK;
    template <int KT>
    static __device__ __forceinline__ void quantize(const Args& a, long tok0, int wave, bool writes_r, int8_t* lds_x,
                                                    float* lds_scale) {
        const int row0 = wave * (kWave / LANES);
        if (tok0 + row0 >= a.M) return;   // (uniform)
        const RowsInLds<kRows> out{lds_x, lds_scale, row0};
        produce_and_quantize<PRODUCER, NCH, LANES, false>(a, tok0 + row0, threadIdx.x & (kWave - 1), writes_r, VectorsFromMemory<>{}, out);
    }
};

// Eight wavefronts: two of 32 tokens x 32 channels, times four groups that split K; seven stages of weights in flight.
typedef OneTile<1, 2, 1, 1, 4, 8, 1> SmallTile;
static_assert(SmallTile::kWaves == kSmallWaves, "every wavefront quantizes");
constexpr int kSmallNch = 3, kSmallLanes = 64;   // a token of up to 1536 channels per wavefront

template <int PRODUCER>
hipError_t launch_small_producer(const TileArgs& t, const FusedArgs& f, int w_bits, hipStream_t stream) {
    typedef Quantizes<PRODUCER, kSmallNch, kSmallLanes> Rows;
    return w_bits == 8 ? launch_tile_shape<SmallTile, Rows, 8>(t, f, stream) : launch_tile_shape<SmallTile, Rows, 4>(t, f, stream);
}

}  // namespace
}  // namespace vq
