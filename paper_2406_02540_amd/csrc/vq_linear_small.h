// A layer of few tokens in one launch: workgroups that quantize their tokens themselves
// (vq_fused_kernel.h), straight into the LDS operand layout, and multiply them like vq_gemm_split.h, every
// wavefront its own lines of K.  ViDiT-Q Sec. 5.1 integrates the quantizer into the operation in front of it;
// this integrates both into the GEMM.
//
// Two launches of such a layer are two latencies (2.4 us for the quantizer, 3.1 for the GEMM) around less than
// a microsecond of work each, and 2.1 us of host time each.  In one launch every workgroup of the same tokens
// quantizes them again: eight tokens, one per wavefront, so that this takes a wavefront 300 to 450 vector
// instructions.  The order is what counts: first the token and its per-channel vectors are asked for, then all the
// weights that the wavefront will need, so that the latency of the weights lies under the quantizer and the quantizer
// does not wait for the weights; then one barrier, and nothing is left to wait for.  The matrix cores work on blocks a
// quarter full.
// In a captured graph, us, with shared weight stages asked for ahead of the token / as it is (two launches: 5.7 at 1 x
// 1152 -> 1152): plain 1 x 1152 -> 1152 4.96 / 4.1 (4-bit weights 5.66 / 4.1), 8 x 1152 -> 4608 5.4 / 4.65, 32 x 1152 ->
// 1152 5.65 / 4.9 (5.85 / 4.6), 100 x 1152 -> 1152 6.2 / 5.3 (6.0 / 4.9), 64 x 512 -> 320 3.95 / 3.5; at one token GELU 5.4 /
// 4.55, Hadamard 6.1 / 4.85, residual 5.8 / 4.7.
//
// LayerNorm is not among them: its sums keep the order of the stand-alone kernel's lanes (32 for 1152
// channels).
#pragma once
#include "vq_fused_kernel.h"
#include "vq_gemm_common.h"

namespace vq {
namespace {

constexpr int kSmallWaves = 8, kSmallTokens = 8, kSmallChannels = 64;   // a token per wavefront
constexpr int kSmallNch = 3, kSmallLanes = 64;                          // of up to 1536 channels
constexpr int kSmallLines = kSmallNch * kSmallLanes * 8 / kLine, kSmallTurns = (kSmallLines + kSmallWaves - 1) / kSmallWaves;

// Codes and scales of a wavefront's token into the workgroup's LDS: lines of [tokens][128], 16-byte pieces
// XOR-ed by (row/2)%8, as direct loads would have laid them out.
struct RowsInLds {
    int8_t* x;
    float* x_scale;
    int row;   // the wavefront's token within the tile
    __device__ __forceinline__ void scale(int, float s) const { x_scale[row] = s; }
    __device__ __forceinline__ void codes(int, int chunk, bool exists, int2v o) const {
        if (!exists) return;
        *(int2v*)(x + (chunk >> 4) * (kSmallTokens * kLine) + row * kLine + ((((chunk >> 1) & 7) ^ ((row >> 1) & 7)) << 4) +
                  (chunk & 1) * 8) = o;
    }
};

// The per-channel vectors in registers, asked for with the token; behind() runs when all of that is on its
// way (the weights' loads, which complete behind it: memory answers in the order it was asked).
template <int PRODUCER, class Behind>
struct VectorsAsked {
    static constexpr bool kByChunk = false, kScale = true, kShift = true;
    static constexpr int kVecs = vector_count(PRODUCER);
    Behind behind;
    bool used[2];
    int sub, row;   // lane of the token; the sample whose gate it takes
    Vec8 v[kVecs][kSmallNch];
    __device__ __forceinline__ bool staged(int which) const { return which < kVecs; }
    __device__ __forceinline__ Vec8 chunk(int which, int, int i) const { return v[which < kVecs ? which : 0][i]; }
    template <class Rs>
    __device__ __forceinline__ void ask(const Rs& rs_cm, const Rs& rs_a, const Rs&, int K8) {
#pragma unroll
        for (int w = 0; w < kVecs; ++w)
            if (used[w])   // (uniform)
#pragma unroll
                for (int i = 0; i < kSmallNch; ++i) {
                    const int off = ((w == kVecMul ? 0 : row * K8) + min(i * kSmallLanes + sub, K8 - 1)) * 32;
                    v[w][i].lo = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(w == kVecMul ? rs_cm : rs_a, off, 0, 0));
                    v[w][i].hi = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(w == kVecMul ? rs_cm : rs_a, off + 16, 0, 0));
                }
    }
    __device__ __forceinline__ void park(int) {
        __builtin_amdgcn_sched_barrier(0);
        behind();
        __builtin_amdgcn_sched_barrier(0);
    }
};

struct SmallArgs {
    TileArgs t;
    FusedArgs f;
};

template <int PRODUCER, int W_BITS>
__global__ __launch_bounds__(64 * kSmallWaves, kSmallWaves / 4) void linear_small(const SmallArgs a) {
    constexpr int kWDiv = (W_BITS == 8) ? 1 : 2, kWLine = kSmallChannels * kLine / kWDiv, kSlot = kSmallTurns * kWLine;
    constexpr int kXBytes = kSmallTokens * kSmallLines * kLine;
    static_assert(kSlot >= kSmallTokens * kSmallChannels * 4, "a wavefront's sums take the place of its weights");
    __shared__ __attribute__((aligned(1024))) int8_t lds[kSmallWaves * kSlot + kXBytes];
    __shared__ float x_scale[kSmallTokens];
    int row, col;
    if (!locate_tile(a.t.grid, row, col)) return;
    const int tok0 = row * kSmallTokens, ch0 = col * kSmallChannels;   // (< M, < N)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int N = a.t.N, K = a.t.K;
    const int rows_w = min(kSmallChannels, N - ch0);
    const int nl = (K + kLine - 1) / kLine;
    int8_t* const lds_x = lds + kSmallWaves * kSlot;
    int8_t* const mine = lds + wave * kSlot;

    // A wavefront's lines of weights (wave and wave + 8): 8 rows x 128 B per load or, for packed nibbles, 16 rows x
    // 64 B, swizzled as everywhere; rows past N and pieces past K lie behind the buffer and arrive as zeros.
    // (Through the builtin: the waits for the token must not wait for these.)
    auto weights = [&]() __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc(
            (void*)((const int8_t*)a.t.w + (long)ch0 * (K / kWDiv)), 0, rows_w * (K / kWDiv), kRsrcFlags);
        constexpr int kRowsPer = 8 * kWDiv, kPieces = 8 / kWDiv, kLoads = kSmallChannels / kRowsPer;
#pragma unroll
        for (int t = 0; t < kSmallTurns; ++t) {
            const int k0 = (wave + t * kSmallWaves) * (kLine / kWDiv);
            if (t > 0 && wave + t * kSmallWaves >= nl) break;   // (uniform; the first turn always, so that the waits can count it)
#pragma unroll
            for (int g = 0; g < kLoads; ++g) {
                const int r = g * kRowsPer + lane / kPieces;
                const int at = ((lane % kPieces) ^ (W_BITS == 8 ? (r >> 1) & 7 : (r >> 2) & 3)) << 4;
                const int off = k0 + at < K / kWDiv ? __mul24(r, K / kWDiv) + at + k0 : kPastEnd;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_w, (lds_ptr)(mine + t * kWLine + g * 1024), 16, off, 0, 0, 0);
            }
        }
    };
    // a channel of a token per thread on the way out
    const int c = ch0 + min(lane, rows_w - 1);
    const float ws = a.t.w_scale[c];
    const _Float16 bias = a.t.bias ? a.t.bias[c] : (_Float16)0.0f;
    if (tok0 + wave < a.t.M) {   // (uniform)
        typedef VectorsAsked<PRODUCER, decltype(weights)> Vectors;
        const int sample = PRODUCER == kResidual ? (int)((unsigned)(tok0 + wave) / (unsigned)a.f.tokens_per_sample) : 0;
        const Vectors vectors{weights, {a.f.chan_mul != nullptr, PRODUCER == kResidual && a.f.mod_a != nullptr}, lane, sample, {}};
        produce_and_quantize<PRODUCER, kSmallNch, kSmallLanes, false>(a.f, tok0 + wave, lane, col == 0, vectors,
                                                                      RowsInLds{lds_x, x_scale, wave});
    } else {
        weights();
    }
    wait_loads_and_barrier();

    v16i acc[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][r] = acc[1][r] = 0;
    // (the block's rows behind the eight tokens repeat them, and are not written)
    const int fr_row = lane & 31, x_row = fr_row & (kSmallTokens - 1);
    const int x_off0 = x_row * kLine + (((lane >> 5) ^ ((x_row >> 1) & 7)) << 4);
    const int w_off0 = (W_BITS == 8) ? fr_row * kLine + (((lane >> 5) ^ ((fr_row >> 1) & 7)) << 4)
                                     : fr_row * (kLine / 2) + (((fr_row >> 2) & 3) << 4) + (lane >> 5) * 8;
#pragma unroll
    for (int t = 0; t < kSmallTurns; ++t) {
        const int line = wave + t * kSmallWaves;
        if (line >= nl) break;   // (uniform)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const v4i x = *(const v4i*)(lds_x + line * (kSmallTokens * kLine) + (x_off0 ^ (ks << 5)));
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                const int8_t* const at = mine + t * kWLine + (w_off0 ^ (ks << (W_BITS == 8 ? 5 : 4))) + cb * 32 * (kLine / kWDiv);
                v4i w;
                if constexpr (W_BITS == 8) w = *(const v4i*)at;
                else w = widen_nibbles(*(const v2i*)at);
                acc[cb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w, x, acc[cb], 0, 0, 0);
            }
        }
    }

    // ---- the sums, through LDS: [8 tokens][64 channels] of every wavefront where its weights were, 16-byte chunks
    // XOR-ed by the token; then a thread adds up one output
    if (wave < nl && fr_row < kSmallTokens) {
        int8_t* const sums = mine + fr_row * (kSmallChannels * 4);
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int j = 0; j < 4; ++j) {   // register 4j + i is channel 8j + 4 (lane/32) + i of the block
                const int chunk = cb * 8 + 2 * j + (lane >> 5);
                *(v4i*)(sums + ((chunk ^ fr_row) << 4)) = v4i{acc[cb][4 * j], acc[cb][4 * j + 1], acc[cb][4 * j + 2], acc[cb][4 * j + 3]};
            }
    }
    wait_lds_and_barrier();
    if (tok0 + wave >= a.t.M || lane >= rows_w) return;
    int v = 0;
#pragma unroll
    for (int g = 0; g < kSmallWaves; ++g) {
        if (g >= nl) break;   // (uniform)
        v += *(const int*)(lds + g * kSlot + wave * (kSmallChannels * 4) + ((((lane >> 2) ^ wave) << 4) | ((lane & 3) << 2)));
    }
    const float xs = x_scale[wave] * ((W_BITS == 4) ? 0.0625f : 1.0f);
    const unsigned b = (unsigned)__builtin_bit_cast(unsigned short, bias);
    const unsigned out = dequant_pair((float)v, xs * ws, 0.0f, 0.0f, b);
    a.t.y[(long)(tok0 + wave) * N + ch0 + lane] = __builtin_bit_cast(_Float16, (unsigned short)out);
}

template <int PRODUCER>
hipError_t launch_small_producer(SmallArgs a, int w_bits, hipStream_t stream) {
    if (!tile_grid(a.t.grid, a.t.M, a.t.N, kSmallTokens, kSmallChannels, 64 * kSmallWaves)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(a.t.grid.tiles_per_xcd * kTileXcds)), block(64 * kSmallWaves);
    return enqueue(w_bits == 8 ? linear_small<PRODUCER, 8> : linear_small<PRODUCER, 4>, grid, block, stream, a);
}

}  // namespace
}  // namespace vq
