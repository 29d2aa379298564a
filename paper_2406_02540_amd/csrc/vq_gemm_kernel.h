// int8 x int8 -> int32 MFMA GEMM with the dequantization epilogue, for gfx950: the kernel
// template.  vq_gemm.hip and vq_gemm_192.hip instantiate it for two workgroup tiles and
// vq_gemm.hip chooses between them.
//
// Computes, for tokens m and output channels n (ViDiT-Q appendix "Hardware
// implementation of quantized linear layers"; Sec. 4.1 for the grouping):
//     acc[m,n] = sum_k xq[m,k] * wq[n,k]
//     y[m,n]   = fp16(float(acc) * x_scale[m] * w_scale[n] + bias[n])
// W4A8 (appendix "Performance under lower bitwidth"): 4-bit weights are staged
// in LDS packed and widened to int8 on their way from LDS into the MFMA operand
// registers; the mainloop is otherwise the same.  (256 x 192 with 4-bit weights: vq_gemm_192w4.hip.)
//
// Shape of the kernel
//   - workgroup tile: 256 tokens x (64 WC) output channels, WT x WC wavefronts, each
//     wavefront (16 XB) tokens x 64 channels = XB x 4 MFMA 16x16x64 blocks.  Two tiles:
//       256 x 256: 2 x 4 wavefronts of 128 x 64 (128 int32 accumulators per lane), two
//                  wavefronts per SIMD;
//       256 x 192: 4 x 3 wavefronts of 64 x 64 (64 accumulators), three per SIMD: for
//                  channel counts that 256 does not divide well (1152 = 6 x 192: no
//                  half-empty column of tiles, and 768 tiles of 3/4 of the work fill 256
//                  CUs in three even rounds where 640 tiles of 256 x 256 need three
//                  rounds of whole tiles for 2.25 rounds of work).
//     The tile is large because the L2 -> CU path, not HBM, is what the operand traffic
//     loads: bytes per multiply-add fall with the tile edge.
//   - What bounds the large launches back to back is power: a cycle taken out of them comes back as a lower clock.  Between the
//     quantizers of a step it is waiting: 2.2 to 2.5 GHz, the matrix cores 38 to 57 % busy, 28 to 38 % of the wavefronts' cycles
//     waiting for something and 38 to 42 % for their turn to issue.  A loop of nothing but products over quantized-Gaussian
//     operands, two waves to a SIMD, runs at 2.19 GHz with blocks of 16x16x64 and at 1.82 with 32x32x32 (half of the sums move
//     per multiply-add); with every operand read from LDS 1.98 and 1.69, with a stage's loads beside that 1.78.  us in 32x32x32
//     blocks, double buffered / as it is: 32768 x 1152 -> 4608 154 to 161 / 144 to 148, -> 3456 123 / 113, -> 1152 45.3 / 41 to 42,
//     32768 x 4608 -> 1152 164 to 169 / 147 to 150, 8192 x 1152 -> 4608 45.0 / 41.5, 8192 x 4608 -> 1152 43.7 / 40.0, with 4-bit
//     weights 32768 x 1152 -> 4608 154 / 145; fp16 operands 32768 x 4608 -> 1152 322 / 293.  Where power is no bound the shorter
//     products are the slower ones: one or two stages of K 1 to 3 % longer in 256 x 256, fp16 operands of few tokens 3 to 5 %.
//   - K is walked in stages of 128 bytes.  A stage takes one full 128-byte cache line per row, so every L2 request is a
//     whole line (with 64-byte stages the same bytes cost twice the requests and the
//     CU's address path saturates).  Activations and weights go global -> LDS directly
//     (buffer_load ... lds, 16 B per lane, no registers in between).  4-bit weights
//     travel packed (half the bytes).
//   - LDS holds two stages of weights and three of activations: those come from memory, a new panel for every tile, and a
//     request that is one stage old when it is needed has not been answered by then.  32768 x 4608 -> 1152 with two of both
//     162 us, 147.5 so; 8192 x 4608 -> 1152 39.9 and 39.8.  Packed weights, whose stages are as long and whose bytes are
//     fewer, gain nothing (32768 x 1152 -> 4608 143 and 147): two of both, as in 256 x 192 with few stages of K.
//   - In 256 x 256 the four older waves (one per SIMD) ask for the weights, which are needed a stage later, and the younger ones,
//     which come to their products last, for the activations, which have two: with every wave asking for its share of both
//     32768 x 1152 -> 4608 took 151 us, 146 so.  In 256 x 192 it is the other way round (32768 x 4608 -> 1152 148 and 152).
//   - The direct loads are issued from inline assembly and waited for with an
//     explicit s_waitcnt: the compiler would otherwise wait for all of them
//     before every LDS read and undo the prefetch.  They are paced, one load behind the products of a block of tokens: the
//     CU's load path takes 64 bytes per cycle, and a wave that queues there issues no MFMA (all at once ahead of the
//     products a stage of 256 x 256 takes 2600 cycles, 2180 so, of 2048 of products).
//   - LDS tiles are [row][128 B] with the eight 16-byte chunks of a row XOR-ed
//     by (row/2)%8, which makes the 16-lane groups of a ds_read_b128 hit 16
//     different bank groups.
//   - The tokens are the MFMA row operand and the weights the column operand, so a lane owns one
//     column of each of its four blocks and, by permuting which weight row sits in which column, four
//     neighbouring output channels, for 4 XB tokens.  The epilogue narrows them to two dwords in
//     registers and stores them: a store of a wave is four token rows x 128 bytes, whole lines,
//     bypassing the caches' retention (nontemporal: the operands keep the L2).  Nothing is turned
//     through LDS: a lane holds its channels' scales, and a token's scale comes from another lane of its row of sixteen.
//     What bounds the way out is vector instructions, about 15 cycles of a SIMD for an output of
//     64 lanes (conversion 4.4, product of the scales 2.4, mixed multiply-add 8.5), and the stores: without them
//     32768 x 1152 -> 4608 takes 120 us.  (A wave's own vector instructions do not run under its MFMAs; those of another
//     wave of the SIMD do, at 6.4 cycles each instead of 4.5, and the MFMAs take no longer for it.)
//   - The kernel is persistent: one workgroup per CU walks a list of tiles.  What is asked for runs ahead of what is
//     multiplied from tile to tile; what a tile's first stage, which is half as long, should ask for is asked for in
//     the first pieces of the epilogue in front; the waves go from the epilogue into the next tile without meeting at a barrier.
//   - Workgroup ids are dealt round-robin to the 8 XCDs by the hardware; each
//     XCD gets a contiguous run of tiles, ordered in bands of 8 token tiles,
//     and the workgroups of an XCD take them in turn, so that its L2 sees each
//     operand panel once.
//
// Integer accumulation is exact and order independent, so the result is the
// same whatever the tiling; the 4-bit path multiplies by 16 * w (nibble left in
// the high half of the byte) and divides the sum by 16 exactly afterwards.
//
// The epilogue computes fp16_rne(float(acc) * fp32(x_scale * w_scale) + bias): the product of
// the two scales is rounded to fp32, the multiply-add is exact and rounded once, to fp16
// (two vector instructions per output instead of four).  An output can differ from the
// value of three separately rounded fp32 operations in the last fp16 place.
//
// W_BITS == 16 instantiates the same kernel for fp16 operands and fp32 sums
// (v_mfma_f32_16x16x32_f16, the same 16 bytes of K per lane and operand): the FP16 layer
// the paper's hardware evaluation compares against (Sec. 5.3), y = fp16(sum + bias).
#pragma once
#include <type_traits>

#include "vq_gemm_common.h"
#include "vq_internal.h"

namespace vq {

namespace {

// WT x WC wavefronts of (16 XB) tokens x 64 channels; XRING stages of activations in LDS.
template <int WT_, int WC_, int XB_, bool ROLES, int XRING = 3>
struct TileShape {
    static constexpr int WT = WT_, WC = WC_, XB = XB_;
    static constexpr bool kFourBits = XB == 8;        // packed weights too (with 64 tokens a wave: vq_gemm_192w4.hip)
    static constexpr int kWaves = WT * WC;
    static constexpr int kThreads = 64 * kWaves;
    static constexpr int kWavesPerSimd = kWaves / 4;
    static constexpr int kTileT = WT * XB * 16;       // tokens per workgroup
    static constexpr int kTileC = WC * 64;            // output channels per workgroup
    static constexpr int kXStage = kTileT * kTileK;   // 32 KiB
    static constexpr int w_stage(int w_bits) { return kTileC * kTileK / (w_bits == 4 ? 2 : 1); }
    // Two stages of weights in LDS; of activations XRING, with 4-bit weights two.
    static constexpr int kWRing = 2;
    static constexpr int x_ring(int w_bits) { return w_bits == 4 ? 2 : XRING; }
    // Global -> LDS loads of 1 KiB (8 rows of int8, 16 rows of nibbles), dealt round to the waves; or (roles) the first four
    // waves, one per SIMD, load the weights and the others the activations.  (Where the X tile's 32 do not divide evenly, the
    // last turn is some waves' only.)
    static constexpr bool roles(int w_bits) { return ROLES && w_bits != 4; }
    static constexpr int x_loaders(int w_bits) { return roles(w_bits) ? kWaves - 4 : kWaves; }
    static constexpr int w_loaders(int w_bits) { return roles(w_bits) ? 4 : kWaves; }
    static constexpr int x_loads(int w_bits) { return (kTileT / 8 + x_loaders(w_bits) - 1) / x_loaders(w_bits); }
    static constexpr int w_loads(int w_bits) { return kTileC / (w_bits == 4 ? 16 : 8) / w_loaders(w_bits); }
    static constexpr int x_last_turn(int w_bits) { return kTileT / 8 - (x_loads(w_bits) - 1) * x_loaders(w_bits); }   // waves of it
    static constexpr int unread(int w_bits) { return x_last_turn(w_bits) < x_loaders(w_bits) ? 1024 : 0; }   // where the others' goes, a line for all rows
    static constexpr int lds_bytes(int w_bits) { return x_ring(w_bits) * kXStage + kWRing * w_stage(w_bits) + unread(w_bits); }
    // The epilogue is 4 XB stores; the loads that it carries go in front of all but the last eight.
    static constexpr int kStores = 4 * XB;
    static constexpr int load_slot(int load, int loads) { return load * (kStores - 8) / loads; }   // the store that it goes ahead of
    static constexpr bool fits(int w_bits) {   // (and a wave's groups have its parity)
        return lds_bytes(w_bits) <= 160 * 1024 && w_loads(w_bits) * w_loaders(w_bits) * (w_bits == 4 ? 16 : 8) == kTileC &&
               x_loaders(w_bits) % 2 == 0 && (!roles(w_bits) || (x_loads(w_bits) == w_loads(w_bits) && !unread(w_bits)));
    }
    static_assert(kTileT == 256 && fits(8) && fits(16) && (!kFourBits || fits(4)), "loads divide evenly, LDS of one CU");
    static_assert(kWaves % 4 == 0 && kWaves >= 8 && XB % 4 == 0, "tile shape");
};

// Where a tile sits in the output (wave-uniform).
struct TilePos {
    long tok0, ch0;
    int rows_x, rows_w;  // rows of the tile that exist (the rest is clamped on load, masked on store)
};
// Which tile: band and place in it (wave-uniform).
struct TileIndex { int band, in_band; };
// What a wave asks for next of an operand: a stage of a tile and its place in the ring, the operand's rows of the tile, and
// per-lane offsets.
template <int LOADS>
struct Cursor {
    TileIndex at;
    int idx, k0;     // tile; byte of the rows
    unsigned to;     // LDS
    v4i rsrc;
    int voff[LOADS];
    int k_end;       // (used with a K tail only: see load_stage_to_lds_16)
    bool full;       // the tile had all its rows: its per-lane offsets hold for any such tile
};

// One 16 x 16 block: int8 operands (64 values of K over four lanes) into int32 sums, or, for the fp16 comparison
// layer, fp16 operands (32 values of K) into fp32 sums.  Both take 16 bytes of each operand per lane and as long to issue.
template <int W_BITS>
struct AccOf { typedef v4i type; };
template <>
struct AccOf<16> { typedef v4f type; };
__device__ __forceinline__ v4i mfma_block(v4i x, v4i w, v4i c) {
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(x, w, c, 0, 0, 0);
}
__device__ __forceinline__ v4f mfma_block(v4i x, v4i w, v4f c) {
    // (a cast between vector types of one size reinterprets the bits)
    return __builtin_amdgcn_mfma_f32_16x16x32_f16((half8)x, (half8)w, c, 0, 0, 0);
}
// LDS row r of the weight tile holds which output channel of the tile.  Rows are kept in MFMA order: r = slab*64 + b*16 + c,
// with c the column of block b and the lane (of each quarter) that holds its sums.  Sending channel slab*64 + 4c + b
// there gives a lane four neighbouring channels.
__device__ __forceinline__ int w_row_to_channel16(int r) { return (r & ~63) + 4 * (r & 15) + ((r >> 4) & 3); }

// Lane `from` of every row of sixteen lanes, for the whole row.
__device__ __forceinline__ float spread_in_row(float v, int from) {
    const int i = __builtin_bit_cast(int, v);
    int o = i;
    switch (from) {   // (a constant wherever this is called; the instruction holds it)
#define VQ_LANE(n) case n: o = __builtin_amdgcn_mov_dpp(i, 0x150 + n, 0xf, 0xf, false); break
        VQ_LANE(0); VQ_LANE(1); VQ_LANE(2); VQ_LANE(3); VQ_LANE(4); VQ_LANE(5); VQ_LANE(6); VQ_LANE(7);
        VQ_LANE(8); VQ_LANE(9); VQ_LANE(10); VQ_LANE(11); VQ_LANE(12); VQ_LANE(13); VQ_LANE(14); VQ_LANE(15);
#undef VQ_LANE
    }
    return __builtin_bit_cast(float, o);
}

// Ends a stage like wait_loads_before_and_barrier, with as many operations in flight as the mode (uniform) allows.  One statement:
// as branches of the program the choice was a dozen scalar instructions and four taken branches between a wave's last product
// and the barrier.
enum StageEnd { kNear = 0, kFarther = 1, kFartherSecond = 2, kFartherFirst = 3, kNearFirst = 4 };
template <int NEAR, int FAR, int FAR_SECOND, int FAR_FIRST, int NEAR_FIRST>
__device__ __forceinline__ void wait_by_mode_and_barrier(int mode) {
    static_assert(NEAR <= FAR && FAR < 64 && FAR_SECOND < 64 && FAR_FIRST < 64 && NEAR_FIRST < 64, "vmcnt is a 6-bit counter");
    asm volatile(
        "s_cmp_gt_u32 %0, 1\n\t"
        "s_cbranch_scc1 .Lvq_rare%=\n\t"
        "s_cmp_lg_u32 %0, 0\n\t"
        "s_cbranch_scc1 .Lvq_far%=\n\t"
        "s_waitcnt vmcnt(%1)\n"
        ".Lvq_far%=:\n\t"
        "s_waitcnt vmcnt(%2)\n"
        ".Lvq_end%=:\n\t"
        "s_waitcnt lgkmcnt(0)\n\t"
        "s_barrier\n\t"
        "s_branch .Lvq_out%=\n"
        ".Lvq_rare%=:\n\t"
        "s_cmp_lg_u32 %0, 2\n\t"
        "s_cbranch_scc1 .Lvq_first%=\n\t"
        "s_waitcnt vmcnt(%3)\n\t"
        "s_branch .Lvq_end%=\n"
        ".Lvq_first%=:\n\t"
        "s_cmp_lg_u32 %0, 3\n\t"
        "s_cbranch_scc1 .Lvq_near%=\n\t"
        "s_waitcnt vmcnt(%4)\n\t"
        "s_branch .Lvq_end%=\n"
        ".Lvq_near%=:\n\t"
        "s_waitcnt vmcnt(%5)\n\t"
        "s_branch .Lvq_end%=\n"
        ".Lvq_out%=:"
        :
        : "s"(mode), "n"(NEAR), "n"(FAR), "n"(FAR_SECOND), "n"(FAR_FIRST), "n"(NEAR_FIRST)
        : "memory", "scc");
}

// K_TAIL:  K is a multiple of 16 but not of 128 (the last stage is partly past K).
// OUT:     how rows of Y are written (vq_gemm_common.h).
template <class S, int W_BITS, bool K_TAIL, Out OUT>
__global__ __launch_bounds__(S::kThreads, S::kWavesPerSimd) void gemm_i8_dequant(const GemmArgs a) {
    constexpr bool GENERIC = OUT == kAnyRow;
    constexpr int XB = S::XB, WB = 4;   // blocks of 16 tokens and of 16 channels
    constexpr int kXStage = S::kXStage, kWStage = S::w_stage(W_BITS), kXRing = S::x_ring(W_BITS), kXArea = kXRing * kXStage, kWArea = S::kWRing * kWStage;
    __shared__ __attribute__((aligned(1024))) int8_t lds[S::lds_bytes(W_BITS)];
    // layout: the ring of X stages, then the ring of W stages; a stage is [rows][128 B] or, for 4-bit weights, [rows][64 B].
    const unsigned lds_addr = (unsigned)(uintptr_t)(lds_ptr)lds;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Waves w, w+4 (and w+8) share a SIMD: they get the same token part and different
    // channel slabs, so a tile that is only partly full of channels still
    // leaves a working wave on every SIMD.
    const int wave_t = wave % S::WT;   // which 16 XB tokens
    const int wave_c = wave / S::WT;   // which 64 channels
    // (W_BITS == 16: fp16 operands, the comparison layer; rows are 2 K bytes and everything up
    // to the MFMA itself treats them like int8 rows of that many bytes)
    const int K = (W_BITS == 16) ? 2 * a.K : a.K;      // bytes per activation row
    constexpr int kWDiv = (W_BITS == 4) ? 2 : 1;        // activation bytes per weight byte
    const int nk = (K + kTileK - 1) / kTileK;

    // What this wave loads per stage.  Weights are asked for one stage before they are multiplied, activations kXRing - 1.
    constexpr bool kRoles = S::roles(W_BITS), kXFar = kXRing == 3;
    constexpr int kXLoads = S::x_loads(W_BITS), kWLoads = S::w_loads(W_BITS), kLoads = kRoles ? kXLoads : kXLoads + kWLoads;
    const bool loads_w = kRoles && wave < 4;
    const bool far = kXFar && !loads_w;    // asks two stages ahead
    // A quantity of the weights' or the activations' cursor or, of roles, of this wave's.  (By arithmetic: the compiler makes
    // selects between constants in vector registers, and these go where only scalar ones can.)
    enum Operand { kX, kW, kMine };
    const int w_mask = (wave - 4) >> 31;
    auto of = [&](auto op, auto w, auto x) __attribute__((always_inline)) {
        if constexpr (decltype(op)::value == kW) return w;
        else if constexpr (decltype(op)::value == kX) return x;
        else return x + ((w - x) & (decltype(x))w_mask);
    };

    // ---- global -> LDS mapping ---------------------------------------------
    // One direct load fills 1 KiB; lane l writes bytes [16 l, 16 l + 16).
    // int8 tiles: 8 rows x 128 B per load, lane l = row l/8, physical chunk l%8,
    // which under the swizzle holds logical chunk (l%8) ^ ((row/2)%8).  A wave's row
    // groups g all have the parity of the wave's number, so row/2 mod 8 is
    // (4 (g%2) + l/16) % 8 for all of them.
    // Packed 4-bit tile [rows][64 B]: 16 rows x 64 B per load, lane l = row l/4,
    // physical chunk l%4 holding logical chunk (l%4) ^ ((row/4)%4) = (l%4) ^ (l/16).
    // The tiles of an XCD are numbered band by band (kBand token tiles), column by column
    // within a band, token tile by token tile within a column.  A workgroup's tiles lie
    // a.slots apart: the first one is located by division, the later ones by stepping.
    const int band_tiles = kBand * a.tiles_c;
    auto step_tile = [&](TileIndex& t) {
        t.in_band += a.slots;
        while (t.in_band >= band_tiles) {
            t.in_band -= band_tiles;
            ++t.band;
        }
    };
    auto decode_tile = [&](const TileIndex& at, TilePos& t) {
        const int band_first = at.band * kBand;
        const int band_rows = min(a.tiles_t - band_first, kBand);
        int row, col;
        if (band_rows == kBand) {
            row = at.in_band % kBand;
            col = at.in_band / kBand;
        } else {  // the last band of a matrix whose token tiles are not a multiple of kBand
            row = at.in_band % band_rows;
            col = at.in_band / band_rows;
        }
        t.tok0 = (long)(band_first + row) * S::kTileT;
        t.ch0 = (long)col * S::kTileC;
        t.rows_x = (int)min((long)S::kTileT, a.M - t.tok0);
        t.rows_w = (int)min((long)S::kTileC, a.N - t.ch0);
    };
    auto tile_exists = [&](int idx) {
        return idx < a.tiles_per_xcd && (int)(blockIdx.x % kXcds) * a.tiles_per_xcd + idx < a.tiles;
    };

    // The per-lane offsets are relative to the tile and clamp rows past the tile: between
    // two full tiles they do not change.  (Rows < 256 and row lengths < 2^24: 24-bit products.)
    // (With a K tail the buffers end with the tile's last row: see load_stage_to_lds_16.)
    auto decode_loads = [&](auto op, const TilePos& t, auto& c) __attribute__((always_inline)) {
        constexpr int LOADS = sizeof(c.voff) / sizeof(int);
        constexpr bool kNibbles = W_BITS == 4 && decltype(op)::value == kW;
        const int rows = of(op, t.rows_w, t.rows_x), row_bytes = of(op, K / kWDiv, K);
        const long first = of(op, t.ch0, t.tok0);
        c.rsrc = make_rsrc((const int8_t*)of(op, (long)a.w, (long)a.xq) + first * row_bytes,
                           K_TAIL ? (unsigned)(rows * row_bytes) : clamp_u32((of(op, a.N, a.M) - first) * (long)row_bytes));
        const bool full = rows == of(op, S::kTileC, S::kTileT);
        if (full && c.full) return;
        c.full = full;
        const int l = opaque(lane), loader = kRoles ? wave - of(op, 0, 4) : wave;
        const int chunk = kNibbles ? ((l & 3) ^ (l >> 4)) << 4 : ((l & 7) ^ ((4 * (wave & 1) + (l >> 4)) & 7)) << 4;
        c.k_end = row_bytes - chunk;
#pragma unroll
        for (int j = 0; j < LOADS; ++j) {
            const int g = loader + of(op, S::w_loaders(W_BITS), S::x_loaders(W_BITS)) * j;
            int r = kNibbles ? g * 16 + (l >> 2) : g * 8 + (l >> 3);
            if (decltype(op)::value == kW || (decltype(op)::value == kMine && loads_w)) r = w_row_to_channel16(r);
            c.voff[j] = __mul24(min(r, rows - 1), row_bytes) + chunk;
        }
    };

    // ---- LDS -> MFMA operand mapping -----------------------------------------
    // Operand rows of a 16x16x64 block: lane l supplies row l%16, 16 bytes of K chosen by l/16; a stage holds two such
    // K steps (chunks 4ks .. 4ks + 3).  The chunk index of K step ks is (4 ks + l/16) ^ swizzle = ((l/16) ^ swizzle) ^ 4 ks,
    // so the byte offset of step ks is that of step 0 with 64 ks XOR-ed in.
    // 4-bit weights: the two K steps share one read of 16 bytes of nibbles, chunk c = nibble_chunk(l/16) of the row, whose first half the
    // lane widens for the one and second half for the other.  The activations follow: chunk 2 c for the first, the one behind
    // it for the second.  (Which 64 bytes of K a step takes does not change the sums.)
    const int fr_row = lane & 15;
    const int x_off0 = (wave_t * 16 * XB + fr_row) * kTileK + (((W_BITS != 4 ? lane >> 4 : nibble_chunk(lane >> 4) << 1) ^ ((fr_row >> 1) & 7)) << 4);
    const int w_off0 = (W_BITS != 4)
                           ? (wave_c * 64 + fr_row) * kTileK + (((lane >> 4) ^ ((fr_row >> 1) & 7)) << 4)
                           : (wave_c * 64 + fr_row) * (kTileK / 2) + ((nibble_chunk(lane >> 4) ^ ((fr_row >> 2) & 3)) << 4);
    auto x_off = [&](int ks) { return x_off0 ^ (W_BITS != 4 ? ks << 6 : ks << 4); };

    // ---- the tiles of this workgroup -------------------------------------------
    int idx = blockIdx.x / kXcds;
    if (!tile_exists(idx)) return;  // uniform per workgroup
    TileIndex at;   // of the tile being multiplied
    TilePos cur;
    {
        const int logical = (blockIdx.x % kXcds) * a.tiles_per_xcd + idx;
        at.band = logical / band_tiles;
        at.in_band = logical - at.band * band_tiles;
    }
    decode_tile(at, cur);
    // Behind the last tile's last stage a cursor's buffer is empty: loads that move nothing, into stages that are not read.
    auto cursor_end = [&](auto op) { return lds_addr + of(op, kXArea + kWArea, kXArea) + (kRoles ? wave - of(op, 0, 4) : wave) * 1024; };
    auto start = [&](auto op, auto& c) {
        c.at = at;
        c.idx = idx;
        c.k0 = 0;
        c.to = cursor_end(op) - of(op, kWArea, kXArea);
        c.full = false;
        decode_loads(op, cur, c);
    };
    const unsigned unread = lds_addr + kXArea + kWArea, last_mask = (unsigned)((wave - S::x_last_turn(W_BITS)) >> 31);
    auto load_one = [&](auto op, const auto& c, int j) __attribute__((always_inline)) {
        constexpr int LOADS = sizeof(c.voff) / sizeof(int);
        unsigned to = c.to + j * of(op, S::w_loaders(W_BITS), S::x_loaders(W_BITS)) * 1024;
        if (decltype(op)::value == kX && S::unread(W_BITS) && j == LOADS - 1) to = unread + ((to - unread) & last_mask);
        load_stage_to_lds_16<K_TAIL>(c.rsrc, to, c.voff[j], c.k0, c.k_end);
    };
    // One stage on.  (Two cursors that are at the same stage, those of rings of two, go as one: `with` is the weights'.)
    auto next_stage = [&](auto op, auto& c, auto&... with) __attribute__((always_inline)) {
        const int stage_bytes = of(op, kTileK / kWDiv, kTileK);
        auto place = [&](auto op, auto& c) __attribute__((always_inline)) {
            c.to += of(op, kWStage, kXStage);
            if (c.to == cursor_end(op)) c.to -= of(op, kWArea, kXArea);
        };
        place(op, c);
        (place(std::integral_constant<int, kW>{}, with), ...);
        c.k0 += stage_bytes;
        if (c.k0 == nk * stage_bytes) {
            c.k0 = 0;
            c.idx += a.slots;
            if (tile_exists(c.idx)) {
                TilePos t;
                step_tile(c.at);
                decode_tile(c.at, t);
                decode_loads(op, t, c);
                (decode_loads(std::integral_constant<int, kW>{}, t, with), ...);
            } else {
                c.rsrc[2] = 0;
                ((with.rsrc[2] = 0), ...);
            }
        }
        ((with.k0 = c.k0 / kWDiv), ...);
        asm volatile("" : "+s"(c.k0), "+s"(c.to));
    };
    // (roles: cx is this wave's, cw is not used)
    typedef std::integral_constant<int, kRoles ? kMine : kX> OpX;
    typedef std::integral_constant<int, kW> OpW;
    Cursor<kXLoads> cx;
    Cursor<kWLoads> cw;
    start(OpX{}, cx);
    if constexpr (!kRoles) start(OpW{}, cw);
    // Load l of the ones that a stage of a tile asks for: weights first.
    auto load = [&](int l) __attribute__((always_inline)) {
        if (!kRoles && l < kWLoads) load_one(OpW{}, cw, l);
        else load_one(OpX{}, cx, kRoles ? l : l - kWLoads);
    };
    auto load_x = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int l = kLoads - kXLoads; l < kLoads; ++l) load(l);
    };
    auto load_w = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int l = 0; l < kLoads - kXLoads; ++l) load(l);
    };
    auto next_loads = [&]() __attribute__((always_inline)) {
        if constexpr (kRoles) {
            next_stage(OpX{}, cx);
        } else if constexpr (kXFar) {
            next_stage(OpW{}, cw);
            next_stage(OpX{}, cx);
        } else {
            next_stage(OpX{}, cx, cw);
        }
    };
    load_w();
    load_x();
    next_loads();
    // Every line of the weight matrix is asked for once, here, by the whole grid (one dword per
    // 128-byte line and lane, 8 KiB per wave and round): the weights are a few MB that every XCD
    // walks through completely, and a column's panel is otherwise first asked for by the eight
    // CUs that need it at that moment, which then wait out the memory latency at every stage of
    // their tile.  Fetched up front the lines are in the memory-side cache when their column's
    // turn comes.  (Range-checked loads: lanes past the end of the matrix fetch nothing.  They go where the ring's last stage of
    // activations will, which is asked for when they have arrived.)
    {
        const long w_bytes = (long)a.N * (K / kWDiv);
        const v4i rsrc_all = make_rsrc(a.w, clamp_u32(w_bytes));
        const unsigned per_round = gridDim.x * (unsigned)S::kWaves * 8192u;
        const unsigned off = (blockIdx.x * (unsigned)S::kWaves + (unsigned)wave) * 8192u + (unsigned)lane * 128u;
#pragma unroll
        for (int i = 0; i < kTouchRounds; ++i)
            if ((long)i * per_round < w_bytes)  // (uniform; all rounds are in flight together)
                load_to_lds_4(rsrc_all, lds_addr + (kXRing - 1) * kXStage + wave * 256, (int)(off + i * per_round));
    }
    // The first tile's first stage (later ones arrive behind an epilogue), and what it should ask for (later: in the epilogue
    // in front): the next stage of weights, of activations two with a ring of three.
    if constexpr (kRoles) {
        if (far) {
            load_x();
            next_loads();
            wait_loads_before_and_barrier<kLoads>();
        } else {
            wait_loads_before_and_barrier<0>();
        }
    } else if constexpr (kXFar) {
        load_x();
        next_stage(OpX{}, cx);
        wait_loads_before_and_barrier<kXLoads>();
    } else {
        wait_loads_before_and_barrier<0>();
    }
    load_w();
    load_x();
    next_loads();
    unsigned x_stage = 0, w_stage = 0;   // the stage about to be multiplied: its place in the rings
    bool stores_in_flight = false;       // this wave wrote outputs in the previous epilogue

    // Invariant at the top of a stage: its operands have landed for every wave, nobody reads the stage before any more, and
    // this wave has asked for one or two stages behind it.
    while (true) {
        const int next_idx = idx + a.slots;
        const bool has_next = tile_exists(next_idx);

        // a wave whose 64 channels (or tokens) lie wholly past the matrix has nothing to multiply
        const bool wave_live = (wave_c * 64 < cur.rows_w) && (wave_t * 16 * XB < cur.rows_x);

        typedef typename AccOf<W_BITS>::type acc_t;
        acc_t acc[XB][WB];
        v4i xf[2][XB], wf[2][WB];  // operand registers; [1] carries K step 1 across stages
        v4i nibbles[WB];           // (4-bit weights: of both K steps)
        const acc_t kZero4 = {0, 0, 0, 0};

        // One stage = two K steps of 4 XB MFMAs per wave.  The schedule is skewed by one K step:
        // the MFMAs of a stage's second K step are issued at the start of the next stage, behind
        // the barrier, where they cover the latency of that stage's first LDS reads (otherwise
        // every wave of the CU would sit idle there).
        //
        // The LDS reads of K step ks+1 are issued among the MFMAs of step ks, which cover their latency.
        // A K step = XB pieces of four MFMAs, one block of tokens each.  A piece carries at most one global load
        // (so that a wave never sits in the load queue while the matrix pipe waits for it)
        // and its share of the LDS reads of the step after; sched_barrier(0) keeps the pieces apart.
        constexpr int kReads = XB + WB;
        constexpr int kReadsPerPiece = (kReads + XB - 2) / (XB - 1);   // spread over all pieces but the last
        // in the order w0 x0 w1 x1 ..
        auto read_one = [&](int ks, int r, v4i(&xo)[XB], v4i(&wo)[WB]) __attribute__((always_inline)) {
            const int8_t* const xs = lds + x_stage;
            const int8_t* const ws = lds + kXArea + w_stage;
            const bool is_w = r < 2 * WB && r % 2 == 0;
            const int b = r < 2 * WB ? r / 2 : r - WB;
            if (!is_w)
                xo[b] = *(const v4i*)(xs + x_off(ks) + b * 16 * kTileK);
            else if (W_BITS != 4)
                wo[b] = *(const v4i*)(ws + (w_off0 ^ (ks << 6)) + b * 16 * kTileK);
            else if (ks == 0)
                nibbles[b] = *(const v4i*)(ws + w_off0 + b * 16 * (kTileK / 2));
        };
        auto widen = [&](int ks, int b, v4i(&wo)[WB]) __attribute__((always_inline)) {
            wo[b] = widen_nibbles(ks ? v2i{nibbles[b][2], nibbles[b][3]} : v2i{nibbles[b][0], nibbles[b][1]});
            asm volatile("" : "+v"(wo[b]));   // (here, not where it is used)
        };
        // A K step.  read_ks < 0: nothing left to read (the tile's last K step).  It carries this wave's loads from .. to - 1,
        // behind a piece's products each.  (Known where it is compiled: a branch in front of each load costs the wave more than
        // the product it should run beside.)
        auto k_step = [&](const v4i(&xi)[XB], const v4i(&wi)[WB], auto zero_tag, int read_ks, v4i(&xo)[XB], v4i(&wo)[WB],
                          int from, int to) __attribute__((always_inline)) {
#pragma unroll
            for (int p = 0; p < XB; ++p) {
#pragma unroll
                for (int m = 0; m < WB; ++m) {
                    const int b = p & 1 ? WB - 1 - m : m;   // (there and back: the weight operand of two MFMAs in a row is the same)
                    if constexpr (decltype(zero_tag)::value)
                        acc[p][b] = mfma_block(xi[p], wi[b], kZero4);
                    else
                        acc[p][b] = mfma_block(xi[p], wi[b], acc[p][b]);
                }
                if (from + p < to) load(from + p);
                if (read_ks >= 0) {
#pragma unroll
                    for (int r = p * kReadsPerPiece; r < (p + 1) * kReadsPerPiece && r < kReads; ++r) read_one(read_ks, r, xo, wo);
                    if (W_BITS != 4 && p * kReadsPerPiece < kReads) {
#pragma unroll
                        for (int r = 0; r < kReadsPerPiece; ++r) {
                            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
                            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
                        }
                    }
                    if (W_BITS == 4) {
                        // (The first step's in its last pieces, when the nibbles have arrived behind the products before; the second's
                        // in all of them.  Left to where they are used, 32768 x 1152 -> 4608 takes 308000 cycles, 292000 so.)
                        const int from = read_ks ? p * WB / XB : p < XB / 2 ? 0 : (p - XB / 2) * WB / (XB / 2);
                        const int to = read_ks ? (p + 1) * WB / XB : p < XB / 2 ? 0 : (p + 1 - XB / 2) * WB / (XB / 2);
#pragma unroll
                        for (int b = 0; b < WB; ++b)
                            if (b >= from && b < to) widen(read_ks, b, wo);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        // Ends a stage: the next one has landed for every wave and every wave is done reading this one.  Vector memory
        // operations complete in the order they were issued: how many of this wave's are behind the loads that have to have landed?
        // Steadily, what is asked for two stages ahead.  Behind an epilogue whose stores are in flight also those behind the
        // last load that is needed: of a ring of two all loads, of three those of weights; a wave that asks for nothing but
        // activations, two stages ahead, waits for that epilogue's at the end of the tile's second stage.
        constexpr int kAhead = kRoles ? kLoads : kXFar ? kXLoads : 0, kNearNeeds = !kRoles && kXFar ? kWLoads - 1 : kLoads - 1;
        constexpr int kStoresBehind = S::kStores - S::load_slot(kNearNeeds, kLoads), kStoresBehindAll = S::kStores - S::load_slot(kLoads - 1, kLoads);
        const int far_mask = kRoles ? ~w_mask : kXFar ? -1 : 0;
        auto next_place = [&]() __attribute__((always_inline)) {
            x_stage = x_stage == (kXRing - 1) * kXStage ? 0 : x_stage + kXStage;
            w_stage = w_stage == kWStage ? 0 : w_stage + kWStage;
        };
        auto end_stage = [&](int& mode) __attribute__((always_inline)) {
            if constexpr (kRoles) {   // (ahead of the barrier)
                next_place();
                asm volatile("" : "+s"(x_stage), "+s"(w_stage));
            }
            if constexpr (kRoles) wait_by_mode_and_barrier<0, kAhead, kAhead + kStoresBehindAll, kAhead + S::kStores, kStoresBehind>(mode);
            else wait_by_mode_and_barrier<0, kAhead, kAhead, kAhead + kStoresBehind, kStoresBehind>(mode);
            mode = far_mask & max(mode - 1, (int)kFarther);
            asm volatile("" : "+s"(mode));
            if constexpr (!kRoles) next_place();
        };
        int mode = (stores_in_flight ? kNearFirst : kNear) + (far_mask & (stores_in_flight ? kFartherFirst - kNearFirst : kFarther - kNear));
        asm volatile("" : "+s"(mode));
        // Which of a stage's loads its first K step carries (K step 1 of the stage before), the rest its second.
        constexpr int kFirst = !kRoles && kXFar ? kWLoads : kLoads < XB ? kLoads : XB;
        static_assert(kFirst <= XB && kLoads - kFirst <= XB, "a load in a piece");
        if (wave_live) {
            constexpr std::true_type kYes{};
            constexpr std::false_type kNo{};
            // The tile's first stage: nothing deferred to cover its first reads, and its first K step starts the accumulators
            // from a constant zero.  What it should ask for was asked for in the epilogue in front.
#pragma unroll
            for (int r = 0; r < kReads; ++r) read_one(0, r, xf[0], wf[0]);
            if (W_BITS == 4)
#pragma unroll
                for (int b = 0; b < WB; ++b) widen(0, b, wf[0]);
            __builtin_amdgcn_sched_barrier(0);
            k_step(xf[0], wf[0], kYes, 1, xf[1], wf[1], 0, 0);
            auto stage = [&]() __attribute__((always_inline)) {
                k_step(xf[1], wf[1], kNo, 0, xf[0], wf[0], 0, kFirst);        // K step 1 of the previous stage
                k_step(xf[0], wf[0], kNo, 1, xf[1], wf[1], kFirst, kLoads);   // K step 0
                next_loads();
            };
            if constexpr (kRoles) {
#pragma unroll 1
                for (int n = nk - 1; n != 0; --n) {
                    end_stage(mode);
                    stage();
                    asm volatile("" : "+s"(n));
                }
            } else if (nk > 1) {
                end_stage(mode);
#pragma unroll 1
                for (int it = 1;; ++it) {
                    stage();
                    if (it == nk - 1) break;
                    wait_loads_before_and_barrier<kAhead>();
                    next_place();
                }
            }
            // Scales and bias: a channel's four, and a token's in lane 4 (block % 4) + i of its row of sixteen lanes, which the
            // epilogue spreads over the row.  Entries past N or M, and a missing bias, are zero.
            constexpr int kXsRegs = XB / 4;
            const int el = opaque(lane);
            const int g = el >> 4, quad = wave_c * 64 + 4 * (el & 15);   // the lane's first channel within the tile
            const int row0 = wave_t * 16 * XB;                           // the wave's first token within the tile
            v4f ws4 = {0.0f, 0.0f, 0.0f, 0.0f};
            float xs_row[kXsRegs];
            if constexpr (W_BITS != 16) {
                const __amdgpu_buffer_rsrc_t rs_ws = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.w_scale) + cur.ch0, 0, cur.rows_w * 4, kRsrcFlags);
                const __amdgpu_buffer_rsrc_t rs_xs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.x_scale) + cur.tok0, 0, cur.rows_x * 4, kRsrcFlags);
                ws4 = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rs_ws, quad * 4, 0, 0));
#pragma unroll
                for (int r = 0; r < kXsRegs; ++r)
                    xs_row[r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                        rs_xs, (row0 + 64 * r + 16 * ((el & 15) >> 2) + 4 * g + (el & 3)) * 4, 0, 0));
            }
            const __amdgpu_buffer_rsrc_t rs_b = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<_Float16*>(a.bias) + cur.ch0, 0, a.bias ? cur.rows_w * 2 : 0, kRsrcFlags);
            v2i bias4 = __builtin_bit_cast(v2i, __builtin_amdgcn_raw_buffer_load_b64(rs_b, quad * 2, 0, 0));
            if (GENERIC && (cur.rows_w & 1) && cur.rows_w - quad < 4) {
                // (the last of an odd number is half of a dword that reaches behind the buffer)
                const int last = (int)__builtin_amdgcn_raw_buffer_load_b16(rs_b, (cur.rows_w - 1) * 2, 0, 0) & 0xFFFF;
                if (cur.rows_w - quad == 1) bias4[0] = last;
                if (cur.rows_w - quad == 3) bias4[1] = last;
            }
            __builtin_amdgcn_sched_barrier(0);
            constexpr int kScaleLoads = W_BITS == 16 ? 1 : 2 + kXsRegs;
            k_step(xf[1], wf[1], kNo, -1, xf[0], wf[0], 0, 0);   // K step 1 of the last stage
            if constexpr (kRoles) wait_by_mode_and_barrier<kScaleLoads, kAhead + kScaleLoads, 0, 0, 0>(far_mask & kFarther);
            else wait_loads_before_and_barrier<kAhead + kScaleLoads>();
            next_place();

            // ---- epilogue ------------------------------------------------------------
            // Lane (g = lane/16, c = lane%16) holds channels 4c .. 4c + 3 of the wavefront's 64 (accumulator blocks 0 .. 3) for
            // the tokens 4g + i of each of its blocks of 16 (register i).  Its four outputs of a token are two dwords, and a
            // store of both per lane is a whole 128-byte line of four token rows.
            const int left = cur.rows_w - quad;                          // channels from there on that exist
            // (all sums are converted first, which covers the way of the scales)
            typedef v4f sums_t;
            sums_t sum[XB][WB];
#pragma unroll
            for (int xb = 0; xb < XB; ++xb)
#pragma unroll
                for (int b = 0; b < WB; ++b)
#pragma unroll
                    for (int i = 0; i < 4; ++i) sum[xb][b][i] = (float)acc[xb][b][i];
            // Stores are range-checked, relative to the first of sixteen token rows: rows past M fall behind the end of
            // the buffer, lanes whose channels lie past N get an offset behind it (N < 2^21 on this path, so nothing
            // wraps).  Of an even N two of a lane's four channels may exist: they are a dword of their own.
            const unsigned y_place = (unsigned)(__mul24(4 * g, GENERIC ? 0 : a.N) + (int)cur.ch0 + quad) * 2u;
            unsigned y_off[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) y_off[i] = left >= 4 ? y_place + (unsigned)checked_bytes<OUT>(i, a.N) : 0x80000000u;
            const _Float16* y_row = a.y + (cur.tok0 + row0) * a.N;
            int y_bytes = checked_bytes<OUT>(cur.rows_x - row0, a.N);   // from there to the end of the tile's rows
            // (Any row: token rows of the wave below which the lane has channels to write; its place in the four rows of a block.  Of
            // 128 tokens a wave it is one place, which the rows step on from by N, and `quad` has an upper half of its own: three
            // more of them, and a zero that is kept for it, were registers held across the stages, where 4-bit weights leave none.
            // With their operands' places reloaded from scratch in every stage 32768 x 1152 -> 4607 took 230 us, 193 so.)
            const int rows_live = left > 0 ? cur.rows_x - row0 - 4 * g : 0;
            constexpr bool kStepped = GENERIC && XB == 8;
            constexpr int kPlaces = kStepped ? 1 : 4;
            long y_any[kPlaces];
#pragma unroll
            for (int i = 0; i < kPlaces; ++i) y_any[i] = (4 * g + i) * (long)a.N + cur.ch0 + (kStepped ? opaque(quad) : quad);
            auto any_place = [&](int i) __attribute__((always_inline)) { return kStepped ? i * (long)a.N + y_any[0] : y_any[i % kPlaces]; };
            if (GENERIC && a.acc_out) {
                typedef v4i v4i_any4 __attribute__((aligned(4)));
                int32_t* acc_row = a.acc_out + (cur.tok0 + row0) * a.N;
#pragma unroll
                for (int xb = 0; xb < XB; ++xb) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (xb * 16 + i < rows_live) {
                            constexpr int kShift = (W_BITS == 4) ? 4 : 0;
                            const v4i sums = v4i{(int)acc[xb][0][i], (int)acc[xb][1][i], (int)acc[xb][2][i], (int)acc[xb][3][i]} >> kShift;
                            if (left >= 4) {
                                *(v4i_any4*)(acc_row + any_place(i)) = sums;
                            } else {
#pragma unroll
                                for (int e = 0; e < 3; ++e)
                                    if (e < left) acc_row[any_place(i) + e] = sums[e];
                            }
                        }
                    acc_row += 16 * (long)a.N;
                    asm volatile("" : "+s"(acc_row));
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            // (here the compiler waits for them, ahead of the next loads)
            if constexpr (W_BITS != 16) asm volatile("" : "+v"(ws4));
            asm volatile("" : "+v"(bias4));
            if constexpr (W_BITS != 16) {
#pragma unroll
                for (int r = 0; r < kXsRegs; ++r) {
                    xs_row[r] *= W_BITS == 4 ? 0.0625f : 1.0f;   // the 4-bit path accumulates 16 * w: the exact 1/16 rides on the token scale
                    asm volatile("" : "+v"(xs_row[r]));
                }
            }
#pragma unroll
            for (int xb = 0; xb < XB; ++xb) {
                const __amdgpu_buffer_rsrc_t rsrc_y =
                    __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(y_row), 0, max(y_bytes, 0), kRsrcFlags);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    // what the next tile's first stage should ask for, a load at a time
#pragma unroll
                    for (int l = 0; l < kLoads; ++l)
                        if (S::load_slot(l, kLoads) == 4 * xb + i && has_next) load(l);
                    float xs = 0.0f;
                    if constexpr (W_BITS != 16) {
                        xs = spread_in_row(xs_row[xb / 4], 4 * (xb % 4) + i);
                        asm volatile("" : "+v"(xs));   // (one instruction, not part of four)
                    }
                    v2i out;
                    // y = fp16(float(acc) * (x_scale * w_scale) + bias): the product of the two scales rounded to
                    // fp32, the rest exact and rounded once (dequant_pair)
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const float a0 = sum[xb][2 * e][i], a1 = sum[xb][2 * e + 1][i];
                        if constexpr (W_BITS == 16)  // the fp32 sum of the fp16 products, plus the bias
                            out[e] = (int)add_bias_pair(a0, a1, (unsigned)bias4[e]);
                        else
                            out[e] = (int)dequant_pair(a0, xs * ws4[2 * e], a1, xs * ws4[2 * e + 1], (unsigned)bias4[e]);
                    }
                    if (!GENERIC) {
                        __builtin_amdgcn_raw_buffer_store_b64(out, rsrc_y, y_off[i], 0, OUT == kHalfLines ? 2 /* nontemporal */ : 0);
                        if (OUT == kDwords && (cur.rows_w & 2))   // (uniform)
                            __builtin_amdgcn_raw_buffer_store_b32(out[0], rsrc_y, left == 2 ? y_place + (unsigned)checked_bytes<OUT>(i, a.N) : 0x80000000u, 0, 0);
                    } else if (xb * 16 + i < rows_live) {
                        // Rows of Y that start at any even address; a lane's last channels one by one.
                        typedef v2i v2i_any __attribute__((aligned(2)));
                        _Float16* const at = const_cast<_Float16*>(y_row) + any_place(i);
                        if (left >= 4) {
                            *(v2i_any*)at = out;
                        } else {
#pragma unroll
                            for (int e = 0; e < 3; ++e)
                                if (e < left) ((unsigned short*)at)[e] = (unsigned short)((unsigned)out[e / 2] >> (e % 2 * 16));
                        }
                    }
                    if (i % 2 == 1) __builtin_amdgcn_sched_barrier(0);
                }
                y_row += 16 * (long)a.N;
                y_bytes -= checked_bytes<OUT>(16, a.N);
                if (GENERIC) asm volatile("" : "+s"(y_row));   // (nothing is made up ahead of its use)
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            // nothing to multiply in this tile, but this wave's share of the loads is needed
#pragma unroll 1
            for (int it = 0; it < nk; ++it) {
                if (it > 0) {
                    load_w();
                    load_x();
                    next_loads();
                }
                mode = far_mask & kFarther;
                end_stage(mode);
            }
            if (has_next) {
                load_w();
                load_x();
            }
        }
        stores_in_flight = wave_live && !GENERIC;
        if (!has_next) break;
        next_loads();
        step_tile(at);
        decode_tile(at, cur);
        idx = next_idx;
    }
    // (nothing may be on its way to LDS when the workgroup ends)
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
}

// Enqueues the kernel for tile shape S; `a` holds the operands and sizes.
template <class S>
hipError_t launch_gemm_shape(GemmArgs a, int w_bits, int num_cus, hipStream_t stream) {
    dim3 grid;
    if (!persistent_grid(a, grid, S::kTileT, S::kTileC, num_cus)) return hipErrorInvalidValue;
    const dim3 block(S::kThreads);
    const bool tail = ((w_bits == 16 ? 2 * a.K : a.K) % kTileK) != 0;  // (in bytes of an activation row)
    const Out out = rows_out(a.N, a.y, a.acc_out);
#define VQ_LAUNCH_GEMM(BITS, TAIL, OUT) \
    return enqueue(gemm_i8_dequant<S, BITS, TAIL, OUT>, grid, block, stream, a)
#define VQ_LAUNCH_OUT(BITS, TAIL)                                      \
    do {                                                               \
        if (out == kHalfLines) VQ_LAUNCH_GEMM(BITS, TAIL, kHalfLines); \
        else if (out == kDwords) VQ_LAUNCH_GEMM(BITS, TAIL, kDwords);  \
        else VQ_LAUNCH_GEMM(BITS, TAIL, kAnyRow);                      \
    } while (0)
#define VQ_LAUNCH_BITS(BITS)                  \
    do {                                      \
        if (tail) VQ_LAUNCH_OUT(BITS, true);  \
        else VQ_LAUNCH_OUT(BITS, false);      \
    } while (0)
    if (w_bits == 8) VQ_LAUNCH_BITS(8);
    else if (w_bits == 16) VQ_LAUNCH_BITS(16);
    else if constexpr (S::kFourBits) VQ_LAUNCH_BITS(4);
#undef VQ_LAUNCH_BITS
#undef VQ_LAUNCH_OUT
#undef VQ_LAUNCH_GEMM
    return hipErrorInvalidValue;
}

}  // namespace
}  // namespace vq
