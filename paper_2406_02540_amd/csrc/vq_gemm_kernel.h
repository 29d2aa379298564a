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
// registers; the mainloop is otherwise the same.
//
// Shape of the kernel
//   - workgroup tile: 256 tokens x (64 WC) output channels, WT x WC wavefronts, each
//     wavefront (32 TB) tokens x 64 channels = 2 x TB MFMA 32x32x32 blocks.  Two tiles:
//       256 x 256: 2 x 4 wavefronts of 128 x 64 (128 int32 accumulators per lane), two
//                  wavefronts per SIMD;
//       256 x 192: 4 x 3 wavefronts of 64 x 64 (64 accumulators), three per SIMD: for
//                  channel counts that 256 does not divide well (1152 = 6 x 192: no
//                  half-empty column of tiles, and 768 tiles of 3/4 of the work fill 256
//                  CUs in three even rounds where 640 tiles of 256 x 256 need three
//                  rounds of whole tiles for 2.25 rounds of work).
//     The tile is large because the L2 -> CU path, not HBM, is what the operand traffic
//     loads: bytes per multiply-add fall with the tile edge.
//   - K is walked in stages of 128 bytes, double buffered in LDS.  A stage
//     takes one full 128-byte cache line per row, so every L2 request is a
//     whole line (with 64-byte stages the same bytes cost twice the requests and the
//     CU's address path saturates).  Activations and weights go global -> LDS directly
//     (buffer_load ... lds, 16 B per lane, no registers in between); the loads
//     of stage i+1 are in flight while stage i is multiplied.  4-bit weights
//     travel packed (half the bytes).
//   - The direct loads are issued from inline assembly and waited for with an
//     explicit s_waitcnt: the compiler would otherwise wait for all of them
//     before every LDS read and undo the prefetch.  They are paced, one load per
//     two MFMAs from the start of a stage: the CU's load path takes 64 bytes
//     per cycle, and a wave that queues there issues no MFMA.
//   - LDS tiles are [row][128 B] with the eight 16-byte chunks of a row XOR-ed
//     by (row/2)%8, which makes the 16-lane groups of a ds_read_b128 hit 16
//     different bank groups.
//   - The tokens are the MFMA row operand and the weights the column operand, so a lane owns one
//     column of each of its two blocks and, by permuting which weight row sits in which column, two
//     neighbouring output channels, for 16 TB tokens.  The epilogue narrows them to one dword in
//     registers and stores it: a store of a wave is two token rows x 128 bytes, whole lines,
//     bypassing the caches' retention (nontemporal: the operands keep the L2).  Nothing is turned
//     through LDS, a channel's scale and bias are one register each, and a token's scale is read
//     for two outputs of every lane at once.
//     What bounds the way out is vector instructions, about 15 cycles of a SIMD for an output of
//     64 lanes (conversion 4.4, product of the scales 2.4, mixed multiply-add 8.5; nothing of it
//     runs under MFMAs of the same SIMD): 3900 of the 29000 cycles that a 256 x 256 tile of nine
//     stages takes, 18400 of them MFMAs.  With a lane owning 32 channels of one token, staged
//     through LDS to be written as 16 bytes a lane, it was 33500: 20 LDS instructions of 16 bytes a
//     lane for 32 outputs bound it.  us, then / now: 32768 x 1152 -> 4608 171 / 159, -> 3456 133 /
//     126, 32768 x 384 -> 3456 73 / 62, 8192 x 1152 -> 3456 with 4-bit weights 37.2 / 33.7.
//   - The kernel is persistent: one workgroup per CU walks a list of tiles.
//     The first stage of the next tile is requested while the last stage of
//     the current one is multiplied, its second stage in the first pieces of the epilogue (all
//     at once ahead of it they kept every wave in the load queue for 850 cycles); the waves go
//     from the epilogue into the next tile without meeting at a barrier.
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
// (v_mfma_f32_32x32x16_f16, the same 16 bytes of K per lane and operand): the FP16 layer
// the paper's hardware evaluation compares against (Sec. 5.3), y = fp16(sum + bias).
#pragma once
#include <type_traits>

#include "vq_gemm_common.h"
#include "vq_internal.h"

namespace vq {

struct GemmArgs {
    const int8_t* xq;
    const float* x_scale;
    const void* w;
    const float* w_scale;
    const _Float16* bias;
    _Float16* y;
    int32_t* acc_out;
    int M, N, K;
    int tiles_t, tiles_c, tiles, tiles_per_xcd;
    int slots;  // workgroups per XCD; workgroup (xcd, slot) takes tiles slot, slot + slots, ... of its XCD
};

// The 256 x 192 tile (vq_gemm_192.hip); the tile fields of `a` are filled in by the callee.
hipError_t launch_gemm_192(const GemmArgs& a, int w_bits, int num_cus, hipStream_t stream);

namespace {

constexpr int kTileK = 128;                 // K bytes per stage (one cache line per row)
constexpr int kStages = 2;
constexpr int kScaleBytes = 3 * 1024;       // w_scale[256] fp32 | bias[256] fp16 (+pad) | x_scale[256] fp32
constexpr int kBand = 8;                    // token tiles per band in the tile order
constexpr int kXcds = 8;
constexpr int kTouchRounds = 4;             // weight lines asked for up front: at most 4 x 8 KiB per wave (64 MiB per 256 CUs)

// WT x WC wavefronts of (32 TB) tokens x 64 channels.
template <int WT_, int WC_, int TB_>
struct TileShape {
    static constexpr int WT = WT_, WC = WC_, TB = TB_;
    static constexpr int kWaves = WT * WC;
    static constexpr int kThreads = 64 * kWaves;
    static constexpr int kWavesPerSimd = kWaves / 4;
    static constexpr int kTileT = WT * TB * 32;       // tokens per workgroup
    static constexpr int kTileC = WC * 64;            // output channels per workgroup
    static constexpr int kXStage = kTileT * kTileK;   // 32 KiB
    static constexpr int kWStage = kTileC * kTileK;   // (half of it used by packed 4-bit weights)
    static constexpr int kLdsBytes = kStages * (kXStage + kWStage);
    // Global -> LDS loads of 1 KiB (8 rows of int8, 16 rows of nibbles).  The X tile is 32 of them.  With
    // eight waves each takes four of those and its share of the W tile; with more the loads of both tiles are
    // one list (groups 0 .. 31 X, the rest W), dealt round.
    static constexpr bool kOneList = kWaves > 8;
    static constexpr int groups(int w_bits) { return 32 + kTileC / (w_bits == 4 ? 16 : 8); }
    static constexpr int kStage = kXStage + kWStage;         // X tile, then W tile
    static constexpr int kWLoaders = 8;
    static constexpr int kWPer8 = kOneList ? 0 : kTileC / 8 / kWLoaders;    // int8 (and fp16) W loads per loading wave
    static constexpr int kWPer4 = kOneList ? 0 : kTileC / 16 / kWLoaders;   // packed 4-bit W loads per loading wave
    // The epilogue is 4 TB pieces of four stores; the next tile's loads go into all but the last four, so at least this
    // many of a wave's stores are behind them.
    static constexpr int kPieces = 4 * TB, kStoresBehind = 16;
    static_assert(kTileT == 256, "scales are fetched by threads 0..255, one token each");
    static_assert(kTileC <= 256 && kWaves % 4 == 0 && kWaves >= 8, "tile shape");
    static_assert(kOneList || (kTileC / 8 % kWLoaders == 0 && kTileC / 16 % kWLoaders == 0), "W loads divide evenly");
    static_assert(!kOneList || (kWaves % 2 == 0 && 2 * kWaves <= 32 && 3 * kWaves >= 32), "one turn of the list is mixed, and a wave's groups have its parity");
    static_assert(kLdsBytes + kScaleBytes <= 160 * 1024, "LDS of one CU");
};

// Where a tile sits in the output (wave-uniform).
struct TilePos {
    long tok0, ch0;
    int rows_x, rows_w;  // rows of the tile that exist (the rest is clamped on load, masked on store)
};
// What this wave's share of a tile's loads needs: buffer descriptors and per-lane offsets.
struct TileLoads {
    v4i rsrc_x, rsrc_w;
    int voff_x[4], voff_w[6];   // (one list: voff_w alone, by turn)
    int k_end_x, k_end_w;   // (used with a K tail only: see load_stage_to_lds_16)
};

// One 32 x 32 block: int8 operands (32 values of K per lane pair) into int32 sums, or,
// for the fp16 comparison layer, fp16 operands (16 values of K) into fp32 sums.  Both take
// 16 bytes of each operand per lane and as long to issue.
typedef float v16f __attribute__((ext_vector_type(16)));
template <int W_BITS>
struct AccOf { typedef v16i type; };
template <>
struct AccOf<16> { typedef v16f type; };
__device__ __forceinline__ v16i mfma_block(v4i x, v4i w, v16i c) {
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(x, w, c, 0, 0, 0);
}
__device__ __forceinline__ v16f mfma_block(v4i x, v4i w, v16f c) {
    // (a cast between vector types of one size reinterprets the bits)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16((half8)x, (half8)w, c, 0, 0, 0);
}

// K_TAIL:  K is a multiple of 16 but not of 128 (the last stage is partly past K).
// OUT:     how rows of Y are written (vq_gemm_common.h).
template <class S, int W_BITS, bool K_TAIL, Out OUT>
__global__ __launch_bounds__(S::kThreads, S::kWavesPerSimd) void gemm_i8_dequant(const GemmArgs a) {
    constexpr bool GENERIC = OUT == kAnyRow;
    constexpr int TB = S::TB;
    constexpr int kXStage = S::kXStage, kLdsBytes = S::kLdsBytes;
    __shared__ __attribute__((aligned(1024))) int8_t lds[kLdsBytes + kScaleBytes];
    // layout: [X buffer 0][W buffer 0][X buffer 1][W buffer 1][scales]; a W
    // buffer is [rows][128 B] of int8 or, for 4-bit weights, [rows][64 B] of nibbles.
    int8_t* const lds_x = lds;
    int8_t* const lds_w = lds + kXStage;
    constexpr int kStage = S::kStage;
    const unsigned lds_x_addr = (unsigned)(uintptr_t)(lds_ptr)lds_x;
    const unsigned lds_w_addr = (unsigned)(uintptr_t)(lds_ptr)lds_w;
    int8_t* const lds_sc = lds + kLdsBytes;  // w_scale | bias | x_scale of the current tile

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Waves w, w+4 (and w+8) share a SIMD: they get the same token part and different
    // channel slabs, so a tile that is only partly full of channels still
    // leaves a working wave on every SIMD.
    const int wave_t = wave % S::WT;   // which 32 TB tokens
    const int wave_c = wave / S::WT;   // which 64 channels
    // (W_BITS == 16: fp16 operands, the comparison layer; rows are 2 K bytes and everything up
    // to the MFMA itself treats them like int8 rows of that many bytes)
    const int K = (W_BITS == 16) ? 2 * a.K : a.K;      // bytes per activation row
    constexpr int kWDiv = (W_BITS == 4) ? 2 : 1;        // activation bytes per weight byte
    const int nk = (K + kTileK - 1) / kTileK;

    // What this wave loads per stage.
    constexpr int kWPer = (W_BITS != 4) ? S::kWPer8 : S::kWPer4;
    constexpr int kGroups = S::groups(W_BITS), kTurns = (kGroups + S::kWaves - 1) / S::kWaves;   // (one list)
    constexpr int kMixed = 32 / S::kWaves;   // the turn in which some waves load X and some W
    const bool mixed_x = wave + kMixed * S::kWaves < 32;
    const int w_loader = wave;

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
    int dec_band, dec_in_band;   // where the tile decoded last sits (wave-uniform)
    bool ld_full = false;        // that tile was a full one: its per-lane offsets hold for any full tile
    auto locate_tile = [&](int idx) {
        const int logical = (blockIdx.x % kXcds) * a.tiles_per_xcd + idx;
        dec_band = logical / band_tiles;
        dec_in_band = logical - dec_band * band_tiles;
    };
    auto step_tile = [&]() {
        dec_in_band += a.slots;
        while (dec_in_band >= band_tiles) {
            dec_in_band -= band_tiles;
            ++dec_band;
        }
    };
    auto decode_tile = [&](TilePos& t, TileLoads& ld) {
        const int band_first = dec_band * kBand;
        const int band_rows = min(a.tiles_t - band_first, kBand);
        int row, col;
        if (band_rows == kBand) {
            row = dec_in_band % kBand;
            col = dec_in_band / kBand;
        } else {  // the last band of a matrix whose token tiles are not a multiple of kBand
            row = dec_in_band % band_rows;
            col = dec_in_band / band_rows;
        }
        t.tok0 = (long)(band_first + row) * S::kTileT;
        t.ch0 = (long)col * S::kTileC;
        t.rows_x = (int)min((long)S::kTileT, a.M - t.tok0);
        t.rows_w = (int)min((long)S::kTileC, a.N - t.ch0);
        // (with a K tail the buffers end with the tile's last row: see load_stage_to_lds_16)
        ld.rsrc_x = make_rsrc(a.xq + t.tok0 * K, K_TAIL ? (unsigned)(t.rows_x * K) : clamp_u32((a.M - t.tok0) * (long)K));
        ld.rsrc_w = make_rsrc((const int8_t*)a.w + t.ch0 * (K / kWDiv),
                              K_TAIL ? (unsigned)(t.rows_w * (K / kWDiv)) : clamp_u32((a.N - t.ch0) * (long)(K / kWDiv)));
        // The per-lane offsets are relative to the tile and clamp rows past the matrix: between
        // two full tiles they do not change.  (Rows < 256 and row lengths < 2^24: 24-bit products.)
        const bool full = t.rows_x == S::kTileT && t.rows_w == S::kTileC;
        if (full && ld_full) return;
        ld_full = full;
        const int l = opaque(lane);
        const int ld_chunk16 = ((l & 7) ^ ((4 * (wave & 1) + (l >> 4)) & 7)) << 4;
        const int ld_chunk16_w4 = ((l & 3) ^ (l >> 4)) << 4;
        ld.k_end_x = K - ld_chunk16;
        ld.k_end_w = W_BITS != 4 ? K - ld_chunk16 : K / 2 - ld_chunk16_w4;
        auto x_offset = [&](int g) {
            return __mul24(min(g * 8 + (l >> 3), t.rows_x - 1), K) + ld_chunk16;
        };
        auto w_offset = [&](int g) {
            if (W_BITS != 4) return __mul24(min(w_row_to_channel(g * 8 + (l >> 3)), t.rows_w - 1), K) + ld_chunk16;
            return __mul24(min(w_row_to_channel(g * 16 + (l >> 2)), t.rows_w - 1), K / 2) + ld_chunk16_w4;
        };
        if constexpr (S::kOneList) {
#pragma unroll
            for (int j = 0; j < kTurns; ++j) {
                const int g = wave + j * S::kWaves;
                if (j < kMixed || (j == kMixed && mixed_x)) ld.voff_w[j] = x_offset(g);
                else ld.voff_w[j] = w_offset(g - 32);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) ld.voff_x[j] = x_offset(wave + 8 * j);
#pragma unroll
            for (int j = 0; j < kWPer; ++j) ld.voff_w[j] = w_offset(w_loader + S::kWLoaders * j);
        }
    };
    auto tile_exists = [&](int idx) {
        return idx < a.tiles_per_xcd && (int)(blockIdx.x % kXcds) * a.tiles_per_xcd + idx < a.tiles;
    };

    // One load of a wave's share of a stage.  A wave with both kinds alternates them (X, W, X,
    // W, ...) as long as it has W loads left.
    auto issue_x = [&](const TileLoads& ld, int buf, int k0, int j) {
        load_stage_to_lds_16<K_TAIL>(ld.rsrc_x, lds_x_addr + buf * kStage + (wave + 8 * j) * 1024, ld.voff_x[j], k0,
                                     ld.k_end_x);
    };
    auto issue_w = [&](const TileLoads& ld, int buf, int k0, int j) {
        load_stage_to_lds_16<K_TAIL>(ld.rsrc_w, lds_w_addr + buf * kStage + (w_loader + S::kWLoaders * j) * 1024,
                                     ld.voff_w[j], W_BITS != 4 ? k0 : k0 / 2, ld.k_end_w);
    };
    constexpr int kMaxSingles = S::kOneList ? kTurns : 4 + kWPer;
    static_assert(kMaxSingles <= 3 * TB, "three K steps carry a stage's loads");
    const int n_singles = S::kOneList ? (wave < kGroups - (kTurns - 1) * S::kWaves ? kTurns : kTurns - 1) : 4 + kWPer;
    auto issue_single = [&](const TileLoads& ld, int buf, int k0, int s) {
        if constexpr (S::kOneList) {
            // (s is a compile-time constant at every call; a mixed turn's kind is wave-uniform)
            const unsigned at = lds_x_addr + buf * kStage + (wave + s * S::kWaves) * 1024;
            if (s < kMixed || (s == kMixed && mixed_x))
                load_stage_to_lds_16<K_TAIL>(ld.rsrc_x, at, ld.voff_w[s], k0, ld.k_end_x);
            else
                load_stage_to_lds_16<K_TAIL>(ld.rsrc_w, at, ld.voff_w[s], W_BITS != 4 ? k0 : k0 / 2, ld.k_end_w);
        } else if (s < 2 * kWPer) {
            if (s & 1) issue_w(ld, buf, k0, s >> 1); else issue_x(ld, buf, k0, s >> 1);
        } else {
            issue_x(ld, buf, k0, s - kWPer);
        }
    };
    // With three wavefronts to a SIMD the youngest one comes to its products last, and loads dealt out among them arrived
    // late: it waited 240 of a stage's 2200 cycles for its own.  It asks for them ahead of its products.  us, then / now,
    // with 8-bit weights: 8192 x 1152 -> 1152 14.7 / 14.3, 8192 x 4096 -> 2304 75.4 / 72.6, 32768 x 4608 -> 1152 162 / 158.6,
    // 32768 x 1152 -> 1152 44.3 / 43.5.  The same for the middle one gives the gain back (75.8, 166, 44.2), as for the younger
    // one of two in 256 x 256 (32768 x 1152 -> 4608 160, 171 so); 4-bit weights, half of the bytes, are in time as it is.
    constexpr bool kYoungestFirst = S::kWavesPerSimd == 3 && W_BITS != 4;
    const int n_paced = kYoungestFirst && wave >= S::kWaves - 4 ? 0 : n_singles;
    auto issue_all = [&](const TileLoads& ld, int buf, int k0) {
#pragma unroll
        for (int s = 0; s < kMaxSingles; ++s)
            if (s < n_singles) issue_single(ld, buf, k0, s);
    };

    // ---- LDS -> MFMA operand mapping -----------------------------------------
    // Operand rows of a 32x32x32 block: lane l supplies row l%32, 16 bytes of K
    // chosen by l/32; a stage holds four such K steps (chunks 2ks and 2ks+1).
    // The chunk index of K step ks is (2 ks + l/32) ^ swizzle = ((l/32) ^ swizzle) ^ 2 ks, so the
    // byte offset of step ks is that of step 0 with 32 ks XOR-ed in.
    // 4-bit weights: two K steps 2j and 2j + 1 share one read of 16 bytes of nibbles, chunk 2j + l/32 of the row, whose
    // first half the lane widens for the one and second half for the other.  The activations follow: chunk 4j + 2 (l/32)
    // for the first, the one behind it for the second.  (Which 32 bytes of K a step takes does not change the sums.)
    // With a read of 8 bytes per step the 32 lanes served together took every other 8 bytes of their rows, half of the
    // banks, and the widening waited for LDS between the products.  us, then / now, in 256 x 192: 32768 x 4608 -> 1152 158 /
    // 152, 32768 x 1152 -> 1152 45.9 / 44.5, 8192 x 4096 -> 2304 76.4 / 73.8; in 256 x 256 32768 x 1152 -> 4608 161 / 159,
    // 8192 x 1152 -> 3456 33.3 / 32.9.
    const int fr_row = lane & 31;
    const int x_off0 = (wave_t * 32 * TB + fr_row) * kTileK + (((W_BITS != 4 ? lane >> 5 : lane >> 5 << 1) ^ ((fr_row >> 1) & 7)) << 4);
    const int w_off0 = (W_BITS != 4)
                           ? (wave_c * 64 + fr_row) * kTileK + (((lane >> 5) ^ ((fr_row >> 1) & 7)) << 4)
                           : (wave_c * 64 + fr_row) * (kTileK / 2) + (((lane >> 5) ^ ((fr_row >> 2) & 3)) << 4);
    auto x_off = [&](int ks) { return x_off0 ^ (W_BITS != 4 ? ks << 5 : (ks >> 1 << 6) + ((ks & 1) << 4)); };
    auto w_off = [&](int ks) { return w_off0 ^ (W_BITS != 4 ? ks << 5 : ks >> 1 << 5); };

    // ---- the tiles of this workgroup -------------------------------------------
    int idx = blockIdx.x / kXcds;
    if (!tile_exists(idx)) return;  // uniform per workgroup
    TilePos cur;   // the tile being multiplied
    TileLoads ld;  // the tile whose stages are being requested (the next one during the last stage)
    locate_tile(idx);
    decode_tile(cur, ld);
    int buf = 0;  // LDS buffer of the stage about to be multiplied
    bool requested1 = false;        // the current tile's second stage was requested in the previous epilogue
    bool stores_in_flight = false;  // this wave wrote outputs in the previous epilogue, kStoresBehind or more behind its loads
    issue_all(ld, 0, 0);
    // Every line of the weight matrix is asked for once, here, by the whole grid (one dword per
    // 128-byte line and lane, 8 KiB per wave and round): the weights are a few MB that every XCD
    // walks through completely, and a column's panel is otherwise first asked for by the eight
    // CUs that need it at that moment, which then wait out the memory latency at every stage of
    // their tile.  Fetched up front the lines are in the memory-side cache when their column's
    // turn comes.  (Range-checked loads: lanes past the end of the matrix fetch nothing.)
    int touched[kTouchRounds];
    {
        const long w_bytes = (long)a.N * (K / kWDiv);
        const __amdgpu_buffer_rsrc_t rsrc_all = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<void*>(a.w), 0, (int)clamp_u32(w_bytes), kRsrcFlags);
        const unsigned per_round = gridDim.x * (unsigned)S::kWaves * 8192u;
        const unsigned off = (blockIdx.x * (unsigned)S::kWaves + (unsigned)wave) * 8192u + (unsigned)lane * 128u;
#pragma unroll
        for (int i = 0; i < kTouchRounds; ++i) {
            touched[i] = 0;
            if ((long)i * per_round < w_bytes)  // (uniform; all rounds are in flight together)
                touched[i] = __builtin_amdgcn_raw_buffer_load_b32(rsrc_all, (int)(off + i * per_round), 0, 0);
        }
    }
    wait_loads_and_barrier();  // the first tile's first stage (later ones arrive behind an epilogue)
#pragma unroll
    for (int i = 0; i < kTouchRounds; ++i) asm volatile("" : : "v"(touched[i]));  // (not used; they have arrived by now)

    // Invariant at the top of a stage: its operands have landed in buffer `buf` for every
    // wave, and nobody reads or writes the other buffer any more.
    while (true) {
        const int next_idx = idx + a.slots;
        const bool has_next = tile_exists(next_idx);
        TilePos nxt = cur;

        // a wave whose 64 channels (or tokens) lie wholly past the matrix has nothing to multiply
        const bool wave_live = (wave_c * 64 < cur.rows_w) && (wave_t * 32 * TB < cur.rows_x);

        // Scales and bias of the tile: threads 0..255 fetch one channel and one token each
        // here and park them in LDS behind the last stage, where every lane of the epilogue
        // finds them.  Entries past N or M, and a missing bias, are zero.
        float pre_ws = 0.0f, pre_xs = 0.0f;
        _Float16 pre_b = (_Float16)0.0f;
        if (wave < 4) {
            const int i = wave * 64 + opaque(lane);
            if (i < S::kTileC && cur.ch0 + i < a.N) {
                if (W_BITS != 16) pre_ws = a.w_scale[cur.ch0 + i];
                if (a.bias) pre_b = a.bias[cur.ch0 + i];
            }
            if (W_BITS != 16 && cur.tok0 + i < a.M) pre_xs = a.x_scale[cur.tok0 + i];
        }

        auto park_scales = [&]() {
            if (wave < 4) {
                const int i = wave * 64 + opaque(lane);
                *(float*)(lds_sc + i * 4) = pre_ws;
                *(_Float16*)(lds_sc + 1024 + i * 2) = pre_b;
                // the 4-bit path accumulates 16 * w: the exact 1/16 rides on the token scale
                *(float*)(lds_sc + 2048 + i * 4) = pre_xs * (W_BITS == 4 ? 0.0625f : 1.0f);
            }
            // (They have arrived for every wave, which the compiler is told here, ahead of a wait for all loads: it
            // would otherwise wait for the next tile's second stage where it takes their registers for something else.)
            asm volatile("" : : "v"(pre_ws), "v"(pre_xs), "v"((int)__builtin_bit_cast(unsigned short, pre_b)));
        };

        typedef typename AccOf<W_BITS>::type acc_t;
        acc_t acc[2][TB];
        v4i xf[2][TB], wf[2][2];  // operand registers, double buffered; [1] carries K step 3 across stages
        v4i nibbles[2];           // (4-bit weights: of the two K steps that are read together)
        const acc_t kZero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};

        // One stage = four K steps of 2 TB MFMAs per wave.  The schedule is skewed by one K step:
        // the MFMAs of a stage's last K step are issued at the start of the next stage, behind
        // the barrier, where they cover the latency of that stage's first LDS reads (otherwise
        // every wave of the CU would sit idle there).  Compile-time flags: FIRST = the tile's
        // first stage (nothing deferred to run; its first K step starts the accumulators from
        // a constant zero), LAST = its last one (nothing is deferred past the epilogue).
        // `requested`: the loads this stage would issue are already in flight.
        auto stage = [&](const int it, auto first_tag, auto last_tag, const bool requested) __attribute__((always_inline)) {
            constexpr bool FIRST = decltype(first_tag)::value;
            constexpr bool LAST = decltype(last_tag)::value;
            // what to request while this stage is multiplied: the next stage of this tile,
            // or the first stage of the next tile
            const bool fetch = (!LAST || has_next) && !requested;
            // (In a stage of its own the next tile is located behind the first products: ahead of them every wave
            // of the CU would be at it at once and the matrix cores idle.)
            constexpr bool kLate = LAST && !FIRST;
            auto next_tile = [&]() __attribute__((always_inline)) {
                if (LAST && has_next) {
                    step_tile();
                    decode_tile(nxt, ld);
                }
            };
            if (!kLate) next_tile();
            const int fk0 = LAST ? 0 : (it + 1) * kTileK;

            const int8_t* xs = lds_x + buf * kStage;
            const int8_t* ws = lds_w + buf * kStage;
            // Operand registers are double buffered: the LDS reads of K step ks+1 are issued
            // among the MFMAs of step ks, which cover their latency.
            // A K step = 2 TB MFMAs in TB pieces of two.  A piece carries at most one global load
            // (so that a wave never sits in the load queue while the matrix pipe waits for it)
            // and its share of the LDS reads of the step after; sched_barrier(0) keeps the pieces
            // apart.  Reads of the next step in the order of their first use: w0 x0 x1 .. w1
            // (128-token waves: w0 x0 | x1 x2 | x3 w1; 64-token waves: w0 x0 x1 w1 in the first piece).
            constexpr int kReads = TB + 2;
            constexpr int kReadsPerPiece = (kReads + TB - 2) / (TB - 1);   // spread over all pieces but the last
            auto read_one = [&](int ks, int r, v4i(&xo)[TB], v4i(&wo)[2]) __attribute__((always_inline)) {
                if (r == 0 || r == kReads - 1) {
                    const int cb = (r == 0) ? 0 : 1;
                    if (W_BITS != 4)
                        wo[cb] = *(const v4i*)(ws + w_off(ks) + cb * 32 * kTileK);
                    else if (!(ks & 1))
                        nibbles[cb] = *(const v4i*)(ws + w_off(ks) + cb * 32 * (kTileK / 2));
                } else {
                    const int tb = r - 1;
                    xo[tb] = *(const v4i*)(xs + x_off(ks) + tb * 32 * kTileK);
                }
            };
            auto widen = [&](int ks, v4i(&wo)[2]) __attribute__((always_inline)) {
#pragma unroll
                for (int cb = 0; cb < 2; ++cb)
                    wo[cb] = widen_nibbles((ks & 1) ? v2i{nibbles[cb][2], nibbles[cb][3]} : v2i{nibbles[cb][0], nibbles[cb][1]});
            };
            auto mfma_one = [&](int i, const v4i(&xi)[TB], const v4i(&wi)[2], auto zero_tag) __attribute__((always_inline)) {
                const int cb = i / TB, tb = i % TB;
                if constexpr (decltype(zero_tag)::value)
                    acc[cb][tb] = mfma_block(xi[tb], wi[cb], kZero16);
                else
                    acc[cb][tb] = mfma_block(xi[tb], wi[cb], acc[cb][tb]);
            };
            // read_ks < 0: nothing left to read (the tile's last K step); first_load < 0: no loads
            auto k_step = [&](const v4i(&xi)[TB], const v4i(&wi)[2], auto zero_tag, int read_ks, v4i(&xo)[TB],
                              v4i(&wo)[2], int first_load) __attribute__((always_inline)) {
#pragma unroll
                for (int p = 0; p < TB; ++p) {
                    if (fetch && first_load >= 0 && first_load + p < kMaxSingles && first_load + p < n_paced)
                        issue_single(ld, buf ^ 1, fk0, first_load + p);
                    mfma_one(2 * p, xi, wi, zero_tag);
                    mfma_one(2 * p + 1, xi, wi, zero_tag);
                    if (read_ks >= 0) {
#pragma unroll
                        for (int r = p * kReadsPerPiece; r < (p + 1) * kReadsPerPiece && r < kReads; ++r)
                            read_one(read_ks, r, xo, wo);
                        if (W_BITS != 4 && p * kReadsPerPiece < kReads) {
                            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                   // one MFMA
                            __builtin_amdgcn_sched_group_barrier(0x100, kReadsPerPiece / 2, 0);  // LDS reads
                            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                            __builtin_amdgcn_sched_group_barrier(0x100, kReadsPerPiece / 2, 0);
                        }
                    }
                    // (in the last piece, which reads nothing: the nibbles have arrived behind the products before it)
                    if (W_BITS == 4 && read_ks >= 0 && p == TB - 1) widen(read_ks, wo);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            constexpr std::false_type kAccumulate{};
            // K steps in the order they are issued; the e-th one of a stage carries the loads
            // e TB .. e TB + TB - 1 of this wave's share.
            if (FIRST) {
                // nothing deferred to cover them: the first K step's operands are read up front
#pragma unroll
                for (int r = 0; r < kReads; ++r) read_one(0, r, xf[0], wf[0]);
                if (kYoungestFirst && fetch && n_paced == 0) issue_all(ld, buf ^ 1, fk0);
                if (W_BITS == 4) widen(0, wf[0]);
                __builtin_amdgcn_sched_barrier(0);
                k_step(xf[0], wf[0], first_tag, 1, xf[1], wf[1], 0);          // K step 0
                k_step(xf[1], wf[1], kAccumulate, 2, xf[0], wf[0], TB);      // K step 1
                k_step(xf[0], wf[0], kAccumulate, 3, xf[1], wf[1], 2 * TB);  // K step 2
            } else {
                constexpr int kAt = kLate ? -TB : 0;
                if (kYoungestFirst && !kLate && fetch && n_paced == 0) issue_all(ld, buf ^ 1, fk0);
                k_step(xf[1], wf[1], kAccumulate, 0, xf[0], wf[0], kAt);           // K step 3 of the previous stage
                if (kLate) {
                    next_tile();
                    if (kYoungestFirst && fetch && n_paced == 0) issue_all(ld, buf ^ 1, fk0);
                    __builtin_amdgcn_sched_barrier(0);
                }
                k_step(xf[0], wf[0], kAccumulate, 1, xf[1], wf[1], kAt + TB);      // K step 0
                k_step(xf[1], wf[1], kAccumulate, 2, xf[0], wf[0], kAt + 2 * TB);  // K step 1
                k_step(xf[0], wf[0], kAccumulate, 3, xf[1], wf[1], kAt + 3 * TB);  // K step 2
            }
            // K step 3 (otherwise at the start of the next stage)
            if (LAST) {
                k_step(xf[1], wf[1], kAccumulate, -1, xf[0], wf[0], -1);
                park_scales();
            }
            // The stage requested above has landed for every wave and every wave is done
            // reading this one.  After the last stage this also says: the scales are in LDS,
            // the next tile's first stage is in, and only stores can be outstanding later.
            // (A stage whose loads were requested in the previous tile's epilogue has stores of this
            // wave behind them: those may stay in flight.  Vector memory operations complete in the
            // order they were issued.)
            if (requested && stores_in_flight)
                wait_loads_before_and_barrier<S::kStoresBehind>();
            else
                wait_loads_and_barrier();
            buf ^= 1;
        };
        constexpr std::true_type kYes{};
        constexpr std::false_type kNo{};
        // (the next tile's second stage is requested before this tile ends)
        const bool request1 = has_next && nk >= 2;
        if (wave_live) {
            if (nk == 1) {
                stage(0, kYes, kYes, false);
            } else {
                stage(0, kYes, kNo, requested1);
#pragma unroll 1
                for (int it = 1; it < nk - 1; ++it) stage(it, kNo, kNo, false);
                stage(nk - 1, kNo, kYes, false);
            }

            // ---- epilogue ------------------------------------------------------------
            // Lane (h = lane/32, c = lane%32) holds channels 2c and 2c + 1 of the wavefront's 64 (accumulator blocks 0 and
            // 1) for the tokens 8j + 4h + i of each of its TB token blocks (register 4j + i).  Two neighbouring outputs are
            // one dword, and a store of one dword per lane is a whole 128-byte line of two token rows.
            const int el = opaque(lane);  // (the epilogue's per-lane values are not kept across the mainloop)
            const int h = el >> 5, pair = wave_c * 64 + 2 * (el & 31);   // the lane's first channel within the tile
            const int left = cur.rows_w - pair;                          // channels from there on that exist
            const int row0 = wave_t * 32 * TB;                           // the wave's first token within the tile
            const float ws0 = *(const float*)(lds_sc + pair * 4), ws1 = *(const float*)(lds_sc + pair * 4 + 4);
            const unsigned bias2 = *(const unsigned*)(lds_sc + 1024 + pair * 2);
            const int8_t* const sc_x = lds_sc + 2048 + (row0 + 4 * h) * 4;
            // Stores are range-checked, relative to the first of eight token rows: rows past M fall behind the end of
            // the buffer, lanes whose channels lie past N get an offset behind it (N < 2^21 on this path, so nothing
            // wraps).
            const unsigned y_place = left > 0 ? (unsigned)(__mul24(4 * h, GENERIC ? 0 : a.N) + (int)cur.ch0 + pair) * 2u : 0x80000000u;
            unsigned y_off[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) y_off[i] = y_place + (unsigned)checked_bytes<OUT>(i, a.N);
            const _Float16* y_row = a.y + (cur.tok0 + row0) * a.N;
            int y_bytes = checked_bytes<OUT>(cur.rows_x - row0, a.N);   // from there to the end of the tile's rows
            // (any row: token rows of the wave below which the lane has two channels to write, or one; its place in them)
            const int rows_live = cur.rows_x - row0 - 4 * h;
            const int rows_pair = left > 1 ? rows_live : 0, rows_single = left == 1 ? rows_live : 0;
            long y_any[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) y_any[i] = (4 * h + i) * (long)a.N + cur.ch0 + pair;
            if (GENERIC && a.acc_out) {
                int32_t* acc_row = a.acc_out + (cur.tok0 + row0) * a.N;
#pragma unroll
                for (int tb = 0; tb < TB; ++tb)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (tb * 32 + 8 * j + i < rows_live && left > 0) {
                                constexpr int kShift = (W_BITS == 4) ? 4 : 0;
                                acc_row[y_any[i]] = (int)acc[0][tb][4 * j + i] >> kShift;
                                if (left > 1) acc_row[y_any[i] + 1] = (int)acc[1][tb][4 * j + i] >> kShift;
                            }
                        acc_row += 8 * (long)a.N;
                        asm volatile("" : "+s"(acc_row));
                    }
            }
            v4f xs = *(const v4f*)sc_x;
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    // the next tile's second stage, a few loads at a time
#pragma unroll
                    for (int l = 0; l < kMaxSingles; ++l)
                        if (l * (S::kPieces - 4) / kMaxSingles == 4 * tb + j && l < n_singles && request1) issue_single(ld, buf ^ 1, kTileK, l);
                    v4f xs_next = xs;
                    if (tb < TB - 1 || j < 3) xs_next = *(const v4f*)(sc_x + (tb * 32 + 8 * (j + 1)) * 4);
                    const __amdgpu_buffer_rsrc_t rsrc_y =
                        __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(y_row), 0, max(y_bytes, 0), kRsrcFlags);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int r = 4 * j + i;
                        unsigned out;
                        // y = fp16(float(acc) * (x_scale * w_scale) + bias): the product of the two scales rounded to
                        // fp32, the rest exact and rounded once (dequant_pair)
                        if constexpr (W_BITS == 16)  // the fp32 sum of the fp16 products, plus the bias
                            out = add_bias_pair(acc[0][tb][r], acc[1][tb][r], bias2);
                        else
                            out = dequant_pair((float)acc[0][tb][r], xs[i] * ws0, (float)acc[1][tb][r], xs[i] * ws1, bias2);
                        if (!GENERIC) {
                            __builtin_amdgcn_raw_buffer_store_b32((int)out, rsrc_y, y_off[i], 0, OUT == kHalfLines ? 2 /* nontemporal */ : 0);
                            continue;
                        }
                        // Rows of Y that start at any even address; the last channel of an odd N alone.
                        typedef unsigned u_any __attribute__((aligned(2)));
                        if (tb * 32 + 8 * j + i < rows_pair) *(u_any*)(y_row + y_any[i]) = out;
                        if ((cur.rows_w & 1) && tb * 32 + 8 * j + i < rows_single)
                            *(unsigned short*)(y_row + y_any[i]) = (unsigned short)out;
                    }
                    xs = xs_next;
                    y_row += 8 * (long)a.N;
                    y_bytes -= checked_bytes<OUT>(8, a.N);
                    if (GENERIC) asm volatile("" : "+s"(y_row), "+v"(xs));   // (nothing is made up ahead of its use)
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        } else {
            // nothing to multiply in this tile, but this wave's share of the loads is needed
#pragma unroll 1
            for (int it = 0; it < nk; ++it) {
                const bool more = it + 1 < nk;
                if (!more && has_next) {
                    step_tile();
                    decode_tile(nxt, ld);
                }
                if ((more || has_next) && !(it == 0 && requested1)) issue_all(ld, buf ^ 1, more ? (it + 1) * kTileK : 0);
                if (!more) park_scales();
                wait_loads_and_barrier();
                buf ^= 1;
            }
            if (request1) issue_all(ld, buf ^ 1, kTileK);
        }
        requested1 = request1;
        stores_in_flight = wave_live && !GENERIC;
        if (!has_next) break;
        // Of LDS the epilogue reads the scales alone, and its loads go to the stage buffer that was free
        // from the last stage's barrier on.  With two stages and more the barrier that ends the next
        // tile's first one comes before that tile's scales are parked, so the waves go on without
        // meeting; a one-stage tile parks them before its only barrier: nobody may still be reading.
        if (nk == 1) wait_lds_and_barrier();
        cur = nxt;
        idx = next_idx;
    }
}

// Enqueues the kernel for tile shape S; `a` holds the operands and sizes.
template <class S>
hipError_t launch_gemm_shape(GemmArgs a, int w_bits, int num_cus, hipStream_t stream) {
    if (a.M > 0x7FFFFF00 || a.N > 0x7FFFFF00) return hipErrorInvalidValue;  // (rows and channels of a last tile fit an int)
    a.tiles_t = (a.M + S::kTileT - 1) / S::kTileT;
    a.tiles_c = (a.N + S::kTileC - 1) / S::kTileC;
    const long tiles = (long)a.tiles_t * a.tiles_c;
    if (tiles > 0x7FFFFFF0l) return hipErrorInvalidValue;
    a.tiles = (int)tiles;
    a.tiles_per_xcd = (a.tiles + kXcds - 1) / kXcds;
    // one workgroup per CU (the kernel needs most of a CU's LDS), fewer if there are fewer tiles
    const int cus_per_xcd = num_cus >= kXcds ? num_cus / kXcds : 1;
    a.slots = a.tiles_per_xcd < cus_per_xcd ? a.tiles_per_xcd : cus_per_xcd;
    const dim3 grid((unsigned)(a.slots * kXcds)), block(S::kThreads);
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
    else VQ_LAUNCH_BITS(4);
#undef VQ_LAUNCH_BITS
#undef VQ_LAUNCH_OUT
#undef VQ_LAUNCH_GEMM
    return hipErrorInvalidValue;
}

}  // namespace
}  // namespace vq
