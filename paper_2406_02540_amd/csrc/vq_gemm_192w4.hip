// The 256 x 192 tile for packed 4-bit weights: the persistent kernel of vq_gemm_kernel.h (same arithmetic, same
// walk through the tiles; ViDiT-Q appendices "Hardware implementation of quantized linear layers" and "Performance under
// lower bitwidth") in 32 x 32 x 32 blocks instead of 16 x 16 x 64.
//
// The template in that shape, 4-bit weights read without bank conflicts, over 70 random problems of this tile takes 1.05 of this
// kernel's time (1.00 to 1.10).  us, 16 x 16 x 64 / 32 x 32 x 32: 8192 x 4608 -> 1152 43.2 / 41.4, 32768 x 4608 -> 1152 165.8 /
// 155.8, 32768 x 1152 -> 1152 47.3 / 44.9, 8192 x 1152 -> 4608 47.4 / 44.6.  Its clock is higher (2.26 GHz and 2.15 in the first,
// 2.07 and 1.90 in the second) and its cycles are a tenth more (117400 and 104300, 326000 and 296000): the matrix cores' are the
// same, the vector instructions a tenth more (64 tokens for 64 channels are two and a half of widening for each 16 x 16 x 64
// product), and wavefronts wait as often.  With three stages of activations 160.0 in the second, 1.05 over the 70; shorter than
// here in 11, long K and few columns of tiles (31465 x 4608 -> 558 93 us, 101 here).  With 128 tokens for 64 channels (256 x 256)
// 16 x 16 x 64 is the faster one.
//
//   - 4 x 3 wavefronts of 64 tokens x 64 channels, 2 x 2 blocks each, three to a SIMD; K in stages of 128 bytes, double
//     buffered in LDS.  4-bit weights travel packed and are widened to 16 * w on their way from LDS into the operand registers.
//   - LDS tiles are [row][128 B] ([row][64 B] of nibbles) with the 16-byte chunks of a row XOR-ed by (row/2)%8 ((row/4)%4).
//   - The tokens are the MFMA row operand, and the weights' rows are interleaved so that a lane owns two neighbouring output
//     channels; the epilogue narrows them to one dword and stores it from the registers, two token rows x 128 bytes a store.
#include <type_traits>

#include "vq_gemm_common.h"
#include "vq_internal.h"

namespace vq {

namespace {

constexpr int kStages = 2;
constexpr int kScaleBytes = 3 * 1024;       // w_scale[256] fp32 | bias[256] fp16 (+pad) | x_scale[256] fp32
// 4 x 3 wavefronts of 64 tokens x 64 channels.
struct S {
    static constexpr int WT = 4, WC = 3, TB = 2;
    static constexpr int kWaves = WT * WC;
    static constexpr int kThreads = 64 * kWaves;
    static constexpr int kWavesPerSimd = kWaves / 4;
    static constexpr int kTileT = WT * TB * 32;       // tokens per workgroup
    static constexpr int kTileC = WC * 64;            // output channels per workgroup
    static constexpr int kXStage = kTileT * kTileK;   // 32 KiB
    static constexpr int kStage = kXStage + kTileC * kTileK / 2;     // X tile, then W tile
    static constexpr int kLdsBytes = kStages * kStage;
    // Global -> LDS loads of 1 KiB (8 rows of int8, 16 rows of nibbles).  The X tile is 32 of them; the loads of both tiles are
    // one list (groups 0 .. 31 X, the rest W), dealt round.
    static constexpr int kGroups = 32 + kTileC / 16;
    // The epilogue is 4 TB pieces of four stores; the next tile's loads go into all but the last four, so at least this
    // many of a wave's stores are behind them.
    static constexpr int kPieces = 4 * TB, kStoresBehind = 16;
    static_assert(kTileT == 256, "scales are fetched by threads 0..255, one token each");
    static_assert(kWaves % 2 == 0 && 2 * kWaves <= 32 && 3 * kWaves >= 32, "one turn of the list is mixed, and a wave's groups have its parity");
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
    int voff[4];            // by turn
    int k_end_x, k_end_w;   // (used with a K tail only: see load_stage_to_lds_16)
};

// K_TAIL:  K is not a multiple of 128 (the last stage is partly past K).
// OUT:     how rows of Y are written (vq_gemm_common.h).
template <bool K_TAIL, Out OUT>
__global__ __launch_bounds__(S::kThreads, S::kWavesPerSimd) void gemm_w4_dequant_192(const GemmArgs a) {
    constexpr bool GENERIC = OUT == kAnyRow;
    constexpr int TB = S::TB;
    constexpr int kXStage = S::kXStage, kLdsBytes = S::kLdsBytes;
    __shared__ __attribute__((aligned(1024))) int8_t lds[kLdsBytes + kScaleBytes];
    // layout: [X buffer 0][W buffer 0][X buffer 1][W buffer 1][scales]; an X buffer is [rows][128 B], a W buffer [rows][64 B]
    // of nibbles.
    int8_t* const lds_x = lds;
    int8_t* const lds_w = lds + kXStage;
    constexpr int kStage = S::kStage;
    const unsigned lds_x_addr = (unsigned)(uintptr_t)(lds_ptr)lds_x;
    int8_t* const lds_sc = lds + kLdsBytes;  // w_scale | bias | x_scale of the current tile

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Waves w, w+4 and w+8 share a SIMD: they get the same token part and different
    // channel slabs, so a tile that is only partly full of channels still
    // leaves a working wave on every SIMD.
    const int wave_t = wave % S::WT;   // which 32 TB tokens
    const int wave_c = wave / S::WT;   // which 64 channels
    const int K = a.K;      // bytes per activation row, twice those of a weight row
    const int nk = (K + kTileK - 1) / kTileK;

    // What this wave loads per stage.
    constexpr int kTurns = (S::kGroups + S::kWaves - 1) / S::kWaves;
    constexpr int kMixed = 32 / S::kWaves;   // the turn in which some waves load X and some W
    const bool mixed_x = wave + kMixed * S::kWaves < 32;

    // ---- global -> LDS mapping ---------------------------------------------
    // One direct load fills 1 KiB; lane l writes bytes [16 l, 16 l + 16).
    // Activations: 8 rows x 128 B per load, lane l = row l/8, physical chunk l%8,
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
        ld.rsrc_w = make_rsrc((const int8_t*)a.w + t.ch0 * (K / 2),
                              K_TAIL ? (unsigned)(t.rows_w * (K / 2)) : clamp_u32((a.N - t.ch0) * (long)(K / 2)));
        // The per-lane offsets are relative to the tile and clamp rows past the matrix: between
        // two full tiles they do not change.  (Rows < 256 and row lengths < 2^24: 24-bit products.)
        const bool full = t.rows_x == S::kTileT && t.rows_w == S::kTileC;
        if (full && ld_full) return;
        ld_full = full;
        const int l = opaque(lane);
        const int ld_chunk16 = ((l & 7) ^ ((4 * (wave & 1) + (l >> 4)) & 7)) << 4;
        const int ld_chunk16_w4 = ((l & 3) ^ (l >> 4)) << 4;
        ld.k_end_x = K - ld_chunk16;
        ld.k_end_w = K / 2 - ld_chunk16_w4;
        auto x_offset = [&](int g) {
            return __mul24(min(g * 8 + (l >> 3), t.rows_x - 1), K) + ld_chunk16;
        };
        auto w_offset = [&](int g) {
            return __mul24(min(w_row_to_channel(g * 16 + (l >> 2)), t.rows_w - 1), K / 2) + ld_chunk16_w4;
        };
#pragma unroll
        for (int j = 0; j < kTurns; ++j) {
            const int g = wave + j * S::kWaves;
            if (j < kMixed || (j == kMixed && mixed_x)) ld.voff[j] = x_offset(g);
            else ld.voff[j] = w_offset(g - 32);
        }
    };
    auto tile_exists = [&](int idx) {
        return idx < a.tiles_per_xcd && (int)(blockIdx.x % kXcds) * a.tiles_per_xcd + idx < a.tiles;
    };

    // One load of a wave's share of a stage.
    static_assert(kTurns <= 3 * TB, "three K steps carry a stage's loads");
    const int n_singles = wave < S::kGroups - (kTurns - 1) * S::kWaves ? kTurns : kTurns - 1;
    auto issue_single = [&](const TileLoads& ld, int buf, int k0, int s) {
        // (s is a compile-time constant at every call; a mixed turn's kind is wave-uniform)
        const unsigned at = lds_x_addr + buf * kStage + (wave + s * S::kWaves) * 1024;
        if (s < kMixed || (s == kMixed && mixed_x))
            load_stage_to_lds_16<K_TAIL>(ld.rsrc_x, at, ld.voff[s], k0, ld.k_end_x);
        else
            load_stage_to_lds_16<K_TAIL>(ld.rsrc_w, at, ld.voff[s], k0 / 2, ld.k_end_w);
    };
    auto issue_all = [&](const TileLoads& ld, int buf, int k0) {
#pragma unroll
        for (int s = 0; s < kTurns; ++s)
            if (s < n_singles) issue_single(ld, buf, k0, s);
    };

    // ---- LDS -> MFMA operand mapping -----------------------------------------
    // Operand rows of a 32x32x32 block: lane l supplies row l%32, 16 bytes of K
    // chosen by l/32; a stage holds four such K steps (chunks 2ks and 2ks+1).
    // Two K steps 2j and 2j + 1 share one read of 16 bytes of nibbles, chunk 2j + l/32 of the row, whose
    // first half the lane widens for the one and second half for the other.  The activations follow: chunk 4j + 2 (l/32)
    // for the first, the one behind it for the second.  (Which 32 bytes of K a step takes does not change the sums.)
    // With a read of 8 bytes per step the 32 lanes served together took every other 8 bytes of their rows, half of the
    // banks, and the widening waited for LDS between the products.  us, then / now: 32768 x 4608 -> 1152 158 /
    // 152, 32768 x 1152 -> 1152 45.9 / 44.5, 8192 x 4096 -> 2304 76.4 / 73.8.
    const int fr_row = lane & 31;
    const int x_off0 = (wave_t * 32 * TB + fr_row) * kTileK + (((lane >> 5 << 1) ^ ((fr_row >> 1) & 7)) << 4);
    const int w_off0 = (wave_c * 64 + fr_row) * (kTileK / 2) + (((lane >> 5) ^ ((fr_row >> 2) & 3)) << 4);
    auto x_off = [&](int ks) { return x_off0 ^ ((ks >> 1 << 6) + ((ks & 1) << 4)); };
    auto w_off = [&](int ks) { return w_off0 ^ (ks >> 1 << 5); };

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
        const long w_bytes = (long)a.N * (K / 2);
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
                pre_ws = a.w_scale[cur.ch0 + i];
                if (a.bias) pre_b = a.bias[cur.ch0 + i];
            }
            if (cur.tok0 + i < a.M) pre_xs = a.x_scale[cur.tok0 + i];
        }

        auto park_scales = [&]() {
            if (wave < 4) {
                const int i = wave * 64 + opaque(lane);
                *(float*)(lds_sc + i * 4) = pre_ws;
                *(_Float16*)(lds_sc + 1024 + i * 2) = pre_b;
                // (the sums are of 16 * w: the exact 1/16 rides on the token scale)
                *(float*)(lds_sc + 2048 + i * 4) = pre_xs * 0.0625f;
            }
            // (They have arrived for every wave, which the compiler is told here, ahead of a wait for all loads: it
            // would otherwise wait for the next tile's second stage where it takes their registers for something else.)
            asm volatile("" : : "v"(pre_ws), "v"(pre_xs), "v"((int)__builtin_bit_cast(unsigned short, pre_b)));
        };

        v16i acc[2][TB];
        v4i xf[2][TB], wf[2][2];  // operand registers, double buffered; [1] carries K step 3 across stages
        v4i nibbles[2];           // of the two K steps that are read together
        const v16i kZero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};

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
            // (w0 x0 x1 w1 in the first piece).
            constexpr int kReads = TB + 2;
            constexpr int kReadsPerPiece = (kReads + TB - 2) / (TB - 1);   // spread over all pieces but the last
            auto read_one = [&](int ks, int r, v4i(&xo)[TB], v4i(&wo)[2]) __attribute__((always_inline)) {
                if (r == 0 || r == kReads - 1) {
                    const int cb = (r == 0) ? 0 : 1;
                    if (!(ks & 1))
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
                    acc[cb][tb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xi[tb], wi[cb], kZero16, 0, 0, 0);
                else
                    acc[cb][tb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xi[tb], wi[cb], acc[cb][tb], 0, 0, 0);
            };
            // read_ks < 0: nothing left to read (the tile's last K step); first_load < 0: no loads
            auto k_step = [&](const v4i(&xi)[TB], const v4i(&wi)[2], auto zero_tag, int read_ks, v4i(&xo)[TB],
                              v4i(&wo)[2], int first_load) __attribute__((always_inline)) {
#pragma unroll
                for (int p = 0; p < TB; ++p) {
                    if (fetch && first_load >= 0 && first_load + p < kTurns && first_load + p < n_singles)
                        issue_single(ld, buf ^ 1, fk0, first_load + p);
                    mfma_one(2 * p, xi, wi, zero_tag);
                    mfma_one(2 * p + 1, xi, wi, zero_tag);
                    if (read_ks >= 0) {
#pragma unroll
                        for (int r = p * kReadsPerPiece; r < (p + 1) * kReadsPerPiece && r < kReads; ++r)
                            read_one(read_ks, r, xo, wo);
                    }
                    // (in the last piece, which reads nothing: the nibbles have arrived behind the products before it)
                    if (read_ks >= 0 && p == TB - 1) widen(read_ks, wo);
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
                widen(0, wf[0]);
                __builtin_amdgcn_sched_barrier(0);
                k_step(xf[0], wf[0], first_tag, 1, xf[1], wf[1], 0);          // K step 0
                k_step(xf[1], wf[1], kAccumulate, 2, xf[0], wf[0], TB);      // K step 1
                k_step(xf[0], wf[0], kAccumulate, 3, xf[1], wf[1], 2 * TB);  // K step 2
            } else {
                constexpr int kAt = kLate ? -TB : 0;
                k_step(xf[1], wf[1], kAccumulate, 0, xf[0], wf[0], kAt);           // K step 3 of the previous stage
                if (kLate) {
                    next_tile();
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
                                constexpr int kShift = 4;
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
                    for (int l = 0; l < kTurns; ++l)
                        if (l * (S::kPieces - 4) / kTurns == 4 * tb + j && l < n_singles && request1) issue_single(ld, buf ^ 1, kTileK, l);
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

}  // namespace

hipError_t launch_gemm_192w4(GemmArgs a, int num_cus, hipStream_t stream) {
    dim3 grid;
    if (!persistent_grid(a, grid, S::kTileT, S::kTileC, num_cus)) return hipErrorInvalidValue;
    const bool tail = a.K % kTileK != 0;
    const Out out = rows_out(a.N, a.y, a.acc_out);
    const dim3 block(S::kThreads);
    if (out == kHalfLines) return enqueue(tail ? gemm_w4_dequant_192<true, kHalfLines> : gemm_w4_dequant_192<false, kHalfLines>, grid, block, stream, a);
    if (out == kDwords) return enqueue(tail ? gemm_w4_dequant_192<true, kDwords> : gemm_w4_dequant_192<false, kDwords>, grid, block, stream, a);
    return enqueue(tail ? gemm_w4_dequant_192<true, kAnyRow> : gemm_w4_dequant_192<false, kAnyRow>, grid, block, stream, a);
}

}  // namespace vq
