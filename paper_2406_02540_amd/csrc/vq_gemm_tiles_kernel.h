// int8 x int8 -> int32 MFMA GEMM with the dequantization epilogue for problems whose tiles of
// 256 tokens would not fill the chip (same arithmetic as vq_gemm_kernel.h; ViDiT-Q appendix
// "Hardware implementation of quantized linear layers").
//
// Such a launch is one or two tiles per CU long, so what counts is what happens once: the start,
// the first stage's memory latency (the caches of an XCD start cold), the way out.  Hence one
// workgroup per tile, not persistent, with a short epilogue, and small tiles (chosen by
// launch_gemm's cost table) so that every CU has one.  A tile is WT x WC wavefronts of (32 BT)
// tokens x (32 BC) channels, times KW groups of such wavefronts: the groups share the tile and
// divide the K steps of every stage among themselves (their sums meet in LDS at the end), which is
// what puts two to four wavefronts on a SIMD where the tile alone has work for one.  K is walked in
// stages of 128 bytes (one cache line per row) through a ring of RING LDS buffers, RING - 1 stages
// of direct-to-LDS loads in flight: a CU takes at most about 54 bytes per cycle on this path
// (0.26 us for the 32 KiB of a 128 x 128 stage out of L2, against 0.21 us for its products), and
// only as many bytes as the ring holds per memory latency (about 0.9 us beyond L2).
//
// GEMM alone in a captured graph, us (8-bit / 4-bit weights): 240 x 4096 -> 2304 in 64 x 64 tiles 9.2 / 11.4, 1001 x
// 1152 -> 4608 in 128 x 256 11.1 / 11.6, 2048 x 1152 -> 1152 in 128 x 128 8.4 / 8.7, 4096 x 1152 -> 1152 in 128 x 256 11.2.
// Of the 11 us at 1001 x 1152 -> 4608 1.7 are the launch, 1.7 the way to the first stage (start, twelve loads per wavefront at
// the load path's rate, memory), nine stages 0.63 each against 0.43 of products, and 1.9 the way out (0.8 of vector
// instructions, the rest stores: 144 CUs write 9.2 MB).  Problems of fewer or smaller tiles: vq_gemm_split.h.
#pragma once
#include <type_traits>

#include "vq_gemm_common.h"
#include "vq_internal.h"

namespace vq {

namespace {

constexpr int kStageK = 128;      // K bytes per stage

template <int WT_, int WC_, int BT_, int BC_, int KW_, int RING_, int WGS_>
struct OneTile {
    static constexpr int WT = WT_, WC = WC_, BT = BT_, BC = BC_, KW = KW_, RING = RING_;
    static constexpr int kSpatial = WT * WC;              // wavefronts of one K group
    static constexpr int kWaves = kSpatial * KW;
    static constexpr int kThreads = 64 * kWaves;
    static constexpr int kWavesPerSimd = (kWaves * WGS_ + 3) / 4;  // WGS_ workgroups share a CU
    static constexpr int kT = WT * BT * 32;               // tokens of the tile
    static constexpr int kC = WC * BC * 32;               // channels of the tile
    static constexpr int kXS = kT * kStageK, kWS = kC * kStageK;
    // The way out: through LDS, or straight from the registers of wavefronts with two blocks of channels.  There the K
    // groups share the tile's token rows, eight at a time: kMine such pieces are a wavefront's own.
    static constexpr bool kDirect = BC == 2;
    static constexpr int kMine = 4 * BT / KW;
    // int32 sums in LDS once the stages are done: every K group's tile, or what the groups hand to each other
    static constexpr int kSums = kDirect ? kWaves * (KW - 1) * kMine * BC * 1024 : KW * kT * kC * 4;
    static constexpr int kScales = kC * 4 + kT * 4 + kC * 2;
    static constexpr int kWgs = WGS_;
    static_assert((4 / KW) * KW == 4, "K groups");
    static_assert(BC <= 2, "blocks of channels");
    static_assert(kThreads == shared_tile_threads(kT), "what launch_gemm counts with");
};

// Stage loads younger than the one needed: LEFT stages of PER loads.
template <int PER, int MAX_LEFT>
__device__ __forceinline__ void wait_stages(int left) {
    if constexpr (MAX_LEFT == 0) {
        wait_loads_before_and_barrier<0>();
    } else {
        if (left >= MAX_LEFT) wait_loads_before_and_barrier<PER * MAX_LEFT>();
        else wait_stages<PER, MAX_LEFT - 1>(left);
    }
}

// OUT: how rows of Y are written where they leave from the registers (vq_gemm_common.h; kAnyRow otherwise).
template <class S, int W_BITS, bool K_TAIL, Out OUT>
__global__ __launch_bounds__(S::kThreads, S::kWavesPerSimd) void gemm_i8_dequant_tile(const TileArgs a) {
    constexpr int BT = S::BT, BC = S::BC, KW = S::KW, RING = S::RING;
    constexpr int kXArea = RING * S::kXS, kStaged = RING * (S::kXS + S::kWS);
    constexpr int kBody = kStaged > S::kSums ? kStaged : S::kSums;
    static_assert((kBody + S::kScales) * S::kWgs <= 160 * 1024, "LDS of one CU");
    __shared__ __attribute__((aligned(1024))) int8_t lds[kBody + S::kScales];
    int8_t* const lds_x = lds;
    int8_t* const lds_w = lds + kXArea;
    int8_t* const lds_sc = lds + kBody;   // w_scale[kC] | x_scale[kT] | bias[kC]
    const unsigned lds_x_addr = (unsigned)(uintptr_t)(lds_ptr)lds_x;
    const unsigned lds_w_addr = (unsigned)(uintptr_t)(lds_ptr)lds_w;

    int row, col;
    if (!locate_tile(a.grid, row, col)) return;
    const int tok0 = row * S::kT, ch0 = col * S::kC;   // (< M, < N)

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave / S::kSpatial, sp = wave % S::kSpatial;
    const int wave_t = sp % S::WT, wave_c = sp / S::WT;
    const int K = a.K;
    constexpr int kWDiv = (W_BITS == 8) ? 1 : 2;
    const int rows_x = min(S::kT, a.M - tok0);
    const int rows_w = min(S::kC, a.N - ch0);
    const int nk = (K + kStageK - 1) / kStageK;

    // ---- global -> LDS ---------------------------------------------------------------------
    // One load fills 1 KiB: 8 rows x 128 B (lane l: row l/8, physical chunk l%8 holding logical
    // chunk (l%8) ^ ((row/2)%8)) or, for packed nibbles, 16 rows x 64 B (row l/4, chunk (l%4) ^
    // ((row/4)%4)).  Row groups 0 .. kXG-1 are activations, the rest weights; wavefront w takes
    // groups w, w + kWaves, ...
    constexpr int kXG = S::kT / 8, kWG = (W_BITS == 8) ? S::kC / 8 : S::kC / 16;
    constexpr int kGroups = kXG + kWG;
    constexpr int kPer = (kGroups + S::kWaves - 1) / S::kWaves;     // loads of a wavefront per stage
    constexpr int kFull = kGroups - (kPer - 1) * S::kWaves;          // wavefronts that have that many
    // (the buffers end with the tile's last row: see load_stage_to_lds_16)
    const v4i rsrc_x = make_rsrc(a.xq + (long)tok0 * K, (unsigned)(rows_x * K));
    const v4i rsrc_w = make_rsrc((const int8_t*)a.w + (long)ch0 * (K / kWDiv), (unsigned)(rows_w * (K / kWDiv)));
    int voff[kPer], k_end[kPer];   // (k_end: used with a K tail only)
    // (Every turn of the list loads one operand, which the compiler is told: with a branch on the wavefront's number in
    // front of every load the 64 x 64 tile took 2 to 4 % longer, with 4-bit weights 5 to 7 %, 128 x 256 2 %.  With 4-bit weights
    // the groups of 32 x 32, 64 x 64 and 128 x 64 fill the last turn in part, which keeps the branch and a second wait count.)
    static_assert(kXG % S::kWaves == 0, "whole turns of activations");
    constexpr int kXTurns = kXG / S::kWaves;
    // (two blocks of channels are interleaved: a lane then owns two neighbours)
    auto channel_of = [](int r) { return S::kDirect ? w_row_to_channel(r) : r; };
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int g = wave + S::kWaves * j;
        if (j < kXTurns) {
            const int r = g * 8 + (lane >> 3);
            const int at = ((lane & 7) ^ ((r >> 1) & 7)) << 4;
            voff[j] = __mul24(min(r, rows_x - 1), K) + at;
            k_end[j] = K - at;
        } else if (W_BITS == 8) {
            const int r = (g - kXG) * 8 + (lane >> 3);
            const int at = ((lane & 7) ^ ((r >> 1) & 7)) << 4;
            voff[j] = __mul24(min(channel_of(r), rows_w - 1), K) + at;
            k_end[j] = K - at;
        } else {
            const int r = (g - kXG) * 16 + (lane >> 2);
            const int at = ((lane & 3) ^ ((r >> 2) & 3)) << 4;
            voff[j] = __mul24(min(channel_of(r), rows_w - 1), K / 2) + at;
            k_end[j] = K / 2 - at;
        }
    }
    auto issue_one = [&](int slot, int k0, int j) {
        const int g = wave + S::kWaves * j;   // (wave-uniform)
        if (j == kPer - 1 && kFull < S::kWaves && wave >= kFull) return;
        if (j < kXTurns)
            load_stage_to_lds_16<K_TAIL>(rsrc_x, lds_x_addr + slot * S::kXS + g * 1024, voff[j], k0, k_end[j]);
        else
            load_stage_to_lds_16<K_TAIL>(rsrc_w, lds_w_addr + slot * S::kWS + (g - kXG) * 1024, voff[j], k0 / kWDiv,
                                         k_end[j]);
    };
    auto issue_stage = [&](int slot, int k0) {
#pragma unroll
        for (int j = 0; j < kPer; ++j) issue_one(slot, k0, j);
    };
    // Waits until stage `it` has landed for every wavefront (up to RING - 2 younger ones stay in flight).
    auto wait_stage = [&](int it) {
        const int left = nk - 1 - it;
        if (kFull < S::kWaves && wave >= kFull)
            wait_stages<kPer - 1, RING - 2>(left);
        else
            wait_stages<kPer, RING - 2>(left);
    };

#pragma unroll
    for (int s = 0; s < RING - 1; ++s)
        if (s < nk) issue_stage(s, s * kStageK);

    // Scales and bias, one channel and token per thread, behind the first stages; parked in LDS behind the mainloop.
    constexpr int kPre = (S::kC > S::kT ? S::kC : S::kT) > S::kThreads ? 2 : 1;
    static_assert(kPre * S::kThreads >= S::kC && kPre * S::kThreads >= S::kT, "scales");
    float pre_ws[kPre], pre_xs[kPre];
    _Float16 pre_b[kPre];
#pragma unroll
    for (int p = 0; p < kPre; ++p) {
        const int i = tid + p * S::kThreads;
        pre_ws[p] = a.w_scale[ch0 + min(i, rows_w - 1)];
        pre_xs[p] = a.x_scale[tok0 + min(i, rows_x - 1)];
        pre_b[p] = a.bias ? a.bias[ch0 + min(i, rows_w - 1)] : (_Float16)0.0f;
    }

    auto park_scales = [&]() {
#pragma unroll
        for (int p = 0; p < kPre; ++p) {
            const int i = tid + p * S::kThreads;
            if (i < S::kC) *(float*)(lds_sc + i * 4) = pre_ws[p];
            if (i < S::kT) *(float*)(lds_sc + S::kC * 4 + i * 4) = pre_xs[p];
            if (i < S::kC) *(_Float16*)(lds_sc + S::kC * 4 + S::kT * 4 + i * 2) = pre_b[p];
        }
    };

    // ---- LDS -> MFMA operands ---------------------------------------------------------------
    // 4-bit weights, kPairs: one read of 16 bytes of nibbles for K steps 2j and 2j + 1, as in vq_gemm_kernel.h, widened behind
    // the products that cover it.  1001 x 1152 -> 4608 in 128 x 256 11.75 us with a read per step, 11.55 so, 240 x 4096 ->
    // 2304 in 128 x 128 18.5 and 18.15.  With one block of channels there is less to widen than to wait for: 128 x 64 there
    // 13.85 and 14.2.
    constexpr int kSteps = 4 / KW;   // K steps of a stage that are this group's
    constexpr bool kPairs = W_BITS == 4 && kSteps > 1 && BC > 1;
    const int fr_row = lane & 31;
    const int x_off0 = (wave_t * 32 * BT + fr_row) * kStageK + (((kPairs ? lane >> 5 << 1 : lane >> 5) ^ ((fr_row >> 1) & 7)) << 4);
    const int w_off0 = (W_BITS == 8)
                           ? (wave_c * 32 * BC + fr_row) * kStageK + (((lane >> 5) ^ ((fr_row >> 1) & 7)) << 4)
                       : kPairs
                           ? (wave_c * 32 * BC + fr_row) * (kStageK / 2) + (((lane >> 5) ^ ((fr_row >> 2) & 3)) << 4)
                           : (wave_c * 32 * BC + fr_row) * (kStageK / 2) + (((fr_row >> 2) & 3) << 4) + (lane >> 5) * 8;

    v16i acc[BC][BT];
#pragma unroll
    for (int cb = 0; cb < BC; ++cb)
#pragma unroll
        for (int tb = 0; tb < BT; ++tb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[cb][tb][r] = 0;
    // (the rows of a block are its first operand: tokens where the outputs leave from the registers)
    auto product = [&](v4i w, v4i x, v16i c) __attribute__((always_inline)) {
        return __builtin_amdgcn_mfma_i32_32x32x32_i8(S::kDirect ? x : w, S::kDirect ? w : x, c, 0, 0, 0);
    };
    // Operand registers are double buffered: the products of a K step are issued behind the LDS
    // reads of the step after it, across the stage barrier too.
    v4i xf[2][BT], wf[2][BC];
#pragma unroll
    for (int tb = 0; tb < BT; ++tb) xf[1][tb] = v4i{0, 0, 0, 0};
#pragma unroll
    for (int cb = 0; cb < BC; ++cb) wf[1][cb] = v4i{0, 0, 0, 0};

    auto stage = [&](int it, int slot, auto parity_tag) __attribute__((always_inline)) {
        constexpr int P = decltype(parity_tag)::value;
        if (S::kDirect && it == nk - 1) park_scales();   // (a barrier of the stages is behind them)
        wait_stage(it);
        const bool fetch = it + RING - 1 < nk;
        const int f_slot = slot == 0 ? RING - 1 : slot - 1, f_k0 = (it + RING - 1) * kStageK;
        const int8_t* xs = lds_x + slot * S::kXS;
        const int8_t* ws = lds_w + slot * S::kWS;
        v4i nibbles[BC];
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            const int cur = (s + P) & 1;
            const int ks = kg * kSteps + s;
#pragma unroll
            for (int cb = 0; cb < BC; ++cb) {
                if (W_BITS == 8)
                    wf[cur][cb] = *(const v4i*)(ws + (w_off0 ^ (ks << 5)) + cb * 32 * kStageK);
                else if (kPairs && s % 2 == 0)
                    nibbles[cb] = *(const v4i*)(ws + (w_off0 ^ (ks >> 1 << 5)) + cb * 32 * (kStageK / 2));
                else if (!kPairs)
                    wf[cur][cb] = widen_nibbles(*(const v2i*)(ws + (w_off0 ^ (ks << 4)) + cb * 32 * (kStageK / 2)));
            }
#pragma unroll
            for (int tb = 0; tb < BT; ++tb)
                xf[cur][tb] = *(const v4i*)(xs + (x_off0 ^ (kPairs ? (ks >> 1 << 6) + (s % 2 << 4) : ks << 5)) + tb * 32 * kStageK);
            __builtin_amdgcn_sched_barrier(0);
            // The stage's loads are spread over its products (the CU's load path takes 64 bytes per
            // cycle: a burst of loads keeps the wavefront from its products).
#pragma unroll
            for (int m = 0; m < BC * BT; ++m) {
                constexpr int kProducts = kSteps * BC * BT;
                const int at = s * BC * BT + m;
#pragma unroll
                for (int j = 0; j < kPer; ++j)
                    if (j * kProducts / kPer == at && fetch) issue_one(f_slot, f_k0, j);
                const int cb = m / BT, tb = m % BT;
                acc[cb][tb] = product(wf[cur ^ 1][cb], xf[cur ^ 1][tb], acc[cb][tb]);
                __builtin_amdgcn_sched_barrier(0);
            }
            // (behind the products, which cover the way from LDS)
            if (kPairs)
#pragma unroll
                for (int cb = 0; cb < BC; ++cb)
                    wf[cur][cb] = widen_nibbles(s % 2 ? v2i{nibbles[cb][2], nibbles[cb][3]} : v2i{nibbles[cb][0], nibbles[cb][1]});
        }
    };
    auto last_products = [&](auto parity_tag) __attribute__((always_inline)) {
        constexpr int P = decltype(parity_tag)::value;
#pragma unroll
        for (int cb = 0; cb < BC; ++cb)
#pragma unroll
            for (int tb = 0; tb < BT; ++tb)
                acc[cb][tb] = product(wf[P][cb], xf[P][tb], acc[cb][tb]);
    };
    typedef std::integral_constant<int, 0> P0;
    typedef std::integral_constant<int, 1> P1;
    int slot = 0;
    auto next_slot = [&] { slot = (slot == RING - 1) ? 0 : slot + 1; };
    if constexpr (kSteps % 2 == 0) {
#pragma unroll 1
        for (int it = 0; it < nk; ++it) {
            stage(it, slot, P0{});
            next_slot();
        }
        last_products(P1{});
    } else {  // one step per stage: the operand buffers alternate from stage to stage
        int it = 0;
#pragma unroll 1
        for (; it + 1 < nk; it += 2) {
            stage(it, slot, P0{});
            next_slot();
            stage(it + 1, slot, P1{});
            next_slot();
        }
        if (it < nk) {
            stage(it, slot, P0{});
            last_products(P0{});
        } else {
            last_products(P1{});
        }
    }

    if constexpr (S::kDirect) {
        // ---- sums of the K groups, dequantization, rows of the output ------------------------------------------------
        // Lane (h = lane/32, c = lane%32) holds channels 2c and 2c + 1 of the wavefront's 64 for the tokens 8j + 4h + i of
        // each of its blocks (register 4j + i): two neighbouring outputs are one dword, stored from the registers.  Pieces
        // of eight token rows are numbered 4 tb + j; group g takes kMine of them from g kMine on: it hands the others their
        // share of its sums through LDS (16 bytes a lane, as they lie in the registers) and adds theirs to its own.
        // All sums through LDS, in the loop below, were 7000 of the 27000 cycles of 1001 x 1152 -> 4608 in 128 x 256: 13.4 us, 11.1
        // as it is (4-bit weights 14.4 and 12.2), 2048 x 1152 -> 1152 in 128 x 128 9.3 and 8.4, in 128 x 64 9.3 and 8.6.  The
        // instructions are seen once, so how rows are written is a template parameter: as a branch the first took 13.1 us again.
        // With one block of channels a dword is two lanes' outputs, and the loop's few instructions are the faster way: 512 x
        // 1152 -> 1152 in 64 x 64 4.8 us through LDS, 5.2 from the registers.
        constexpr int kMine = S::kMine;
        v4i mine[kMine][BC];
        auto sums = [&](int q, int cb) __attribute__((always_inline)) {
            const int tb = q >> 2, j = q & 3;
            return v4i{acc[cb][tb][4 * j], acc[cb][tb][4 * j + 1], acc[cb][tb][4 * j + 2], acc[cb][tb][4 * j + 3]};
        };
        if constexpr (KW > 1) {
            // what group `from` (one of the others, numbered without the taker) hands to group `to` of its piece p
            auto handed = [&](int to, int from, int p, int cb) {
                return (v4i*)(lds + ((((to * S::kSpatial + sp) * (KW - 1) + from) * kMine + p) * BC + cb) * 1024 + lane * 16);
            };
            wait_lds_and_barrier();   // nobody reads the stage buffers any more
#pragma unroll
            for (int g = 0; g < KW; ++g) {
                if (kg == g) continue;   // (uniform)
#pragma unroll
                for (int p = 0; p < kMine; ++p)
#pragma unroll
                    for (int cb = 0; cb < BC; ++cb) *handed(g, kg - (kg > g), p, cb) = sums(g * kMine + p, cb);
            }
            wait_lds_and_barrier();
#pragma unroll
            for (int g = 0; g < KW; ++g)
                if (kg == g)
#pragma unroll
                    for (int p = 0; p < kMine; ++p)
#pragma unroll
                        for (int cb = 0; cb < BC; ++cb) mine[p][cb] = sums(g * kMine + p, cb);
#pragma unroll
            for (int from = 0; from < KW - 1; ++from)
#pragma unroll
                for (int p = 0; p < kMine; ++p)
#pragma unroll
                    for (int cb = 0; cb < BC; ++cb) mine[p][cb] += *handed(kg, from, p, cb);
        } else {
#pragma unroll
            for (int p = 0; p < kMine; ++p)
#pragma unroll
                for (int cb = 0; cb < BC; ++cb) mine[p][cb] = sums(p, cb);
        }
        const int row0 = wave_t * 32 * BT + 8 * kMine * kg;   // the wavefront's first token row within the tile
        if (row0 >= rows_x) return;
        const int h = lane >> 5, pair = wave_c * 64 + 2 * (lane & 31), left = rows_w - pair;   // the lane's channels that exist
        const long y_first = (long)(tok0 + row0) * a.N + ch0;
        long y_at[4];   // a piece's four token rows, the lane's place in them
#pragma unroll
        for (int i = 0; i < 4; ++i) y_at[i] = (long)(4 * h + i) * a.N + pair;
        // (token rows below which the lane has two channels to write, or one)
        const int rows_live = rows_x - row0 - 4 * h;
        const int rows_pair = left > 1 ? rows_live : 0, rows_single = left == 1 ? rows_live : 0;
        if (OUT == kAnyRow && a.acc_out) {
            // Two neighbours are one store of 8 bytes.  us with sums, through LDS in stores of 16 bytes / from the registers in
            // two of 4 / as it is: 1001 x 1152 -> 4608 in 128 x 256 18.7 / 18.7 / 17.2, 2048 x 1152 -> 1152 in 128 x 128 12.7 /
            // 13.1 / 12.3; 2800 random problems in these tiles, over the first way, 1.02 to 1.05 and 0.93 to 0.96 on average.
            typedef v2i v2i_any4 __attribute__((aligned(4)));
            constexpr int kShift = (W_BITS == 4) ? 4 : 0;
#pragma unroll
            for (int p = 0; p < kMine; ++p)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    int32_t* const at = a.acc_out + y_first + 8 * p * (long)a.N + y_at[i];
                    const int sum0 = mine[p][0][i] >> kShift, sum1 = mine[p][1][i] >> kShift;
                    if (8 * p + i < rows_pair) *(v2i_any4*)at = v2i{sum0, sum1};
                    if ((rows_w & 1) && 8 * p + i < rows_single) *at = sum0;
                }
        }
        const int8_t* const sc_x = lds_sc + S::kC * 4 + (row0 + 4 * h) * 4;
        const float ws0 = *(const float*)(lds_sc + pair * 4), ws1 = *(const float*)(lds_sc + pair * 4 + 4);
        const unsigned bias2 = *(const unsigned*)(lds_sc + S::kC * 4 + S::kT * 4 + pair * 2);
        _Float16* y_row = a.y + y_first;
        int y_bytes = OUT == kAnyRow ? 0 : ((rows_x - row0) * a.N - ch0) * 2;   // from there to the end of the tile's rows
#pragma unroll
        for (int p = 0; p < kMine; ++p) {
            // (the 4-bit path summed 16 * w)
            const v4f xs = *(const v4f*)(sc_x + p * 32) * (W_BITS == 4 ? 0.0625f : 1.0f);
            unsigned out[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                out[i] = dequant_pair((float)mine[p][0][i], xs[i] * ws0, (float)mine[p][1][i], xs[i] * ws1, bias2);
            if (OUT != kAnyRow) {
                // (range-checked: rows past M and, by an offset behind the buffer, channels past N are not written)
                const __amdgpu_buffer_rsrc_t rsrc_y = __builtin_amdgcn_make_buffer_rsrc(y_row, 0, max(y_bytes, 0), kRsrcFlags);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    __builtin_amdgcn_raw_buffer_store_b32((int)out[i], rsrc_y, left > 0 ? (int)y_at[i] * 2 : (int)0x80000000, 0,
                                                          OUT == kHalfLines ? 2 /* nontemporal */ : 0);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    typedef unsigned u_any __attribute__((aligned(2)));
                    if (8 * p + i < rows_pair) *(u_any*)(y_row + y_at[i]) = out[i];
                    if ((rows_w & 1) && 8 * p + i < rows_single) *(unsigned short*)(y_row + y_at[i]) = (unsigned short)out[i];
                }
            }
            y_row += 8 * (long)a.N;
            y_bytes -= checked_bytes<OUT>(8, a.N);
        }
        return;
    }

    // ---- the sums, through LDS, to rows of the output ------------------------------------------------
    // Every group leaves its sums as a row-major int32 tile, 16-byte chunks (four channels) XOR-ed by
    // the row; then a thread takes eight consecutive channels of a row at a time, adds the groups'
    // sums, dequantizes and writes 16 bytes, consecutive threads along the row.  A thread's channels
    // are the same in every row it takes, so their scales and biases stay in registers.  (The code is
    // short on purpose: it runs once per workgroup, and instructions not seen before come from L2.)
    park_scales();
    wait_lds_and_barrier();   // nobody reads the stage buffers any more
    constexpr int kXor = (S::kC / 4) % 16 == 0 ? 15 : 7;
    constexpr int kRow = S::kC * 4;
    {
        const int t = wave_t * 32 * BT + (lane & 31);
        int8_t* const mine = lds + kg * (S::kT * kRow) + t * kRow;
#pragma unroll
        for (int cb = 0; cb < BC; ++cb)
#pragma unroll
            for (int tb = 0; tb < BT; ++tb)
#pragma unroll
                for (int j = 0; j < 4; ++j) {   // register 4j + i is channel 8j + 4 (lane/32) + i of the block
                    const int chunk = (wave_c * BC + cb) * 8 + 2 * j + (lane >> 5);
                    *(v4i*)(mine + tb * 32 * kRow + ((chunk ^ (t & kXor)) << 4)) =
                        v4i{acc[cb][tb][4 * j], acc[cb][tb][4 * j + 1], acc[cb][tb][4 * j + 2], acc[cb][tb][4 * j + 3]};
                }
    }
    wait_lds_and_barrier();
    constexpr int kPerRow = S::kC / 8;                       // threads of a row
    constexpr int kRowStep = S::kThreads / kPerRow;          // rows taken at a time
    if (kRowStep * kPerRow < S::kThreads && tid >= kRowStep * kPerRow) return;
    const int c0 = (tid % kPerRow) * 8;
    if (c0 >= rows_w) return;
    const v4f s0 = *(const v4f*)(lds_sc + c0 * 4), s1 = *(const v4f*)(lds_sc + c0 * 4 + 16);
    const v4i bias8 = *(const v4i*)(lds_sc + S::kC * 4 + S::kT * 4 + c0 * 2);
#pragma unroll 1
    for (int t = tid / kPerRow; t < rows_x; t += kRowStep) {
        v4i v0 = {0, 0, 0, 0}, v1 = v0;
#pragma unroll
        for (int g = 0; g < KW; ++g) {
            const int8_t* row = lds + g * (S::kT * kRow) + t * kRow;
            v0 += *(const v4i*)(row + (((c0 >> 2) ^ (t & kXor)) << 4));
            v1 += *(const v4i*)(row + ((((c0 >> 2) + 1) ^ (t & kXor)) << 4));
        }
        const float xsc = *(const float*)(lds_sc + S::kC * 4 + t * 4);
        const long at = (long)(tok0 + t) * a.N + ch0 + c0;
        write_eight<W_BITS>(v0, v1, xsc, s0, s1, bias8, rows_w - c0, a.y + at, a.acc_out ? a.acc_out + at : nullptr);
    }
}

template <class S, int W_BITS>
hipError_t launch_tile_shape(TileArgs a, hipStream_t stream) {
    if (!tile_grid(a.grid, a.M, a.N, S::kT, S::kC, S::kThreads)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(a.grid.tiles_per_xcd * kTileXcds)), block(S::kThreads);
    auto launch = [&](auto out_tag) {
        constexpr Out OUT = decltype(out_tag)::value;
        return enqueue(a.K % kStageK ? gemm_i8_dequant_tile<S, W_BITS, true, OUT> : gemm_i8_dequant_tile<S, W_BITS, false, OUT>, grid,
                       block, stream, a);
    };
    if constexpr (S::kDirect) {
        const Out out = rows_out(a.N, a.y, a.acc_out);
        if (out == kHalfLines) return launch(std::integral_constant<Out, kHalfLines>{});
        if (out == kDwords) return launch(std::integral_constant<Out, kDwords>{});
    }
    return launch(std::integral_constant<Out, kAnyRow>{});
}

}  // namespace
}  // namespace vq
