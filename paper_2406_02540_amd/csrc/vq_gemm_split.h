// int8 x int8 -> int32 MFMA GEMM with the dequantization epilogue for the smallest problems (same
// arithmetic as vq_gemm_kernel.h; ViDiT-Q appendix "Hardware implementation of quantized linear
// layers"): one tile per workgroup, and the wavefronts of a workgroup divide K, not the tile.
//
// A wavefront takes every KW-th line (128 bytes of K) of the tile's rows: it loads the line into LDS
// space of its own, waits for its own loads, multiplies the whole tile over that line and asks for its
// next one.  Nothing is shared until the sums meet at the end, so there is one workgroup barrier in
// the kernel and none per stage; a wavefront that waits for memory holds up nobody, and every operand
// byte is read from LDS once.
//
// What bounds such a launch is the way to the first load, one memory latency and the CU's load path (54
// bytes per cycle).  Where the wavefronts share the tile (vq_gemm_tiles_kernel.h) a stage of a 32 x 32
// tile took 350 cycles, for barrier, LDS latency and one product each, and with 4-bit weights 500.  In a
// captured graph over four sets of operands, shared tiles of 32 x 32 (last line: of 64 x 64) / the best of the tiles here, us:
//   tokens x K -> channels   W8 shared / divided   W4 shared / divided
//   16 x 1152 -> 1152            4.0 / 3.35            4.5 / 3.3
//   16 x 4608 -> 1152            6.7 / 5.0             9.0 / 4.35
//   100 x 512 -> 700             3.3 / 3.45            3.55 / 3.45
//   256 x 1152 -> 1152           4.7 / 3.9             5.25 / 3.85
//   240 x 4096 -> 2304           9.15 / 9.15          11.5 / 8.5
// 48 x 48 in blocks of 16 x 16 x 64 (where: choose_gemm in vq_gemm.hip): 240 of them are 7.3 and 6.8 us there, 144 of 64 x 64 9.2 and 8.2.
// 4-bit weights: a read of 16 bytes of nibbles for two K steps, 0.99 of the time with one of 8 bytes for each.
// A wavefront's next loads leave in a burst as soon as its operands are in registers, ahead of its
// products; dealt out between the products they were up to 10 % later with 32 x 32 tiles.  With many tiles per CU
// the operand bytes count, and larger shared tiles catch up (512 x 1152 -> 1152: 32 x 32 here 4.7 us, 64 x 64 shared 4.7) and
// win (1001 x 1152 -> 4608: here 18.7, 128 x 256 shared 10.4).
#pragma once
#include <type_traits>

#include "vq_gemm_common.h"
#include "vq_internal.h"

namespace vq {
namespace {

// (BLK BT) tokens x (BLK BC) channels in MFMA blocks of BLK x BLK (32 x 32 x 32 or 16 x 16 x 64), KW wavefronts; WGS
// workgroups share a CU.
template <int BT_, int BC_, int KW_, int WGS_, int BLK_ = 32>
struct SplitTile {
    static constexpr int BT = BT_, BC = BC_, KW = KW_, WGS = WGS_, BLK = BLK_;
    static constexpr int kThreads = 64 * KW;
    static constexpr int kWavesPerSimd = (KW * WGS_ + 3) / 4;
    static constexpr int kT = BLK * BT, kC = BLK * BC;
    static constexpr int kSums = kT * kC * 4;
    static constexpr int slot(int w_bits) {   // a wavefront's LDS: its line of both operands, then its sums
        const int line = kT * kLine + kC * kLine * w_bits / 8;
        return line > kSums ? line : kSums;
    }
};

template <int BLK>
struct BlockSums { typedef v16i type; };
template <>
struct BlockSums<16> { typedef v4i type; };
__device__ __forceinline__ v16i split_block(v4i w, v4i x, v16i c) { return __builtin_amdgcn_mfma_i32_32x32x32_i8(w, x, c, 0, 0, 0); }
__device__ __forceinline__ v4i split_block(v4i w, v4i x, v4i c) { return __builtin_amdgcn_mfma_i32_16x16x64_i8(w, x, c, 0, 0, 0); }

template <class S, int W_BITS, bool K_TAIL>
__global__ __launch_bounds__(S::kThreads, S::kWavesPerSimd) void gemm_i8_dequant_split(const TileArgs a) {
    constexpr int BT = S::BT, BC = S::BC, KW = S::KW, BLK = S::BLK;
    constexpr int kSlot = S::slot(W_BITS);
    static_assert(kSlot * KW * S::WGS <= 160 * 1024, "LDS of one CU");
    __shared__ __attribute__((aligned(1024))) int8_t lds[kSlot * KW];
    int row, col;
    if (!locate_tile(a.grid, row, col)) return;
    const int tok0 = row * S::kT, ch0 = col * S::kC;   // (< M, < N)

    const int M = a.M, N = a.N, K = a.K;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int kWDiv = (W_BITS == 8) ? 1 : 2;
    const int rows_x = min(S::kT, M - tok0), rows_w = min(S::kC, N - ch0);
    const int nl = (K + kLine - 1) / kLine;

    // ---- global -> LDS: one load fills 1 KiB, 8 rows x 128 B (lane l: row l/8, physical chunk l%8
    // holding logical chunk (l%8) ^ ((row/2)%8)) or, for packed nibbles, 16 rows x 64 B (row l/4, chunk
    // (l%4) ^ ((row/4)%4)).  Rows past the tile's last one lie behind the buffers.
    int8_t* const mine = lds + wave * kSlot;
    const unsigned mine_addr = (unsigned)(uintptr_t)(lds_ptr)mine;
    constexpr int kXLoads = S::kT / 8, kWLoads = (W_BITS == 8) ? S::kC / 8 : S::kC / 16, kWAt = S::kT * kLine;
    const v4i rsrc_x = make_rsrc(a.xq + (long)tok0 * K, (unsigned)(rows_x * K));
    const v4i rsrc_w = make_rsrc((const int8_t*)a.w + (long)ch0 * (K / kWDiv), (unsigned)(rows_w * (K / kWDiv)));
    int vx[kXLoads], vw[kWLoads];
    // (row groups all have the swizzle of row l/8 with bit 2 of row/2 from the group's parity)
#pragma unroll
    for (int g = 0; g < kXLoads; ++g) {
        const int r = g * 8 + (lane >> 3);
        vx[g] = __mul24(r, K) + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
    }
#pragma unroll
    for (int g = 0; g < kWLoads; ++g) {
        if (W_BITS == 8) {
            const int r = g * 8 + (lane >> 3);
            vw[g] = __mul24(r, K) + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
        } else {
            const int r = g * 16 + (lane >> 2);
            vw[g] = __mul24(r, K / 2) + (((lane & 3) ^ ((r >> 2) & 3)) << 4);
        }
    }
    constexpr int kLoads = kWLoads + kXLoads;
    auto issue_one = [&](int line, int i) __attribute__((always_inline)) {
        const int k0 = line * kLine;
        if (i < kWLoads) {
            constexpr int kRowsPer = (W_BITS == 8) ? 8 : 16;
            const int at = (W_BITS == 8) ? ((lane & 7) ^ (((i * 8 + (lane >> 3)) >> 1) & 7)) << 4
                                         : ((lane & 3) ^ (((i * 16 + (lane >> 2)) >> 2) & 3)) << 4;
            if (i * kRowsPer < rows_w)   // (uniform)
                load_stage_to_lds_16<K_TAIL>(rsrc_w, mine_addr + kWAt + i * 1024, vw[i], k0 / kWDiv, K / kWDiv - at);
        } else {
            const int g = i - kWLoads;
            const int at = ((lane & 7) ^ (((g * 8 + (lane >> 3)) >> 1) & 7)) << 4;
            if (g * 8 < rows_x) load_stage_to_lds_16<K_TAIL>(rsrc_x, mine_addr + g * 1024, vx[g], k0, K - at);
        }
    };
    auto issue = [&](int line) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) issue_one(line, i);
    };
    if (wave < nl) issue(wave);

    // What the way out needs, asked for here (in three loads: eight scales, eight biases and a token's scale one
    // by one were 0.5 us of 3.7 at 16 x 1152 -> 1152): a thread takes eight consecutive channels of kItems tokens.
    constexpr int kPerRow = S::kC / 8, kRowStep = S::kThreads / kPerRow;
    constexpr int kItems = (S::kT + kRowStep - 1) / kRowStep;
    static_assert(kRowStep * kPerRow == S::kThreads || kItems == 1, "whole rows of threads");
    const int c0 = (tid % kPerRow) * 8, t0 = tid / kPerRow;
    // (the tile's own scales: 4 N is past an int from 2^29 channels on; range-checked, dword by dword: channels past N
    // read as zero)
    const __amdgpu_buffer_rsrc_t rs_ws =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.w_scale) + ch0, 0, rows_w * 4, kRsrcFlags);
    const v4f s0 = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rs_ws, c0 * 4, 0, 0));
    const v4f s1 = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rs_ws, c0 * 4 + 16, 0, 0));
    v4i bias8 = {0, 0, 0, 0};
    if (a.bias) {
        if (c0 + 8 <= rows_w) {
            bias8 = *(const v4i*)(a.bias + ch0 + c0);
        } else {
            half8 b{};
#pragma unroll
            for (int e = 0; e < 7; ++e)
                if (c0 + e < rows_w) b[e] = a.bias[ch0 + c0 + e];
            bias8 = (v4i)b;
        }
    }
    float xsc[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) xsc[i] = a.x_scale[tok0 + min(t0 + i * kRowStep, rows_x - 1)];

    // ---- a line at a time ------------------------------------------------------------------
    // A line is kSteps K steps; a lane takes 16 bytes of K of each, by its group: with blocks of 32
    // (two groups) chunk 2 ks + group, of 16 (four) 4 ks + group.  (4-bit weights: 16 bytes of nibbles serve two K steps, as in
    // vq_gemm_kernel.h.)
    constexpr int kSteps = BLK / 8, kGroups = 64 / BLK;
    const int fr_row = lane & (BLK - 1), group = lane / BLK;
    const int part = W_BITS == 4 && BLK == 16 ? nibble_chunk(group) : group;   // of the row
    const int x_off0 = fr_row * kLine + (((W_BITS == 8 ? part : part << 1) ^ ((fr_row >> 1) & 7)) << 4);
    const int w_off0 = kWAt + ((W_BITS == 8) ? x_off0 : fr_row * (kLine / 2) + ((part ^ ((fr_row >> 2) & 3)) << 4));
    typedef typename BlockSums<BLK>::type sums_t;
    sums_t acc[BC][BT];
#pragma unroll
    for (int cb = 0; cb < BC; ++cb)
#pragma unroll
        for (int tb = 0; tb < BT; ++tb)
#pragma unroll
            for (int r = 0; r < BLK * BLK / 64; ++r) acc[cb][tb][r] = 0;
    constexpr int kWReads = W_BITS == 8 ? kSteps : kSteps / 2;
#pragma unroll 1
    for (int line = wave; line < nl; line += KW) {
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        v4i xf[kSteps][BT];
        v4i wf[kWReads][BC];
#pragma unroll
        for (int ks = 0; ks < kSteps; ++ks) {
            constexpr int kSkip = 16 * kGroups;   // bytes of a row that a step's (of nibbles, two steps') read takes
            if (ks % (kSteps / kWReads) == 0)
#pragma unroll
                for (int cb = 0; cb < BC; ++cb)
                    wf[ks * kWReads / kSteps][cb] = *(const v4i*)(mine + (w_off0 ^ (ks * kWReads / kSteps * kSkip)) + cb * BLK * (kLine / kWDiv));
            const int at = W_BITS == 8 ? ks * kSkip : ks / 2 * 2 * kSkip + (ks % 2 << 4);
#pragma unroll
            for (int tb = 0; tb < BT; ++tb) xf[ks][tb] = *(const v4i*)(mine + (x_off0 ^ at) + tb * BLK * kLine);
        }
        if (line + KW < nl) {   // (the operands are in registers: the space is free)
            asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
            issue(line + KW);
        }
#pragma unroll
        for (int ks = 0; ks < kSteps; ++ks)
#pragma unroll
            for (int cb = 0; cb < BC; ++cb) {
                v4i wv;
                if constexpr (W_BITS == 8) wv = wf[ks][cb];
                else wv = widen_nibbles(ks % 2 ? v2i{wf[ks / 2][cb][2], wf[ks / 2][cb][3]} : v2i{wf[ks / 2][cb][0], wf[ks / 2][cb][1]});
#pragma unroll
                for (int tb = 0; tb < BT; ++tb)
                    acc[cb][tb] = split_block(wv, xf[ks][tb], acc[cb][tb]);
            }
    }

    // ---- the sums, through LDS, to rows of the output ------------------------------------------------
    // Every wavefront leaves its sums where its lines were, as a row-major int32 tile, 16-byte chunks
    // (four channels) XOR-ed by the row; a thread adds up eight consecutive channels of a token,
    // dequantizes and writes 16 bytes.
    constexpr int kXor = (S::kC / 4) % 16 == 0 ? 15 : (S::kC / 4) % 8 == 0 ? 7 : 3;   // (chunks stay in their row)
    constexpr int kRow = S::kC * 4;
    if (wave < nl) {
        int8_t* const row = mine + fr_row * kRow;
#pragma unroll
        for (int cb = 0; cb < BC; ++cb)
#pragma unroll
            for (int tb = 0; tb < BT; ++tb)
#pragma unroll
                for (int j = 0; j < BLK * BLK / 256; ++j) {   // register 4j + i is channel 8j + 4 group + i of the block (of 16: j = 0)
                    const int chunk = cb * (BLK / 4) + 2 * j + group;
                    *(v4i*)(row + tb * BLK * kRow + ((chunk ^ (lane & kXor)) << 4)) =
                        v4i{acc[cb][tb][4 * j], acc[cb][tb][4 * j + 1], acc[cb][tb][4 * j + 2], acc[cb][tb][4 * j + 3]};
                }
    }
    wait_lds_and_barrier();
    if (c0 >= rows_w) return;
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const int t = t0 + i * kRowStep;
        if (t >= rows_x) return;
        v4i v0 = {0, 0, 0, 0}, v1 = v0;
#pragma unroll
        for (int g = 0; g < KW; ++g) {
            if (g >= nl) break;   // (uniform)
            const int8_t* sums = lds + g * kSlot + t * kRow;
            v0 += *(const v4i*)(sums + (((c0 >> 2) ^ (t & kXor)) << 4));
            v1 += *(const v4i*)(sums + ((((c0 >> 2) + 1) ^ (t & kXor)) << 4));
        }
        const long at = (long)(tok0 + t) * N + ch0 + c0;
        write_eight<W_BITS>(v0, v1, xsc[i], s0, s1, bias8, rows_w - c0, a.y + at, a.acc_out ? a.acc_out + at : nullptr);
    }
}

template <class S, int W_BITS>
hipError_t launch_split_tile(TileArgs a, hipStream_t stream) {
    if (!tile_grid(a.grid, a.M, a.N, S::kT, S::kC, S::kThreads)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(a.grid.tiles_per_xcd * kTileXcds)), block(S::kThreads);
    return enqueue(a.K % kLine ? gemm_i8_dequant_split<S, W_BITS, true> : gemm_i8_dequant_split<S, W_BITS, false>, grid, block,
                   stream, a);
}

}  // namespace
}  // namespace vq
