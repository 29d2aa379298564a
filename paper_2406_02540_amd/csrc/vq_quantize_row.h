// The register-resident token row of the quantizers: how a wavefront holds a token,
// and the steps from the fp32 row to int8 codes and the token's scale (ViDiT-Q Sec. 4.1,
// Sec. 3.1 Eq. 2 in symmetric form, activation side of Sec. 4.2 Eq. 3).  Shared by the
// quantizers of activations and of weights.
//
// LANES (64, 32 or 16) lanes of a wavefront share a token, so a wavefront holds
// 64 / LANES tokens.  Lane s of a token owns its 16-byte chunks s, s + LANES, ...
// (8 fp16 each): every load instruction of the wave covers contiguous pieces of
// 16 * LANES bytes and every store half of that.  NCH = chunks per lane.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "vq_lanes.h"

namespace vq {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef int int2v __attribute__((ext_vector_type(2)));

constexpr int kWave = 64;
constexpr int kQuantThreads = 256;
constexpr int kRowsPerBlock = kQuantThreads / kWave;

// Rounds to the nearest integer (halves to even), clamps to [-qmax, qmax].
__device__ __forceinline__ int quantize_one(float t, float inv, float qmax) {
    float q = __builtin_rintf(t * inv);
    q = fminf(fmaxf(q, -qmax), qmax);
    return (int)q;
}

__device__ __forceinline__ int pack4(int a, int b, int c, int d) {
    return (a & 0xFF) | ((b & 0xFF) << 8) | ((c & 0xFF) << 16) | (d << 24);
}

// The same for activations (qmax 127), four codes into the bytes of one register.  The scaled value is
// clamped first (the bounds are integers, so the order does not matter; NaN gives -127 as above) and
// rounded by adding 1.5 * 2^23: the sum's unit in the last place is one, the addition rounds halves to
// even, and the low byte of the sum is the code.  Three vector instructions per code and three per four
// codes to gather the bytes (rint, convert, mask and shift are five and a half): with the vector unit
// as busy as memory in these kernels, 3-4 % of the plain quantizer (32768 x 1152: 21.5 -> 20.7 us).
__device__ __forceinline__ unsigned code_bits(float t, float inv) {
    const float q = fminf(fmaxf(t * inv, -127.0f), 127.0f);
    return __builtin_bit_cast(unsigned, q + 12582912.0f);
}
__device__ __forceinline__ int quantize4(float t0, float t1, float t2, float t3, float inv) {
    const unsigned lo = __builtin_amdgcn_perm(code_bits(t1, inv), code_bits(t0, inv), 0x0C0C0400u);
    const unsigned hi = __builtin_amdgcn_perm(code_bits(t3, inv), code_bits(t2, inv), 0x04000C0Cu);
    return (int)(lo | hi);
}

// Sum (or maximum) over the LANES lanes of a token; every lane gets the result.
// Data moves between lanes without LDS round trips where the hardware allows it: DPP quad
// permutes (lane ^ 1, lane ^ 2), then the mirrored lane of the other half of 8 and of 16
// lanes (by then both halves are uniform, so any lane of the other half will do), and the swaps of
// rows of 16 and of halves of 32 lanes between two registers: with the same value in both, one ends up
// with the lower row's (half's) everywhere and the other with the upper one's.  (Through LDS, a swizzle and
// a permute, the last two steps took 100 to 130 cycles each, on the way of every token.)
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
// op(lower, upper) of the two rows of 16 (halves of 32) lanes, in every lane of both.
template <int ROW, class Op>
__device__ __forceinline__ float op_swapped(float v, Op op) {
    unsigned a = __builtin_bit_cast(unsigned, v), b = a;
    asm("" : "+v"(b));   // (a second register for the compiler: of one value in both it returns one result)
    const auto r = ROW == 16 ? __builtin_amdgcn_permlane16_swap(a, b, false, false) : __builtin_amdgcn_permlane32_swap(a, b, false, false);
    return op(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1]));
}
template <int LANES, class Op>
__device__ __forceinline__ float group_reduce(float v, Op op) {
    static_assert(LANES == 16 || LANES == 32 || LANES == 64, "lane groups are 16, 32 or 64 wide");
    v = op(v, dpp_move<0xB1>(v));   // quad_perm [1,0,3,2]
    v = op(v, dpp_move<0x4E>(v));   // quad_perm [2,3,0,1]
    v = op(v, dpp_move<0x141>(v));  // row_half_mirror
    v = op(v, dpp_move<0x140>(v));  // row_mirror
    if (LANES >= 32) v = op_swapped<16>(v, op);
    if (LANES >= 64) v = op_swapped<32>(v, op);
    return v;
}
template <int LANES>
__device__ __forceinline__ float group_sum(float v) {
    return group_reduce<LANES>(v, [](float a, float b) { return a + b; });
}
template <int LANES>
__device__ __forceinline__ float group_max(float v) {
    return group_reduce<LANES>(v, [](float a, float b) { return fmaxf(a, b); });
}

}  // namespace vq
