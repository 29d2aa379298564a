// The per-token quantizer fused behind the operation that produces its input
// (ViDiT-Q Sec. 5.1 "Hardware Implementation Settings": the quantization is integrated
// into the preceding LayerNorm, GELU and residual operations; Sec. 4.1 notes that the
// dynamic parameters only need the extrema of the token and can be fused with the
// previous operation).  The producer's output never goes to memory as fp16: a token is
// read once, transformed in registers as fp32, and its int8 codes and scale are written
// (the residual variant also writes the new fp16 residual stream, which the model needs).
//
// HBM-bound: 3 bytes per element (residual: 7; kPlain is the quantizer with nothing in front, 32768 x
// 1152 in 19.6 us, 5.8 TB/s), against the
// 7 (11) bytes of running the producer and the quantizer as two kernels.  The vector unit is a close
// second (12 to 18 instructions per element), so instructions count: without selects for chunks
// that are always inside the row or for a missing scale and shift, LayerNorm takes 17 per element
// instead of 24 (32768 x 1152: 30.9 -> 27.8 us).
//
// The textbook producers, the paper giving no formulas for them:
//   LayerNorm over the channels of a token (biased variance, eps inside the root, no
//   learned affine) followed by the DiT feature modulation (1 + scale[b]) y + shift[b]
//   of the token's sample b; GELU x Phi(x) exactly (erf) or in its tanh form;
//   r = x + gate[b] y.
//
// Compiled with -ffp-contract=off: every fp32 operation rounds on its own.
#pragma once
#include "vq_internal.h"
#include "vq_quantize_row.h"

namespace vq {


struct FusedArgs {
    const half8* x;          // [M,K8] the producer's input
    const half8* y;          // residual: the branch output added to x
    half8* r_out;            // residual: the sum, fp16
    const float4v* mod_a;    // LayerNorm: scale [B,K]; residual: gate [B,K]; or null
    const float4v* mod_b;    // LayerNorm: shift [B,K]; or null
    const float4v* chan_mul; // [K] or null
    int2v* xq;
    float* x_scale;
    int M, K8;
    int tokens_per_sample, n_samples;
    float eps;
};

inline FusedArgs fused_args(const ProducerArgs& p, int8_t* xq, float* x_scale, int M, int K) {
    FusedArgs a{};
    a.x = (const half8*)p.x;
    a.y = (const half8*)p.y;
    a.r_out = (half8*)p.r;
    a.mod_a = (const float4v*)p.mod_a;
    a.mod_b = (const float4v*)p.mod_b;
    a.chan_mul = (const float4v*)p.chan_mul;
    a.xq = (int2v*)xq;
    a.x_scale = x_scale;
    a.M = M;
    a.K8 = K / 8;
    a.tokens_per_sample = p.tokens_per_sample;
    a.n_samples = (int)((M + (long)p.tokens_per_sample - 1) / p.tokens_per_sample);
    a.eps = p.eps;
    return a;
}

// The stand-alone quantizers are compiled in two translation units: each combination of producer, chunks and
// lanes is a kernel of its own, some in two or more ways to read their vectors.
hipError_t launch_producer_gelu(int producer, const FusedArgs& a, hipStream_t stream);   // vq_fused_gelu.hip: both GELU forms
hipError_t launch_producer_other(int producer, const FusedArgs& a, hipStream_t stream);  // vq_fused.hip

namespace {


__device__ __forceinline__ float gelu_erf(float x) {
    return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f));
}

// x Phi(x) with Phi(x) ~ (1 + tanh(u)) / 2 = 1 / (1 + exp(-2u)), u = sqrt(2/pi) (x + 0.044715 x^3).
// exp(-2u) = exp2(x (c1 + c2 x^2)) with log2(e) folded into c1 = -2 sqrt(2/pi) log2(e) and
// c2 = 0.044715 c1: one fma, two multiplies, v_exp_f32, v_rcp_f32 (1 ulp each).  exp2
// overflows to +inf for very negative x, where the product with the reciprocal 0 is the
// correct -0.
__device__ __forceinline__ float gelu_tanh(float x) {
    constexpr float c1 = -2.302208198f;   // -2 * 0.7978845608 * 1.4426950409
    constexpr float c2 = -0.1029432397f;  // 0.044715 * c1
    const float e = __builtin_amdgcn_exp2f(x * __builtin_fmaf(x * x, c2, c1));
    return x * __builtin_amdgcn_rcpf(1.0f + e);
}

// One stage of the Walsh-Hadamard transform across lanes, index bit MASK (1, 2, 4 or 8) of the lane: the
// lane with the bit clear gets a + b, the one with it set a - b (a = the clear lane's value).  Every lane
// computes own + s * other with s = -1 where the bit is set, one multiply-add that reads the other lane's
// register as it goes (DPP inside a row of 16: quad permutes for 1 and 2, a rotation by half the row for
// 8; 4 takes a half-row mirror, lane ^ 7, and a quad reversal); that is s times the value wanted, exactly, so
// the product of the s of all stages comes off at the end (hadamard_sign).  32768 x 1152 with the
// quantizer: 27.7 us with an xor and an add per element and stage and ds_swizzle for 4, 23.2 as it is;
// 64 x 1152 4.0 -> 3.0.  A register that a vector
// instruction wrote may be read through DPP two wait states later, which the compiler cannot see to
// inside inline assembly: each block waits first, and its instructions read only registers written before it.
template <int MASK, int NCH>
__device__ __forceinline__ void hadamard_lane_stage(float (&t)[NCH][8], int sub, int used = NCH) {
    const float s = (sub & MASK) ? -1.0f : 1.0f;
#define VQ_STAGE(CTRL)                                                                                               \
    asm("s_nop 1\n\t"                                                                                                \
        "v_fmac_f32_dpp %0, %0, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                                          \
        "v_fmac_f32_dpp %1, %1, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                                          \
        "v_fmac_f32_dpp %2, %2, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                                          \
        "v_fmac_f32_dpp %3, %3, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                                          \
        "v_fmac_f32_dpp %4, %4, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                                          \
        "v_fmac_f32_dpp %5, %5, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                                          \
        "v_fmac_f32_dpp %6, %6, %8 " CTRL " row_mask:0xf bank_mask:0xf\n\t"                                          \
        "v_fmac_f32_dpp %7, %7, %8 " CTRL " row_mask:0xf bank_mask:0xf"                                              \
        : "+v"(t[i][0]), "+v"(t[i][1]), "+v"(t[i][2]), "+v"(t[i][3]), "+v"(t[i][4]), "+v"(t[i][5]), "+v"(t[i][6]),   \
          "+v"(t[i][7])                                                                                              \
        : "v"(s))
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        if (i >= used) continue;   // (uniform; a constant where every chunk is used)
        if constexpr (MASK == 1) VQ_STAGE("quad_perm:[1,0,3,2]");
        else if constexpr (MASK == 2) VQ_STAGE("quad_perm:[2,3,0,1]");
        else if constexpr (MASK == 8) VQ_STAGE("row_ror:8");
        else {
            float m0, m1, m2, m3, m4, m5, m6, m7;
            asm("s_nop 1\n\t"
                "v_mov_b32_dpp %8, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
                "v_mov_b32_dpp %9, %1 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
                "v_mov_b32_dpp %10, %2 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
                "v_mov_b32_dpp %11, %3 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
                "v_mov_b32_dpp %12, %4 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
                "v_mov_b32_dpp %13, %5 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
                "v_mov_b32_dpp %14, %6 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
                "v_mov_b32_dpp %15, %7 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
                "v_fmac_f32_dpp %0, %8, %16 quad_perm:[3,2,1,0] row_mask:0xf bank_mask:0xf\n\t"
                "v_fmac_f32_dpp %1, %9, %16 quad_perm:[3,2,1,0] row_mask:0xf bank_mask:0xf\n\t"
                "v_fmac_f32_dpp %2, %10, %16 quad_perm:[3,2,1,0] row_mask:0xf bank_mask:0xf\n\t"
                "v_fmac_f32_dpp %3, %11, %16 quad_perm:[3,2,1,0] row_mask:0xf bank_mask:0xf\n\t"
                "v_fmac_f32_dpp %4, %12, %16 quad_perm:[3,2,1,0] row_mask:0xf bank_mask:0xf\n\t"
                "v_fmac_f32_dpp %5, %13, %16 quad_perm:[3,2,1,0] row_mask:0xf bank_mask:0xf\n\t"
                "v_fmac_f32_dpp %6, %14, %16 quad_perm:[3,2,1,0] row_mask:0xf bank_mask:0xf\n\t"
                "v_fmac_f32_dpp %7, %15, %16 quad_perm:[3,2,1,0] row_mask:0xf bank_mask:0xf"
                : "+v"(t[i][0]), "+v"(t[i][1]), "+v"(t[i][2]), "+v"(t[i][3]), "+v"(t[i][4]), "+v"(t[i][5]),
                  "+v"(t[i][6]), "+v"(t[i][7]), "=&v"(m0), "=&v"(m1), "=&v"(m2), "=&v"(m3), "=&v"(m4), "=&v"(m5),
                  "=&v"(m6), "=&v"(m7)
                : "v"(s));
        }
    }
#undef VQ_STAGE
}
// The sign that the four stages above leave on a lane's values.
__device__ __forceinline__ float hadamard_sign(int sub) { return (__builtin_popcount(sub & 15) & 1) ? -1.0f : 1.0f; }

constexpr float kHadamardScale = 0.08838834764831845f;  // 1 / sqrt(128)

// Stages of the Walsh-Hadamard transform inside a lane's chunks of 8 values: index bits FROM .. TO - 1.
template <int FROM, int TO, int NCH>
__device__ __forceinline__ void hadamard_register_stages(float (&t)[NCH][8], int used = NCH) {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        if (i >= used) continue;
#pragma unroll
        for (int bit = 1 << FROM; bit < 1 << TO; bit <<= 1)
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (!(j & bit)) {
                    const float lo = t[i][j], hi = t[i][j | bit];
                    t[i][j] = lo + hi;
                    t[i][j | bit] = lo - hi;
                }
    }
}

typedef unsigned int uint4v __attribute__((ext_vector_type(4)));
constexpr int kBufFlags = 0x00020000;          // raw buffer, 32-bit data format
constexpr int kPastEnd = 0x7FFFFFF0;           // a buffer offset behind every buffer: loads give zero, stores are dropped

// The per-channel vectors: the balancing factor, and LayerNorm's scale and shift or the residual's gate.
enum VectorSlot { kVecMul = 0, kVecA = 1, kVecB = 2 };
constexpr int vector_count(int producer) { return producer == kLayerNorm ? 3 : producer == kResidual ? 2 : 1; }
struct Vec8 { float4v lo, hi; };   // one chunk of a vector

// Read from memory, every lane its chunks: four bytes per element and vector through the load path, for
// each token again.
// BY_CHUNK: so is the residual's branch, in fewer registers, instead of up front with the token.
// SCALE, SHIFT: LayerNorm has them (or reads an empty buffer's zeros, which takes the load path as long).
template <bool BY_CHUNK = false, bool SCALE = true, bool SHIFT = true>
struct VectorsFromMemory {
    static constexpr bool kByChunk = BY_CHUNK, kScale = SCALE, kShift = SHIFT;
    __device__ __forceinline__ bool staged(int) const { return false; }
    __device__ __forceinline__ Vec8 chunk(int, int, int) const { return {}; }
    template <class Rs>
    __device__ __forceinline__ void ask(const Rs&, const Rs&, const Rs&, int) {}
    __device__ __forceinline__ void park(int) {}
};

// Read once per workgroup into LDS (the rows of one sample; a workgroup whose tokens belong to several
// takes scale, shift and gate from memory): asked for ahead of the tokens, so that one latency covers
// both, and a quarter to an eighth of the bytes through the load path, which at 4 to 12 bytes of
// vectors for 3 of data was as busy as memory.  Chunks are split in halves: 16 bytes per lane, no bank conflict.
// 32768 tokens with all their vectors, us, from memory / as it is: 1152 channels LayerNorm 35.1 / 26.7,
// Hadamard 29.6 / 24.3, balanced 22.2 / 20.0; 4608 channels LayerNorm 123.6 / 84.9, GELU 97.0 / 82.2,
// Hadamard 103.4 / 81.5, balanced 85.4 / 76.0.  1001 x 1152: balanced 4.5 / 3.1, LayerNorm 4.8 / 4.2.
template <int PRODUCER, int CHUNKS, int THREADS>
struct VectorsInLds {
    static constexpr bool kByChunk = false, kScale = true, kShift = true;
    static constexpr int kVecs = vector_count(PRODUCER), kFloat4 = 2 * CHUNKS;
    static constexpr int kPer = (kFloat4 + THREADS - 1) / THREADS;
    float4v* lds;        // [kVecs][2][CHUNKS]
    bool used[3];        // (uniform) the vector exists and is staged
    int row;             // the sample whose rows are staged
    float4v v[kVecs][kPer];
    __device__ __forceinline__ bool staged(int which) const { return which < kVecs && used[which]; }
    __device__ __forceinline__ Vec8 chunk(int which, int c, int) const {
        const float4v* p = lds + which * kFloat4 + c;
        return Vec8{p[0], p[CHUNKS]};
    }
    template <class Rs>
    __device__ __forceinline__ void ask(const Rs& rs_cm, const Rs& rs_a, const Rs& rs_b, int K8) {
#pragma unroll
        for (int w = 0; w < kVecs; ++w)
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                const int e = i * THREADS + (int)threadIdx.x;   // which 16 bytes of the row
                if (used[w])
                    v[w][i] = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(
                        w == kVecMul ? rs_cm : w == kVecA ? rs_a : rs_b, e < 2 * K8 ? ((w == kVecMul ? 0 : row * K8 * 2) + e) * 16 : kPastEnd,
                        0, 0));
            }
    }
    __device__ __forceinline__ void park(int K8) {
        bool any = false;
#pragma unroll
        for (int w = 0; w < kVecs; ++w) {
            any = any || used[w];
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                const int e = i * THREADS + (int)threadIdx.x;
                if (used[w] && e < kFloat4) lds[w * kFloat4 + (e & 1) * CHUNKS + (e >> 1)] = v[w][i];
            }
        }
        if (any) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory");
        __builtin_amdgcn_sched_barrier(0);   // (the tokens are not waited for ahead of the barrier)
    }
};

// A wavefront takes 64 / LANES tokens.  Everything it reads or writes goes through range-checked
// buffers: the rows through buffers that start at the wavefront's first token and end behind its
// last one, so that tokens past M and chunks past K (whose offset is pushed behind the buffer) read
// as zero and are never written, without a branch; the per-channel vectors (balancing factor,
// modulation scale and shift or gate) through buffers over the whole arrays, addressed by 32-bit
// offsets from a scalar base (a pointer per chunk and vector would cost two registers each).  A
// kernel without branches and with few registers keeps many wavefronts per SIMD resident, and that,
// not a loop over tokens with a prefetch, is what overlaps the producers' arithmetic with the memory
// time of other wavefronts' rows (the loop was built and measured: slower for every producer but one).
//
// Where the codes and scales go is `out`'s business: out.scale(token of the wavefront, value) by one lane
// per existing token, out.codes(token of the wavefront, chunk of the row, whether it exists, 8 codes).
// EXACT: NCH is the row's chunk count over LANES, rounded up; otherwise it is an upper bound, and chunk
// groups past the row are skipped (a wave-uniform branch each).  writes_r: this wavefront writes the
// residual sum (where several compute it, one does).
template <int PRODUCER, int NCH, int LANES, bool EXACT, class Vectors, class Out>
__device__ __forceinline__ void produce_and_quantize(const FusedArgs& a, long w_first, int lane, bool writes_r,
                                                     Vectors vectors, const Out& out) {
    constexpr int kTokensPerWave = kWave / LANES;
    const int sub = lane & (LANES - 1);
    const int K8 = a.K8;
    const long m = w_first + lane / LANES;
    const bool row_ok = m < a.M;

    const int ntok = (int)max(0l, min((long)kTokensPerWave, a.M - w_first));
    const __amdgpu_buffer_rsrc_t rs_x =
        __builtin_amdgcn_make_buffer_rsrc((void*)(a.x + w_first * K8), 0, ntok * K8 * 16, kBufFlags);
    const __amdgpu_buffer_rsrc_t rs_y = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(PRODUCER == kResidual ? a.y + w_first * K8 : a.x), 0, PRODUCER == kResidual ? ntok * K8 * 16 : 0, kBufFlags);
    const __amdgpu_buffer_rsrc_t rs_r = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(PRODUCER == kResidual ? a.r_out + w_first * K8 : (half8*)a.x), 0,
        PRODUCER == kResidual && writes_r ? ntok * K8 * 16 : 0, kBufFlags);
    const __amdgpu_buffer_rsrc_t rs_cm =
        __builtin_amdgcn_make_buffer_rsrc((void*)a.chan_mul, 0, a.chan_mul ? K8 * 32 : 0, kBufFlags);
    const __amdgpu_buffer_rsrc_t rs_a =
        __builtin_amdgcn_make_buffer_rsrc((void*)a.mod_a, 0, a.mod_a ? a.n_samples * K8 * 32 : 0, kBufFlags);
    const __amdgpu_buffer_rsrc_t rs_b =
        __builtin_amdgcn_make_buffer_rsrc((void*)a.mod_b, 0, a.mod_b ? a.n_samples * K8 * 32 : 0, kBufFlags);

    // (with EXACT only a lane's last chunk can lie past the row)
    auto chunk_in_row = [&](int i) { return (EXACT && i + 1 < NCH) || i * LANES + sub < K8; };
    const int used = EXACT ? NCH : (K8 + LANES - 1) / LANES;   // chunk groups of the row
    int voff[NCH];  // byte offset of this lane's chunk i in the fp16 rows (half of it in the int8 rows)
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int c = i * LANES + sub;
        voff[i] = (c < K8) ? ((lane / LANES) * K8 + c) * 16 : kPastEnd;
    }
    // The 8 floats of a per-channel vector that belong to chunk i of this lane, row `row` of a
    // [rows][K] array (chunks past K take the last chunk's: finite values that meet only zeros).
    auto vec_chunk = [&](int which, int row, int i) {
        const int c = min(i * LANES + sub, K8 - 1);
        if (vectors.staged(which)) return vectors.chunk(which, c, i);
        const __amdgpu_buffer_rsrc_t& rs = which == kVecMul ? rs_cm : which == kVecA ? rs_a : rs_b;
        const int off = (row * K8 + c) * 32;
        Vec8 v;
        v.lo = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
        v.hi = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16, 0, 0));
        return v;
    };
    // The vectors are asked for one chunk ahead of their use.  After every chunk a barrier for
    // memory accesses that also pins the chunk's results keeps the compiler from asking for the
    // vectors of all chunks first and doing the arithmetic afterwards (16 to 32 registers per chunk).
    auto chunk_done = [](float(&c)[8]) {
        asm volatile("" : "+v"(c[0]), "+v"(c[1]), "+v"(c[2]), "+v"(c[3]), "+v"(c[4]), "+v"(c[5]), "+v"(c[6]), "+v"(c[7])
                     :
                     : "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    // which sample's modulation this token takes
    const int b = (int)((unsigned)(row_ok ? m : a.M - 1) / (unsigned)a.tokens_per_sample);

    vectors.ask(rs_cm, rs_a, rs_b, K8);
    half8 raw[NCH];   // (chunk groups past the row are asked for too: a branch would hide from the waits what is behind it)
#pragma unroll
    for (int i = 0; i < NCH; ++i)
        raw[i] = __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(rs_x, voff[i], 0, 2 /* nontemporal */));
    constexpr bool kBranchFirst = PRODUCER == kResidual && !Vectors::kByChunk;   // the residual's branch with them
    auto branch_chunk = [&](int i) {
        return __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(rs_y, voff[i], 0, 2 /* nontemporal */));
    };
    half8 branch[kBranchFirst ? NCH : 1];
    if constexpr (kBranchFirst) {
#pragma unroll
        for (int i = 0; i < NCH; ++i)
            branch[i] = branch_chunk(i);
    }
    vectors.park(K8);   // (a workgroup barrier where the vectors are staged: every wavefront gets here)
    if (ntok == 0) return;
    float t[NCH][8];
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        if (i >= used) continue;
#pragma unroll
        for (int j = 0; j < 8; ++j) t[i][j] = (float)raw[i][j];
    }

    if (PRODUCER == kHadamard) {
        // Rotation-based balancing (Sec. 4.2): t = (x * chan_mul) Q with Q block diagonal,
        // blocks H_128 / sqrt(128).  A block is 16 consecutive chunks = the 16 lanes sub%16 of a
        // token with one chunk index i, so element 8 (sub%16) + j of the block sits in lane
        // sub, register t[i][j]: three butterfly stages inside the registers, four across lanes.
        if (a.chan_mul) {
            Vec8 nxt = vec_chunk(kVecMul, 0, 0);
#pragma unroll
            for (int i = 0; i < NCH; ++i) {
                if (i >= used) continue;
                const Vec8 cm = nxt;
                if (i + 1 < NCH) nxt = vec_chunk(kVecMul, 0, i + 1);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    t[i][j] = t[i][j] * cm.lo[j];
                    t[i][4 + j] = t[i][4 + j] * cm.hi[j];
                }
                chunk_done(t[i]);
            }
        }
        hadamard_register_stages<0, 3>(t, used);
        hadamard_lane_stage<1>(t, sub, used);
        hadamard_lane_stage<2>(t, sub, used);
        hadamard_lane_stage<4>(t, sub, used);
        hadamard_lane_stage<8>(t, sub, used);
        const float signed_scale = hadamard_sign(sub) * kHadamardScale;
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            if (i >= used) continue;
#pragma unroll
            for (int j = 0; j < 8; ++j) t[i][j] = t[i][j] * signed_scale;
        }
    }

    if (PRODUCER == kGeluErf || PRODUCER == kGeluTanh) {
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            if (i >= used) continue;
#pragma unroll
            for (int j = 0; j < 8; ++j) t[i][j] = (PRODUCER == kGeluErf) ? gelu_erf(t[i][j]) : gelu_tanh(t[i][j]);
            // one chunk at a time: interleaving all of them would need a register per
            // temporary of every element
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    if (PRODUCER == kLayerNorm) {
        // two passes over the registers: the mean, then the variance about it
        float s = 0.0f;
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            if (i >= used) continue;
#pragma unroll
            for (int j = 0; j < 8; ++j) s = s + t[i][j];  // (chunks past the row hold zeros)
        }
        const float mean = group_sum<LANES>(s) / (float)(8 * K8);
        float ss = 0.0f;
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            if (i >= used) continue;
            const bool in_row = chunk_in_row(i);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                t[i][j] = in_row ? t[i][j] - mean : 0.0f;
                ss = __builtin_fmaf(t[i][j], t[i][j], ss);
            }
        }
        const float var = group_sum<LANES>(ss) / (float)(8 * K8);
        const float rstd = 1.0f / __builtin_sqrtf(var + a.eps);
        // t = (x - mean) rstd (1 + scale) + shift as one multiply and one fma per element (a missing scale
        // or shift is an empty buffer, which reads as zero)
        if constexpr (Vectors::kScale && Vectors::kShift) {
            Vec8 nxt_a = vec_chunk(kVecA, b, 0), nxt_b = vec_chunk(kVecB, b, 0);
#pragma unroll
            for (int i = 0; i < NCH; ++i) {
                if (i >= used) continue;
                const Vec8 sc = nxt_a, sh = nxt_b;
                if (i + 1 < NCH) nxt_a = vec_chunk(kVecA, b, i + 1), nxt_b = vec_chunk(kVecB, b, i + 1);
                float mul[8], add[8];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    mul[j] = rstd * (1.0f + sc.lo[j]);
                    mul[4 + j] = rstd * (1.0f + sc.hi[j]);
                    add[j] = sh.lo[j];
                    add[4 + j] = sh.hi[j];
                }
#pragma unroll
                for (int j = 0; j < 8; ++j) t[i][j] = __builtin_fmaf(t[i][j], mul[j], add[j]);
                chunk_done(t[i]);
            }
        } else {
            constexpr int kGiven = Vectors::kScale ? kVecA : kVecB;
            Vec8 nxt{};
            if constexpr (Vectors::kScale || Vectors::kShift) nxt = vec_chunk(kGiven, b, 0);
#pragma unroll
            for (int i = 0; i < NCH; ++i) {
                if (i >= used) continue;
                const Vec8 v = nxt;
                if constexpr (Vectors::kScale || Vectors::kShift)
                    if (i + 1 < NCH) nxt = vec_chunk(kGiven, b, i + 1);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float e = j < 4 ? v.lo[j & 3] : v.hi[j & 3];
                    if constexpr (Vectors::kScale) t[i][j] = t[i][j] * (rstd * (1.0f + e));
                    else if constexpr (Vectors::kShift) t[i][j] = __builtin_fmaf(t[i][j], rstd, e);
                    else t[i][j] = t[i][j] * rstd;
                }
                if constexpr (Vectors::kScale || Vectors::kShift) chunk_done(t[i]);
            }
        }
    }

    if constexpr (PRODUCER == kResidual) {
        Vec8 nxt{};
        if (a.mod_a) nxt = vec_chunk(kVecA, b, 0);
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            if (i >= used) continue;
            const Vec8 gate = nxt;
            if (a.mod_a && i + 1 < NCH) nxt = vec_chunk(kVecA, b, i + 1);
            half8 yv;
            if constexpr (kBranchFirst) yv = branch[i];
            else yv = branch_chunk(i);
            float p[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) p[j] = (float)yv[j];
            if (a.mod_a) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    p[j] = gate.lo[j] * p[j];
                    p[4 + j] = gate.hi[j] * p[4 + j];
                }
            }
            half8 r;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                float sum = t[i][j] + p[j];
                asm("" : "+v"(sum));     // (the fp32 sum is rounded before it is narrowed)
                r[j] = (_Float16)sum;    // the new residual stream is fp16 ...
                t[i][j] = (float)r[j];   // ... and that is what the next layer quantizes
            }
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uint4v, r), rs_r, voff[i], 0, 0);
        }
    }

    // ---- the quantizer: balancing factor, absmax of the token, its scale, int8 codes ----
    // (two IEEE divisions per token, none per element)
    float amax = 0.0f;
    const bool fold = PRODUCER != kHadamard && a.chan_mul;  // (the rotation has the scaling before itself)
    Vec8 nxt_cm{};
    if (fold) nxt_cm = vec_chunk(kVecMul, 0, 0);
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        if (i >= used) continue;
        if (fold) {
            const Vec8 cm = nxt_cm;
            if (i + 1 < NCH) nxt_cm = vec_chunk(kVecMul, 0, i + 1);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                t[i][j] = t[i][j] * cm.lo[j];
                t[i][4 + j] = t[i][4 + j] * cm.hi[j];
            }
        }
        const bool in_row = chunk_in_row(i);
#pragma unroll
        for (int j = 0; j < 8; ++j) amax = fmaxf(amax, in_row ? fabsf(t[i][j]) : 0.0f);
        if (fold) {
            asm volatile("" : : : "memory");
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    amax = group_max<LANES>(amax);
    float scale = 0.0f, inv = 0.0f;
    if (amax != 0.0f) {
        scale = amax / 127.0f;
        inv = 127.0f / amax;
    }
    if (row_ok && sub == 0) out.scale(lane / LANES, scale);
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        if (i >= used) continue;
        int2v o;
        o.x = quantize4(t[i][0], t[i][1], t[i][2], t[i][3], inv);
        o.y = quantize4(t[i][4], t[i][5], t[i][6], t[i][7], inv);
        out.codes(lane / LANES, i * LANES + sub, voff[i] != kPastEnd, o);
    }
}

// The stand-alone kernels: codes and scales go to memory.
struct RowsInMemory {
    __amdgpu_buffer_rsrc_t rs_q;   // the wavefront's rows of codes
    float* x_scale;                // and its first token's scale
    int K8;
    __device__ __forceinline__ void scale(int token, float s) const { x_scale[token] = s; }
    __device__ __forceinline__ void codes(int token, int chunk, bool exists, int2v o) const {
        __builtin_amdgcn_raw_buffer_store_b64(o, rs_q, exists ? (token * K8 + chunk) * 8 : kPastEnd, 0, 0);
    }
};

// Which kernels stage their vectors, and with how many threads: workgroups of four wavefronts share up to
// 20 KiB (eight of them fit a CU's LDS); LayerNorm's up to 56 KiB are shared by eight (two workgroups, four
// wavefronts per SIMD), and only from kManyTokens on: with fewer there is nothing to wait for but the staging
// itself.  LayerNorm of short rows, and longer rows of all, read them from memory.  The residual's long rows
// (two fp16 tokens of more than 5 chunks per lane) take the branch chunk by chunk from kManyTokens on, where
// the registers of asking first cost a wavefront per SIMD (32768 x 4608: 191 us, 197 asked first; 1000 x
// 4608 11.8 and 9.1).
constexpr int kFewVectorBytes = 20 * 1024, kManyVectorBytes = 56 * 1024, kManyTokens = 4096;
constexpr int vector_bytes(int producer, int nch, int lanes) { return vector_count(producer) * nch * lanes * 32; }
enum Staging { kNotStaged, kStaged, kStagedWide, kByChunk, kNoScale, kNoShift, kNeither };
constexpr Staging staging(int producer, int nch, int lanes) {   // (from kManyTokens on; below, the last two are kNotStaged)
    const int bytes = vector_bytes(producer, nch, lanes);
    if (producer == kLayerNorm && nch <= 2) return kNotStaged;
    if (bytes <= kFewVectorBytes) return kStaged;
    if (producer == kResidual) return kByChunk;
    return producer == kLayerNorm && bytes <= kManyVectorBytes ? kStagedWide : kNotStaged;
}
constexpr int fused_threads(Staging s) { return s == kStagedWide ? 512 : kQuantThreads; }

// (LayerNorm of up to five chunks per lane: held to the 96 registers that five wavefronts per SIMD have)
template <int PRODUCER, int NCH, int LANES, Staging STAGING>
__global__ __launch_bounds__(fused_threads(STAGING), PRODUCER == kLayerNorm && NCH <= 5 ? 5 : 1) void produce_quantize_tokens(
    const FusedArgs a) {
    constexpr int kTokensPerWave = kWave / LANES;
    constexpr int kThreads = fused_threads(STAGING), kRows = kThreads / kWave * kTokensPerWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // (uniform: the buffer descriptors are scalar)
    const long first = (long)blockIdx.x * kRows;
    const long w_first = first + wave * kTokensPerWave;  // first token of this wavefront
    const int ntok = (int)max(0l, min((long)kTokensPerWave, a.M - w_first));
    const RowsInMemory out{__builtin_amdgcn_make_buffer_rsrc((void*)(a.xq + w_first * a.K8), 0, ntok * a.K8 * 8, kBufFlags),
                           a.x_scale + w_first, a.K8};
    const int lane = threadIdx.x & (kWave - 1);
    if constexpr (STAGING == kStaged || STAGING == kStagedWide) {
        typedef VectorsInLds<PRODUCER, NCH * LANES, kThreads> Staged;
        __shared__ float4v lds[Staged::kVecs * Staged::kFloat4];
        Staged vectors;
        vectors.lds = lds;
        const int s_first = (int)((unsigned)first / (unsigned)a.tokens_per_sample);
        const int s_last = (int)((unsigned)min(first + kRows - 1, (long)a.M - 1) / (unsigned)a.tokens_per_sample);
        vectors.row = s_first;
        // (the residual's gate alone is not worth a barrier; LayerNorm reads a missing scale or shift as zeros,
        // from LDS or memory alike)
        const bool sample = s_first == s_last && (PRODUCER == kLayerNorm || (a.chan_mul && a.mod_a));
        vectors.used[kVecMul] = a.chan_mul != nullptr;
        vectors.used[kVecA] = vectors.used[kVecB] = sample;
        produce_and_quantize<PRODUCER, NCH, LANES, true>(a, w_first, lane, true, vectors, out);
    } else {
        typedef VectorsFromMemory<STAGING == kByChunk, STAGING != kNoScale && STAGING != kNeither,
                                  STAGING != kNoShift && STAGING != kNeither> FromMemory;
        produce_and_quantize<PRODUCER, NCH, LANES, true>(a, w_first, lane, true, FromMemory{}, out);
    }
}

template <int PRODUCER, int NCH, int LANES, Staging STAGING>
hipError_t launch_fused_staging(const FusedArgs& a, hipStream_t stream) {
    constexpr int threads = fused_threads(STAGING), rows_per_block = threads / LANES;
    const dim3 grid((unsigned)((a.M + (long)rows_per_block - 1) / rows_per_block)), block(threads);
    return enqueue(produce_quantize_tokens<PRODUCER, NCH, LANES, STAGING>, grid, block, stream, a);
}
template <int PRODUCER, int NCH, int LANES>
hipError_t launch_fused(const FusedArgs& a, hipStream_t stream) {
    constexpr Staging kind = staging(PRODUCER, NCH, LANES);
    if constexpr (kind == kStagedWide || kind == kByChunk)
        if (a.M < kManyTokens) return launch_fused_staging<PRODUCER, NCH, LANES, kNotStaged>(a, stream);
    if constexpr (PRODUCER == kLayerNorm && kind == kNotStaged && NCH > 2) {
        // Rows too long to stage, many of them: a missing scale or shift is not asked for (us, asked for / as it
        // is, 20000 x 6144: neither given 85.1 / 66.1, shift only 103.5 / 92.5, scale only 86.4 / 76.1; with few
        // tokens there is nothing to gain, and a run-time branch around each load cost the kernel that has both 10
        // to 20 %).
        if (a.M >= kManyTokens && !a.mod_a && !a.mod_b) return launch_fused_staging<PRODUCER, NCH, LANES, kNeither>(a, stream);
        if (a.M >= kManyTokens && !a.mod_a) return launch_fused_staging<PRODUCER, NCH, LANES, kNoScale>(a, stream);
        if (a.M >= kManyTokens && !a.mod_b) return launch_fused_staging<PRODUCER, NCH, LANES, kNoShift>(a, stream);
    }
    return launch_fused_staging<PRODUCER, NCH, LANES, kind>(a, stream);
}

// NCH is a template parameter: pick the instantiation for the run-time chunk count.
template <int PRODUCER, int LANES, int NCH = 1>
hipError_t launch_fused_nch(int nch, const FusedArgs& a, hipStream_t stream) {
    if constexpr (NCH > 16) {
        return hipErrorInvalidValue;
    } else {
        if (nch == NCH) return launch_fused<PRODUCER, NCH, LANES>(a, stream);
        return launch_fused_nch<PRODUCER, LANES, NCH + 1>(nch, a, stream);
    }
}

template <int PRODUCER>
hipError_t launch_producer(const FusedArgs& a, hipStream_t stream) {
    const int k8 = a.K8;
    // (many short plain rows: four tokens to a wavefront, 32768 x 512 11.8 -> 10.0 us; few: 1001 x 512 2.1, 2.25 so)
    switch (PRODUCER == kPlain && k8 <= 64 && a.M >= kManyTokens ? 16 : lanes_for_row(k8)) {
        case 16: return launch_fused_nch<PRODUCER, 16>((k8 + 15) / 16, a, stream);
        case 32: return launch_fused_nch<PRODUCER, 32>((k8 + 31) / 32, a, stream);
        default: return launch_fused_nch<PRODUCER, 64>((k8 + 63) / 64, a, stream);
    }
}

}  // namespace
}  // namespace vq
