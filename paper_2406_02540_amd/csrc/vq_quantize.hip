// Quantizers for gfx950.
//
// 1. Dynamic per-token activation quantizer (ViDiT-Q Sec. 4.1; Eq. 2 of Sec. 3.1
//    in symmetric form; activation side of the channel balancing, Eq. 3 of
//    Sec. 4.2) for rows of any length and alignment; rows of whole 16-byte chunks go to the
//    kernel that holds them in registers (vq_fused_kernel.h with nothing in front).
// 2. Offline per-output-channel weight quantizer (same recipe, qmax 127 or 7,
//    weight side of Eq. 3), with the 4-bit packer fused.
//
// This file is compiled with -ffp-contract=off: every fp32 operation rounds on
// its own, the two divisions per row are the correctly rounded IEEE ones, and
// rounding to integer is v_rndne_f32 (halves to even).
#include "vq_internal.h"
#include "vq_quantize_row.h"

namespace vq {
namespace {

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, kWave));
    return v;
}

__device__ __forceinline__ float block_max(float v, float* red) {
    v = wave_max(v);
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x >> 6;
    if (lane == 0) red[w] = v;
    __syncthreads();
    float r = red[0];
#pragma unroll
    for (int i = 1; i < kRowsPerBlock; ++i) r = fmaxf(r, red[i]);
    __syncthreads();
    return r;
}

// Any K, any alignment: one workgroup per token, two passes over the row
// (the second one hits in cache).  Used when K is not a multiple of 8 or the
// row does not fit the register-resident kernel.
template <bool HAS_MUL>
__global__ __launch_bounds__(kQuantThreads) void quantize_tokens_generic(
    const _Float16* __restrict__ x, const float* __restrict__ chan_mul, int8_t* __restrict__ xq,
    float* __restrict__ x_scale, int K) {
    __shared__ float red[kRowsPerBlock];
    const long m = blockIdx.x;
    const _Float16* row = x + m * (long)K;
    float amax = 0.0f;
    for (int k = threadIdx.x; k < K; k += kQuantThreads) {
        float t = (float)row[k];
        if (HAS_MUL) t = t * chan_mul[k];
        amax = fmaxf(amax, fabsf(t));
    }
    amax = block_max(amax, red);
    float scale = 0.0f, inv = 0.0f;
    if (amax != 0.0f) {
        scale = amax / 127.0f;
        inv = 127.0f / amax;
    }
    if (threadIdx.x == 0) x_scale[m] = scale;
    int8_t* qrow = xq + m * (long)K;
    for (int k = threadIdx.x; k < K; k += kQuantThreads) {
        float t = (float)row[k];
        if (HAS_MUL) t = t * chan_mul[k];
        qrow[k] = (int8_t)quantize_one(t, inv, 127.0f);
    }
}

// Static quantizer (the comparison point: one scale for the whole tensor, fixed beforehand).
// Rows of whole 16-byte chunks: a wavefront takes CHUNKS KiB of contiguous input, a thread
// its chunks one wavefront width apart (every load and store instruction of a wavefront is
// contiguous), all loads first: a thread's chunks are four registers each and the eight wavefronts per SIMD
// leave 64, so with chan_mul nine chunks are the most that fit.  (Ten spilled 16 registers: 40000 x 2048 with
// chan_mul 58.4 us, 46.0 as it is; 10000 x 4096 35.7 and 26.3.  Stepping the chunk of the row instead of one
// division per chunk: 8192 x 1152 9.0 and 8.1.)
template <bool HAS_MUL, int CHUNKS>
__global__ __launch_bounds__(kQuantThreads, 8) void quantize_static_chunks(
    const half8* __restrict__ x, const float4v* __restrict__ chan_mul, float inv, int2v* __restrict__ xq,
    unsigned chunks, unsigned K8) {
    const unsigned base = blockIdx.x * (kQuantThreads * CHUNKS) + (threadIdx.x >> 6) * (kWave * CHUNKS) +
                          (threadIdx.x & (kWave - 1));
    half8 v[CHUNKS];
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
        const unsigned c = base + i * kWave;
        if (c < chunks) v[i] = __builtin_nontemporal_load(x + c);
    }
    int2v o[CHUNKS];
    unsigned k8 = HAS_MUL ? base % K8 : 0u;   // chunk of its row, stepped by a wavefront's width
    const unsigned step = HAS_MUL ? kWave % K8 : 0u;
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
        const unsigned c = base + i * kWave;
        if (c < chunks) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {   // (four values and factors at a time: fewer registers)
                float t[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) t[j] = (float)v[i][4 * h + j];
                if (HAS_MUL) {
                    const float4v m = chan_mul[2 * k8 + h];
#pragma unroll
                    for (int j = 0; j < 4; ++j) t[j] = t[j] * m[j];
                }
                int q = quantize4(t[0], t[1], t[2], t[3], inv);
                if (HAS_MUL) asm volatile("" : "+v"(q) : : "memory");
                o[i][h] = q;
            }
        }
        if (HAS_MUL) {
            k8 += step;
            if (k8 >= K8) k8 -= K8;
        }
    }
    // the stores leave together, behind the last load (reads and writes in bursts, not mixed)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
        const unsigned c = base + i * kWave;
        if (c < chunks) xq[c] = o[i];
    }
}

// Any K: element by element.
__global__ __launch_bounds__(kQuantThreads) void quantize_static_elems(
    const _Float16* __restrict__ x, const float* __restrict__ chan_mul, float inv, int8_t* __restrict__ xq,
    long total, int K) {
    const long step = (long)gridDim.x * kQuantThreads;
    for (long e = (long)blockIdx.x * kQuantThreads + threadIdx.x; e < total; e += step) {
        float t = (float)x[e];
        if (chan_mul) t = t * chan_mul[e % K];
        xq[e] = (int8_t)quantize_one(t, inv, 127.0f);
    }
}

// Calibration side of Eq. 3 (Sec. 4.2): per-input-channel absmax over the rows of a matrix
// (tokens of a calibration batch, or output channels of a weight).  Slabs of rows are combined
// with an integer atomic max on the bit pattern (non-negative floats order like their bits).
// amax must hold valid non-negative values on entry (zeros, or the running maximum of earlier
// batches).
//
// Memory-bound: every element is read once and nothing is written but the maxima.  A workgroup
// takes 16 chunks of 16 bytes (two cache lines of a row) x a slab of rows, a thread one chunk of
// every 32nd row with kAbsmaxUnroll loads in flight, and the 32 maxima of a channel meet in LDS, so
// that one atomic per channel and slab leaves the workgroup.  The slab is a range-checked buffer:
// rows behind it and chunks past K read as zero, which no maximum notices.
// 32768 x 1152 fp16: 12.2-14.6 us (5.2-6.2 TB/s), 4608 x 1152 fp32: 4.5-5.9 us; with one column per
// thread, 2 or 4 bytes per load and each load waited for: 48.8 and 27.3 us.
constexpr int kAbsmaxThreads = 512, kAbsmaxCols = 16, kAbsmaxRows = kAbsmaxThreads / kAbsmaxCols, kAbsmaxUnroll = 4;
constexpr int kAbsmaxOneSlab = 256;   // so few rows that a slab of their own costs less than clearing amax first (a launch, 2 us)
constexpr int kAbsmaxFewRows = 4;
template <typename T>
struct AbsmaxChunk { typedef half8 type; };
template <>
struct AbsmaxChunk<float> { typedef float4v type; };

template <typename T>
__global__ __launch_bounds__(kAbsmaxThreads, 8) void channel_absmax_chunks(const T* __restrict__ a,
                                                                           float* __restrict__ amax, int R, int K,
                                                                           int rows_per_block, int overwrite) {
    typedef typename AbsmaxChunk<T>::type chunk_t;
    constexpr int kElems = 16 / sizeof(T);
    __shared__ chunk_t red[kAbsmaxRows][kAbsmaxCols];
    const int col = threadIdx.x % kAbsmaxCols, row = threadIdx.x / kAbsmaxCols;
    const int c = blockIdx.x * kAbsmaxCols + col;   // chunk of the row
    const long r0 = (long)blockIdx.y * rows_per_block;
    const int rows = (int)(R - r0 < rows_per_block ? R - r0 : rows_per_block);
    const int row_bytes = K * (int)sizeof(T);
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void*)(a + r0 * K), 0, rows * row_bytes, 0x00020000);
    const bool in_k = c * kElems < K;
    chunk_t m{};
    for (int r = row; r < rows; r += kAbsmaxUnroll * kAbsmaxRows) {
        chunk_t v[kAbsmaxUnroll];
#pragma unroll
        for (int u = 0; u < kAbsmaxUnroll; ++u) {
            const unsigned off = (unsigned)(r + u * kAbsmaxRows) * (unsigned)row_bytes + (unsigned)c * 16u;
            v[u] = __builtin_bit_cast(chunk_t, __builtin_amdgcn_raw_buffer_load_b128(rs, in_k ? off : 0xFFFFFFF0u, 0,
                                                                                     2 /* nontemporal */));
        }
#pragma unroll
        for (int u = 0; u < kAbsmaxUnroll; ++u) m = __builtin_elementwise_max(m, __builtin_elementwise_abs(v[u]));
    }
    red[row][col] = m;
    __syncthreads();
    const int e = threadIdx.x;   // channel of the workgroup's chunks
    const long k = (long)blockIdx.x * kAbsmaxCols * kElems + e;
    if (e >= kAbsmaxCols * kElems || k >= K) return;
    T best = (T)0.0f;
#pragma unroll
    for (int i = 0; i < kAbsmaxRows; ++i) best = __builtin_elementwise_max(best, red[i][e / kElems][e % kElems]);
    if (overwrite) amax[k] = (float)best;   // (one slab: nothing to combine with)
    else atomicMax((int*)amax + k, __builtin_bit_cast(int, (float)best));
}

// The same for rows that are not whole 16-byte chunks (K % 8 in fp16, K % 4 in fp32), and for a few rows
// more: thread t of a block owns column 256 b_x + t for a slab of rows.
template <typename T>
__global__ __launch_bounds__(kQuantThreads) void channel_absmax_cols(const T* __restrict__ a,
                                                                     float* __restrict__ amax, int R, int K,
                                                                     int rows_per_block) {
    const int k = blockIdx.x * kQuantThreads + threadIdx.x;
    if (k >= K) return;
    const long r0 = (long)blockIdx.y * rows_per_block;
    const long r1 = r0 + rows_per_block < R ? r0 + rows_per_block : R;
    float m = 0.0f;
    for (long r = r0; r < r1; ++r) m = fmaxf(m, fabsf((float)a[r * K + k]));
    atomicMax((int*)amax + k, __builtin_bit_cast(int, m));
}

__global__ __launch_bounds__(kQuantThreads) void fill_zero_f32(float* __restrict__ p, int n) {
    const int i = blockIdx.x * kQuantThreads + threadIdx.x;
    if (i < n) p[i] = 0.0f;
}

// s = max|X|^alpha / max|W|^(1 - alpha) per channel, statistics raised to 1e-5, s kept in
// [1e-5, 1e5]; chan_mul = 1 / s (IEEE division).
__global__ __launch_bounds__(kQuantThreads) void balance_mask_elems(const float* __restrict__ ax,
                                                                    const float* __restrict__ aw, float alpha,
                                                                    float* __restrict__ s_out,
                                                                    float* __restrict__ chan_mul, int K) {
    const int k = blockIdx.x * kQuantThreads + threadIdx.x;
    if (k >= K) return;
    const float x = fmaxf(ax[k], 1e-5f), w = fmaxf(aw[k], 1e-5f);
    float s = powf(x, alpha) / powf(w, 1.0f - alpha);
    s = fminf(fmaxf(s, 1e-5f), 1e5f);
    s_out[k] = s;
    chan_mul[k] = 1.0f / s;
}

// Offline weight quantizer, rows of whole 16-byte chunks that a wavefront holds in registers: one
// output channel per wavefront, a lane the chunks lane, lane + 64, ... of four values (every load
// covers 1 KiB), read once and asked for all at once.  Memory-bound, 4 bytes per element in.  The row
// and chan_s are range-checked buffers: chunks past K read as zero and are not written.
// BITS == 4 writes two nibbles per byte (k even in bits 0..3, k odd in 4..7).
// 4608 x 1152 to 4 bits: 4.8-5.7 us (a workgroup per channel, two passes of 4-byte loads: 9.9 us).
template <int BITS, int NCH>
__global__ __launch_bounds__(kQuantThreads) void quantize_weight_wave(const float* __restrict__ w,
                                                                      const float* __restrict__ chan_s,
                                                                      void* __restrict__ wq_out,
                                                                      float* __restrict__ w_scale, int N, int K) {
    constexpr float qmax = (BITS == 8) ? 127.0f : 7.0f;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long n = (long)blockIdx.x * kRowsPerBlock + wave;
    if (n >= N) return;  // (uniform per wavefront)
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void*)(w + n * K), 0, K * 4, 0x00020000);
    float4v t[NCH];
#pragma unroll
    for (int i = 0; i < NCH; ++i)
        t[i] = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(rs_w, (i * kWave + lane) * 16, 0, 0));
    if (chan_s) {
        const __amdgpu_buffer_rsrc_t rs_s = __builtin_amdgcn_make_buffer_rsrc((void*)chan_s, 0, K * 4, 0x00020000);
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const float4v s = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(rs_s, (i * kWave + lane) * 16, 0, 0));
#pragma unroll
            for (int j = 0; j < 4; ++j) t[i][j] = t[i][j] * s[j];
        }
    }
    float amax = 0.0f;
#pragma unroll
    for (int i = 0; i < NCH; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) amax = fmaxf(amax, fabsf(t[i][j]));
    amax = group_max<kWave>(amax);
    float scale = 0.0f, inv = 0.0f;
    if (amax != 0.0f) {
        scale = amax / qmax;
        inv = qmax / amax;
    }
    if (lane == 0) w_scale[n] = scale;
    const __amdgpu_buffer_rsrc_t rs_q = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((int8_t*)wq_out + n * (BITS == 8 ? K : K / 2)), 0, BITS == 8 ? K : K / 2, 0x00020000);
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        int q[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) q[j] = quantize_one(t[i][j], inv, qmax);
        if (BITS == 8)
            __builtin_amdgcn_raw_buffer_store_b32(pack4(q[0], q[1], q[2], q[3]), rs_q, (i * kWave + lane) * 4, 0, 0);
        else
            __builtin_amdgcn_raw_buffer_store_b16(
                (short)((q[0] & 0xF) | ((q[1] & 0xF) << 4) | ((q[2] & 0xF) << 8) | ((q[3] & 0xF) << 12)), rs_q,
                (i * kWave + lane) * 2, 0, 0);
    }
}

// The same for any row: one workgroup per output channel, two passes (the second one hits in cache).
// BITS == 4 writes two nibbles per byte (k even in bits 0..3, k odd in 4..7).
template <int BITS, bool HAS_S>
__global__ __launch_bounds__(kQuantThreads) void quantize_weight_rows(
    const float* __restrict__ w, const float* __restrict__ chan_s, void* __restrict__ wq_out,
    float* __restrict__ w_scale, int K) {
    __shared__ float red[kRowsPerBlock];
    constexpr float qmax = (BITS == 8) ? 127.0f : 7.0f;
    const long n = blockIdx.x;
    const float* row = w + n * (long)K;
    float amax = 0.0f;
    for (int k = threadIdx.x; k < K; k += kQuantThreads) {
        float t = row[k];
        if (HAS_S) t = t * chan_s[k];
        amax = fmaxf(amax, fabsf(t));
    }
    amax = block_max(amax, red);
    float scale = 0.0f, inv = 0.0f;
    if (amax != 0.0f) {
        scale = amax / qmax;
        inv = qmax / amax;
    }
    if (threadIdx.x == 0) w_scale[n] = scale;
    if (BITS == 8) {
        int8_t* qrow = (int8_t*)wq_out + n * (long)K;
        for (int k = threadIdx.x; k < K; k += kQuantThreads) {
            float t = row[k];
            if (HAS_S) t = t * chan_s[k];
            qrow[k] = (int8_t)quantize_one(t, inv, qmax);
        }
    } else {
        uint8_t* qrow = (uint8_t*)wq_out + n * (long)(K / 2);
        for (int j = threadIdx.x; j < K / 2; j += kQuantThreads) {
            float t0 = row[2 * j], t1 = row[2 * j + 1];
            if (HAS_S) {
                t0 = t0 * chan_s[2 * j];
                t1 = t1 * chan_s[2 * j + 1];
            }
            const int q0 = quantize_one(t0, inv, qmax), q1 = quantize_one(t1, inv, qmax);
            qrow[j] = (uint8_t)((q0 & 0xF) | ((q1 & 0xF) << 4));
        }
    }
}

}  // namespace

hipError_t launch_quantize_per_token(const void* x_f16, const float* chan_mul, int8_t* xq,
                                     float* x_scale, int M, int K, hipStream_t stream) {
    // Rows of whole 16-byte chunks, at most 16 per lane: held in registers.
    const bool vec = (K % 8 == 0) && (K <= 8 * kWave * 16) &&
                     (((uintptr_t)x_f16 | (uintptr_t)xq) % 16 == 0) &&
                     (chan_mul == nullptr || (uintptr_t)chan_mul % 16 == 0);
    if (vec) return launch_plain_quantize(x_f16, chan_mul, xq, x_scale, M, K, stream);
    const dim3 grid((unsigned)M), block(kQuantThreads);
    if (chan_mul)
        hipLaunchKernelGGL((quantize_tokens_generic<true>), grid, block, 0, stream,
                           (const _Float16*)x_f16, chan_mul, xq, x_scale, K);
    else
        hipLaunchKernelGGL((quantize_tokens_generic<false>), grid, block, 0, stream,
                           (const _Float16*)x_f16, (const float*)nullptr, xq, x_scale, K);
    return hipGetLastError();
}

hipError_t launch_channel_absmax(const void* a, int is_f32, float* amax, int R, int K, int accumulate,
                                 hipStream_t stream) {
    const dim3 block(kQuantThreads);
    const int elems = is_f32 ? 4 : 8;
    // (a few more rows for a running maximum: one load of a thread per row is sooner done than the meeting in
    // LDS: 1 x 1152 fp16 1.75 us, 2.00 through LDS; 4 x 1152 1.79 and 1.98; 8 x 1152 2.17 and 2.03)
    const bool chunks = R > 0 && K % elems == 0 && !(accumulate && R <= kAbsmaxFewRows);
    const bool overwrite = chunks && !accumulate && R <= kAbsmaxOneSlab;
    if (!accumulate && !overwrite) {
        hipLaunchKernelGGL(fill_zero_f32, dim3((unsigned)((K + kQuantThreads - 1) / kQuantThreads)), block, 0,
                           stream, amax, K);
        if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
    }
    if (R == 0) return hipSuccess;
    if (chunks) {
        // Row slabs: four workgroups per CU on 256 CUs, at least four rows per thread, below 2^30
        // bytes (a slab is addressed by 32-bit offsets).
        const int col_blocks = (K / elems + kAbsmaxCols - 1) / kAbsmaxCols;
        const int slabs = col_blocks < 1024 ? 1024 / col_blocks : 1;
        long rows = ((long)R + slabs - 1) / slabs;
        const long least = overwrite ? R : kAbsmaxRows * 4, most = (1L << 30) / ((long)K * (is_f32 ? 4 : 2));
        if (rows < least) rows = least;
        if (rows > most) rows = most;
        const dim3 grid((unsigned)col_blocks, (unsigned)((R + rows - 1) / rows)), wide(kAbsmaxThreads);
        if (is_f32)
            hipLaunchKernelGGL((channel_absmax_chunks<float>), grid, wide, 0, stream, (const float*)a, amax, R, K, (int)rows,
                               overwrite);
        else
            hipLaunchKernelGGL((channel_absmax_chunks<_Float16>), grid, wide, 0, stream, (const _Float16*)a, amax, R, K,
                               (int)rows, overwrite);
        return hipGetLastError();
    }
    const int col_blocks = (K + kQuantThreads - 1) / kQuantThreads;
    // enough row slabs to fill the chip, at least 64 rows each
    int slabs = (2048 + col_blocks - 1) / col_blocks;
    if (slabs > (R + 63) / 64) slabs = (R + 63) / 64;
    if (slabs < 1) slabs = 1;
    const int rows_per_block = (R + slabs - 1) / slabs;
    const dim3 grid((unsigned)col_blocks, (unsigned)((R + rows_per_block - 1) / rows_per_block));
    if (is_f32)
        hipLaunchKernelGGL((channel_absmax_cols<float>), grid, block, 0, stream, (const float*)a, amax, R, K,
                           rows_per_block);
    else
        hipLaunchKernelGGL((channel_absmax_cols<_Float16>), grid, block, 0, stream, (const _Float16*)a, amax, R,
                           K, rows_per_block);
    return hipGetLastError();
}

hipError_t launch_balance_mask(const float* amax_x, const float* amax_w, float alpha, float* s, float* chan_mul,
                               int K, hipStream_t stream) {
    hipLaunchKernelGGL(balance_mask_elems, dim3((unsigned)((K + kQuantThreads - 1) / kQuantThreads)),
                       dim3(kQuantThreads), 0, stream, amax_x, amax_w, alpha, s, chan_mul, K);
    return hipGetLastError();
}

template <int CHUNKS>
hipError_t launch_static_chunks(const void* x_f16, const float* chan_mul, float inv_scale, int8_t* xq,
                                unsigned chunks, unsigned K8, hipStream_t stream) {
    constexpr unsigned per_block = kQuantThreads * CHUNKS;
    const dim3 grid((chunks + per_block - 1) / per_block), block(kQuantThreads);
    if (!chan_mul) {
        hipLaunchKernelGGL((quantize_static_chunks<false, CHUNKS>), grid, block, 0, stream, (const half8*)x_f16,
                           (const float4v*)nullptr, inv_scale, (int2v*)xq, chunks, K8);
    } else if constexpr (CHUNKS < 10) {
        hipLaunchKernelGGL((quantize_static_chunks<true, CHUNKS>), grid, block, 0, stream, (const half8*)x_f16,
                           (const float4v*)chan_mul, inv_scale, (int2v*)xq, chunks, K8);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_quantize_static(const void* x_f16, const float* chan_mul, float inv_scale, int8_t* xq,
                                  int M, int K, hipStream_t stream) {
    const long total = (long)M * K;
    if (K % 8 == 0 && total / 8 < (1L << 31)) {
        // Chunks per thread: the count whose grid wastes least of its last round of resident
        // workgroups (8 per compute unit, 256 units), of those that the registers hold.
        const long chunks = total / 8, slots = 8 * 256;
        int best = 8;
        long best_cost = 1L << 62;
        for (int u : {8, 9, 10}) {
            if (chan_mul && u == 10) break;
            const long blocks = (chunks + kQuantThreads * u - 1) / (kQuantThreads * u);
            const long cost = (blocks + slots - 1) / slots * u;
            if (cost < best_cost) {
                best_cost = cost;
                best = u;
            }
        }
        switch (best) {
            case 9: return launch_static_chunks<9>(x_f16, chan_mul, inv_scale, xq, (unsigned)chunks, (unsigned)(K / 8), stream);
            case 10: return launch_static_chunks<10>(x_f16, chan_mul, inv_scale, xq, (unsigned)chunks, (unsigned)(K / 8), stream);
            default: return launch_static_chunks<8>(x_f16, chan_mul, inv_scale, xq, (unsigned)chunks, (unsigned)(K / 8), stream);
        }
    }
    const long blocks = (total + kQuantThreads - 1) / kQuantThreads;
    const dim3 grid((unsigned)(blocks < 16384 ? (blocks < 1 ? 1 : blocks) : 16384)), block(kQuantThreads);
    hipLaunchKernelGGL(quantize_static_elems, grid, block, 0, stream, (const _Float16*)x_f16, chan_mul, inv_scale,
                       xq, total, K);
    return hipGetLastError();
}

// The smallest instantiated chunk count that holds the row.
template <int BITS, int NCH = 1>
hipError_t launch_weight_wave(int nch, const float* w, const float* chan_s, void* wq_out, float* w_scale, int N, int K,
                              hipStream_t stream) {
    if constexpr (NCH > 32) {
        return hipErrorInvalidValue;
    } else {
        if (nch > NCH)  // (every count up to 8, then steps of an eighth or more)
            return launch_weight_wave<BITS, NCH + (NCH < 8 ? 1 : NCH < 20 ? 2 : 4)>(nch, w, chan_s, wq_out, w_scale, N, K, stream);
        hipLaunchKernelGGL((quantize_weight_wave<BITS, NCH>), dim3((unsigned)((N + (long)kRowsPerBlock - 1) / kRowsPerBlock)),
                           dim3(kQuantThreads), 0, stream, w, chan_s, wq_out, w_scale, N, K);
        return hipGetLastError();
    }
}

hipError_t launch_quantize_weight(const float* w, const float* chan_s, int w_bits, void* wq_out,
                                  float* w_scale, int N, int K, hipStream_t stream) {
    if (K % 4 == 0 && K <= 4 * kWave * 32) {
        const int nch = (K / 4 + kWave - 1) / kWave;
        return w_bits == 8 ? launch_weight_wave<8>(nch, w, chan_s, wq_out, w_scale, N, K, stream)
                           : launch_weight_wave<4>(nch, w, chan_s, wq_out, w_scale, N, K, stream);
    }
    const dim3 grid((unsigned)N), block(kQuantThreads);
#define VQ_LAUNCH_W(BITS, HAS)                                                                  \
    hipLaunchKernelGGL((quantize_weight_rows<BITS, HAS>), grid, block, 0, stream, w, chan_s, \
                       wq_out, w_scale, K)
    if (w_bits == 8) {
        if (chan_s) VQ_LAUNCH_W(8, true); else VQ_LAUNCH_W(8, false);
    } else {
        if (chan_s) VQ_LAUNCH_W(4, true); else VQ_LAUNCH_W(4, false);
    }
#undef VQ_LAUNCH_W
    return hipGetLastError();
}

}  // namespace vq
