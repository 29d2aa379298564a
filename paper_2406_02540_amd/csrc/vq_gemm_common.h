// Device helpers shared by the GEMM kernels of this library (vq_gemm.hip: large
// persistent tiles; vq_gemm_tiles.hip, vq_gemm_split.hip: one tile per workgroup for problems that do not fill the
// chip).  gfx950 only.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace vq {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) void* lds_ptr;

constexpr unsigned kRsrcFlags = 0x00020000;  // raw buffer, 32-bit data format

// LDS row r of the weight tile holds which output channel of the tile.
// Rows are kept in MFMA order: r = slab*64 + b*32 + c, with c the column of MFMA block b and the lane (of both halves)
// that holds its sums.  Sending channel slab*64 + 2c + b there gives a lane two neighbouring channels.
__device__ __forceinline__ int w_row_to_channel(int r) { return (r & ~63) + 2 * (r & 31) + ((r >> 5) & 1); }

__device__ __forceinline__ unsigned clamp_u32(long v) {
    return v > 0xFFFFFFFFl ? 0xFFFFFFFFu : (unsigned)v;
}

// Raw buffer descriptor: base address, no stride, size in bytes (accesses past
// it read as zero and never fault), 32-bit data format.
__device__ __forceinline__ v4i make_rsrc(const void* base, unsigned bytes) {
    const unsigned long long p = (unsigned long long)base;
    v4i r;
    // (base and size are the same for every lane of a wave: saying so keeps the descriptor in
    // scalar registers, where the buffer instructions want it, however it was computed)
    r[0] = __builtin_amdgcn_readfirstlane((int)(unsigned)p);
    r[1] = __builtin_amdgcn_readfirstlane((int)(unsigned)(p >> 32) & 0xFFFF);
    r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
    r[3] = (int)kRsrcFlags;
    return r;
}

// (M0 is a reserved register: naming it as clobbered is what tells the compiler that these
// statements change it, and the compiler answers with a warning that says no more than that.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// 16 bytes per lane from buffer offset voff + soff straight into LDS at
// lds_addr + 16 * lane (lds_addr is wave-uniform and goes through M0, which the
// statement declares as clobbered).  Counts in vmcnt; the compiler does not know
// about it, see wait_loads_and_barrier().
__device__ __forceinline__ void load_to_lds_16(v4i rsrc, unsigned lds_addr, int voff, int soff) {
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "buffer_load_dwordx4 %1, %2, %3 offen lds"
        :
        : "s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff)
        : "memory", "m0");
}
// The same with 4 bytes per lane, to lds_addr + 4 * lane.
__device__ __forceinline__ void load_to_lds_4(v4i rsrc, unsigned lds_addr, int voff) {
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "buffer_load_dword %1, %2, 0 offen lds"
        :
        : "s"(lds_addr), "v"(voff), "s"(rsrc)
        : "memory", "m0");
}

#pragma clang diagnostic pop

// A 16-byte load for a stage at byte k0 of the rows.  K a multiple of the stage: k0 rides in the scalar
// offset.  Otherwise (the last stage reaches past K) it is added to the per-lane offset, the part
// of the address that the buffer's range check looks at, and the lanes whose piece lies at or past
// the end of the row (k0 >= k_end, the row's bytes less the piece's place in the stage) get an
// offset behind the buffer: their pieces arrive in LDS as zeros, so that nothing behind this knows
// of the tail.  (Zeroing the weight operand after its LDS read instead took eight vector
// instructions of every K step, which a SIMD does not run under its products: 8192 x 1168 -> 3456
// 45.3 us, 42.9 as it is; with 4-bit weights 1001 x 1184 -> 4608 18.4 and 16.3.)
// The buffer is shorter than 2^31 bytes.
template <bool K_TAIL>
__device__ __forceinline__ void load_stage_to_lds_16(v4i rsrc, unsigned lds_addr, int voff, int k0, int k_end) {
    if (K_TAIL)
        load_to_lds_16(rsrc, lds_addr, k0 < k_end ? voff + k0 : 0x7FFFFFF0, 0);
    else
        load_to_lds_16(rsrc, lds_addr, voff, k0);
}

// Waits until all of this wave's direct loads (and stores) have completed and all
// its LDS accesses are done, then joins the workgroup barrier.
__device__ __forceinline__ void wait_loads_and_barrier() {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" : : : "memory");
}

// The same, but the newest N vector memory operations of this wave may stay in flight
// (they complete in the order of issue: everything older has completed).
template <int N>
__device__ __forceinline__ void wait_loads_before_and_barrier() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(N) : "memory");
}

// Barrier for LDS traffic only: loads in flight stay in flight.
__device__ __forceinline__ void wait_lds_and_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory");
}

// 16 nibbles (two dwords) -> 16 bytes holding 16 * w: the nibble is moved to
// the high half of its byte, sign bit included, in the order of K.
__device__ __forceinline__ v4i widen_nibbles(v2i p) {
    v4i o;
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        const unsigned w = (unsigned)p[d];
        const unsigned even = (w << 4) & 0xF0F0F0F0u;  // k = 0,2,4,6 of this dword
        const unsigned odd = w & 0xF0F0F0F0u;          // k = 1,3,5,7
        o[2 * d] = (int)__builtin_amdgcn_perm(odd, even, 0x05010400u);      // k = 0,1,2,3
        o[2 * d + 1] = (int)__builtin_amdgcn_perm(odd, even, 0x07030602u);  // k = 4,5,6,7
    }
    return o;
}

// The dequantization of two neighbouring outputs into one register of two fp16 values:
//     y = fp16( a * s + float(bias) ),
// the multiply-add exact and rounded once, to nearest even, straight to fp16 (the mixed-precision
// multiply-add takes fp32 a and s and the fp16 bias as they are).  bias2 holds the two bias
// values as they lie in memory (low half first).  Every GEMM kernel of the library narrows
// through these, so that an output does not depend on which kernel computed it.
__device__ __forceinline__ unsigned dequant_pair(float a0, float s0, float a1, float s1, unsigned bias2) {
    unsigned d;
    asm("v_fma_mixlo_f16 %0, %1, %2, %3 op_sel:[0,0,0] op_sel_hi:[0,0,1]" : "=v"(d) : "v"(a0), "v"(s0), "v"(bias2));
    asm("v_fma_mixhi_f16 %0, %1, %2, %3 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "+v"(d) : "v"(a1), "v"(s1), "v"(bias2));
    return d;
}
// The same without a scale (the fp16 comparison layer): y = fp16( a + float(bias) ), rounded once.
__device__ __forceinline__ unsigned add_bias_pair(float a0, float a1, unsigned bias2) {
    unsigned d;
    asm("v_fma_mixlo_f16 %0, %1, 1.0, %2 op_sel:[0,0,0] op_sel_hi:[0,0,1]" : "=v"(d) : "v"(a0), "v"(bias2));
    asm("v_fma_mixhi_f16 %0, %1, 1.0, %2 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "+v"(d) : "v"(a1), "v"(bias2));
    return d;
}

// Returns v unchanged but opaque to the optimiser: what is derived from the result is
// recomputed where it is used instead of being kept in registers across the mainloop.
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// ---- how rows of Y are written by the kernels that store them from the registers -------------------------
// A store is two dwords (four channels) per lane over four token rows x 128 bytes in the persistent kernel, a dword over two of them
// in 256 x 192 with 4-bit weights and the tiles of one per workgroup.
//   kHalfLines: rows start on 64-byte boundaries (N % 32 == 0): range-checked, past the caches (nontemporal).  Through them
//               over random problems 4 to 6 % longer in the persistent tiles (fp16 operands 2 to 3 %), 7 % in 128 x 256, 4 % in
//               128 x 128, 2 % in 128 x 64: 32768 x 1152 -> 4608 169 us and 161 (4-bit weights 168 and 160), 1001 x 1152 -> 4608
//               12.6 and 11.7.  Nor does a quantizer that reads Y right behind it want them there: both together 1 % shorter to 3 %
//               longer through them.
//   kDwords:    rows start on dwords (N even): range-checked, through the caches.  A piece of 128 bytes that begins elsewhere
//               than a memory sector does is two part-written sectors, which the L2 puts together with those of the
//               neighbouring pieces and memory does not.  us past the caches / through them / as any row: 20120 x 352 -> 3464
//               103 / 65 / 66, 8192 x 1152 -> 3472 46.0 / 37.7 / 38.3, 8192 x 1152 -> 1156 22.2 / 17.4 / 17.6, 1001 x 1152 -> 4610
//               13.5 / 12.9 / 14.4; fp16 operands 20120 x 352 -> 3464 109 / 81 / 82.  Over random problems past them 1.21 to
//               1.26 of the time through them in the persistent tiles (fp16 operands 1.03 to 1.12), 1.01 in 128 x 128, 1.04 in 128 x
//               64 and 128 x 256; as any row 1.00 to 1.03 and 1.03 to 1.09.
//   kAnyRow:    odd N, whose every other row starts between dwords, N from 2^21, and an optional copy of the integer sums:
//               64-bit addresses, and a comparison for every row.
enum Out { kHalfLines, kDwords, kAnyRow };
inline Out rows_out(int N, const void* y, const void* acc_out) {
    if (N % 2 != 0 || acc_out || N >= (1 << 21)) return kAnyRow;   // (a tile's rows within 2^31 bytes)
    return N % 32 == 0 && (uintptr_t)y % 64 == 0 ? kHalfLines : kDwords;
}
// `rows` rows of Y in bytes, where stores are range-checked: a tile's are within 2^31 there.  0 for any row: those are addressed in
// 64 bits, and with their N the product may not fit (an overflow is undefined even where nothing uses it).
template <Out OUT>
__host__ __device__ constexpr int checked_bytes(int rows, int N) {
    return OUT == kAnyRow ? 0 : rows * N * 2;
}
static_assert(checked_bytes<kDwords>(256, (1 << 21) - 1) > 0 && checked_bytes<kAnyRow>(256, 0x7FFFFFFF) == 0, "nothing overflows");

// Blocks of 16x16x64, 4-bit weights: which 16 bytes of nibbles of a row (0 .. 3: 0, 3, 1, 2) the lanes of group l/16 read for two K
// steps, and so which two 16-byte chunks of the activations.  The LDS serves sixteen lanes of a ds_read_b128 at a time, rows 0 to 3
// and 12 to 15 of one group with rows 4 to 11 of its neighbour (and the other way round), and the XOR by the row keeps those
// apart only where the two groups' chunks differ by 1, 6 or 7 of the activations and by 3 of the nibbles.  With group l/16 at chunk
// l/16 every read took four cycles more: 640 a stage of 256 x 256, 15 % of a launch's cycles (SQ_LDS_BANK_CONFLICT), none so.
__device__ __forceinline__ int nibble_chunk(int group) { return (group << 1 & 2) | (group >> 1 ^ (group & 1)); }

// ---- persistent kernels: tiles of 256 tokens ---------------------------------------------------
constexpr int kTileK = 128;                 // K bytes per stage (one cache line per row)
constexpr int kBand = 8;                    // token tiles per band in the tile order
constexpr int kXcds = 8;
constexpr int kTouchRounds = 4;             // weight lines asked for up front: at most 4 x 8 KiB per wave (64 MiB per 256 CUs)

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

// The grid for tiles of t x c outputs and the tile fields of `a`; false if they are more than the kernel counts.
inline bool persistent_grid(GemmArgs& a, dim3& grid, int t, int c, int num_cus) {
    if (a.M > 0x7FFFFF00 || a.N > 0x7FFFFF00) return false;  // (rows and channels of a last tile fit an int)
    a.tiles_t = (a.M + t - 1) / t;
    a.tiles_c = (a.N + c - 1) / c;
    const long tiles = (long)a.tiles_t * a.tiles_c;
    if (tiles > 0x7FFFFFF0l) return false;
    a.tiles = (int)tiles;
    a.tiles_per_xcd = (a.tiles + kXcds - 1) / kXcds;
    // one workgroup per CU (the kernels need most of a CU's LDS), fewer if there are fewer tiles
    const int cus_per_xcd = num_cus >= kXcds ? num_cus / kXcds : 1;
    a.slots = a.tiles_per_xcd < cus_per_xcd ? a.tiles_per_xcd : cus_per_xcd;
    grid = dim3((unsigned)(a.slots * kXcds));
    return true;
}

// The 256 x 192 tile: 8-bit weights and fp16 operands (vq_gemm_192.hip), 4-bit weights (vq_gemm_192w4.hip).
hipError_t launch_gemm_192(const GemmArgs& a, int w_bits, int num_cus, hipStream_t stream);
hipError_t launch_gemm_192w4(GemmArgs a, int num_cus, hipStream_t stream);

// ---- kernels that take one tile per workgroup ------------------------------------------------
// ceil(2^32 / d): the high half of n times this is n / d for 2 <= d and n * d < 2^32 (the product exceeds
// n / d by less than n / 2^32 < 1 / d).  The kernel begins with two divisions, and a division by a number
// that is not known is 25 dependent instructions.
inline unsigned reciprocal_of(unsigned d) { return 0xFFFFFFFFu / d + 1u; }

constexpr int kLine = 128;       // K bytes per line of the kernels whose wavefronts divide K
constexpr int kTileXcds = 8;
constexpr int kTileBand = 8;     // token tiles per band in the tile order

struct TileGrid {
    int tiles, tiles_per_xcd, tiles_c, tiles_t;
    unsigned div_band, div_last;   // reciprocals of a band's tiles and of the last band's rows (reciprocal_of), or 0
};

// Whether tiles of t x c outputs, a workgroup of so many threads each, are one launch: HIP takes less than 2^32 threads.
inline bool tiles_launchable(int M, int N, int t, int c, int threads) {
    const long tiles = (((long)M + t - 1) / t) * (((long)N + c - 1) / c);
    return tiles <= 0x7FFFFF00l && (tiles + kTileXcds - 1) / kTileXcds * kTileXcds * threads < (1l << 32);
}

// The grid for tiles of t x c outputs; false if they are more than a launch takes.
inline bool tile_grid(TileGrid& g, int M, int N, int t, int c, int threads) {
    if (!tiles_launchable(M, N, t, c, threads)) return false;
    g.tiles_t = (int)(((long)M + t - 1) / t);
    g.tiles_c = (int)(((long)N + c - 1) / c);
    const long tiles = (long)g.tiles_t * g.tiles_c;
    g.tiles = (int)tiles;
    g.tiles_per_xcd = (g.tiles + kTileXcds - 1) / kTileXcds;
    const int last = g.tiles_t % kTileBand;
    const bool small = g.tiles < 65536 && kTileBand * (long)g.tiles_c < 65536;
    g.div_band = small ? reciprocal_of((unsigned)(kTileBand * g.tiles_c)) : 0;
    g.div_last = small && last > 1 ? reciprocal_of((unsigned)last) : 0;
    return true;
}

struct TileArgs {
    const int8_t* xq;
    const float* x_scale;
    const void* w;
    const float* w_scale;
    const _Float16* bias;
    _Float16* y;
    int32_t* acc_out;
    int M, N, K;
    TileGrid grid;
};

// vq_gemm_tiles.hip: 32 x 32, 64 x 64, 128 x 64, 128 x 128 or 128 x 256, the wavefronts sharing the tile.  w_bits 8 or 4.
constexpr int shared_tile_threads(int tile_t) { return tile_t == 32 ? 256 : 512; }
hipError_t launch_gemm_tiles(int tile_t, int tile_c, const TileArgs& a, int w_bits, hipStream_t stream);
// vq_gemm_split.hip: 32 x 32 (3, 6 or 8 wavefronts), 64 x 32 (4), 64 x 64 (8) or 48 x 48 (8), the wavefronts dividing K.
hipError_t launch_gemm_split(int tile_t, int tile_c, int waves, const TileArgs& a, int w_bits, hipStream_t stream);

// The workgroup's tile, or false.  Workgroup ids are dealt round-robin to the XCDs: each gets a contiguous
// run of tiles, in bands of token tiles, column by column within a band, so that its L2 sees few panels.
__device__ __forceinline__ bool locate_tile(const TileGrid& g, int& row, int& col) {
    const int logical = (blockIdx.x % kTileXcds) * g.tiles_per_xcd + blockIdx.x / kTileXcds;
    if ((int)(blockIdx.x / kTileXcds) >= g.tiles_per_xcd || logical >= g.tiles) return false;
    const int band_tiles = kTileBand * g.tiles_c;
    const int band = g.div_band ? (int)__umulhi((unsigned)logical, g.div_band) : logical / band_tiles;
    const int in_band = logical - band * band_tiles;
    const int band_rows = min(g.tiles_t - band * kTileBand, kTileBand);
    if (band_rows == kTileBand) col = in_band / kTileBand;
    else if (g.div_last) col = (int)__umulhi((unsigned)in_band, g.div_last);
    else col = in_band / band_rows;
    row = band * kTileBand + in_band - col * band_rows;
    return true;
}

// Eight neighbouring channels of a token: sums, dequantized and written; `left` of them exist.
// (Rows of Y start at any even address.  The 4-bit path summed 16 * w.)
template <int W_BITS>
__device__ __forceinline__ void write_eight(v4i v0, v4i v1, float xs, v4f s0, v4f s1, v4i bias8, int left, _Float16* y, int32_t* acc) {
    typedef v4i v4i_any __attribute__((aligned(2)));
    typedef v4i v4i_any4 __attribute__((aligned(4)));
    constexpr int kAccShift = (W_BITS == 4) ? 4 : 0;
    xs *= (W_BITS == 4) ? 0.0625f : 1.0f;
    v4i out;
    out[0] = (int)dequant_pair((float)v0[0], xs * s0[0], (float)v0[1], xs * s0[1], (unsigned)bias8[0]);
    out[1] = (int)dequant_pair((float)v0[2], xs * s0[2], (float)v0[3], xs * s0[3], (unsigned)bias8[1]);
    out[2] = (int)dequant_pair((float)v1[0], xs * s1[0], (float)v1[1], xs * s1[1], (unsigned)bias8[2]);
    out[3] = (int)dequant_pair((float)v1[2], xs * s1[2], (float)v1[3], xs * s1[3], (unsigned)bias8[3]);
    if (left >= 8) {
        *(v4i_any*)y = out;
    } else {
        const half8 o = (half8)out;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (e < left) y[e] = o[e];
    }
    if (acc) {
        if (left >= 8) {
            *(v4i_any4*)acc = v0 >> kAccShift;
            *(v4i_any4*)(acc + 4) = v1 >> kAccShift;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (e < left) acc[e] = (e < 4 ? v0[e & 3] : v1[e & 3]) >> kAccShift;
        }
    }
}

}  // namespace vq
