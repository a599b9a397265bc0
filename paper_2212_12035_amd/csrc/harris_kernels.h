// Device code of the fused Harris coarsity kernels for gfx950 (MI355X): included by the
// translation units that instantiate them (harris_tiles_f32.hip, harris_tiles_u8.hip,
// harris_bands.hip), never by host-only code.
//
// One kernel computes every stage of the Harris operator (thesis chapter 4,
// section 4.2: grayscale, Sobel pair, products, 3x3 window sums, coarsity) and
// touches device memory only to read the RGB planes once and to write the result
// once.  The schedule is this library's own; what it keeps from the thesis's
// section 4.3 is the idea of a pipeline over image lines with separated 3x3
// kernels and rotating registers, re-cut for a 64-lane wavefront:
//
//  * A wavefront owns a vertical strip of the image.  Lane l holds PX adjacent
//    columns; one row of one plane is a single coalesced load of 64*PX elements
//    (128 bits per lane for float32 at PX = 4).
//  * Vertical taps never touch memory: the last two gray rows and what the window sums
//    need of the rows of (Ix^2, Ix*Iy, Iy^2) live in registers ("register rotation").  Row
//    steps are unrolled, so the rotation is a renaming, not a copy.
//  * Both 3x3 stages are separated (section 4.3, "Convolution Separation"):
//    taps down the column from registers, taps along the row from the lanes beside (the window
//    sums and 8-bit input down the column first; float32 input takes [-1 0 1] along the row
//    first, row_step says why).  Horizontal neighbours come from the lane to the right through a DPP
//    wave shift; each stage consumes two columns from the right, so a lane's
//    output columns start at the lane's own first input column and the result row
//    is stored with aligned vector stores.
//  * The strip of a wavefront overlaps its right neighbour by the 4-column halo;
//    the last lane(s) only supply that halo.
//
// Two schedules run this pipeline:
//  * Tiles (the default, harris_tile_kernel): a workgroup of NW wavefronts takes NW*RW
//    input rows of one strip; every wavefront requests its RW rows at once, hands its
//    first four gray rows to the wavefront above through LDS (one barrier), and
//    stores its RW result rows in one burst at the end.
//  * Bands (harris_fused_kernel): one long-lived wavefront walks a band of R result
//    rows with a register queue of D input rows in flight; no LDS, no barrier.  Odd
//    bands walk upwards, so two neighbouring bands begin on the rows they share.
// In both, tiles are dealt to workgroups so that each XCD (own L2) gets contiguous runs of
// tiles: one, or in launches of many tiles several by turns.
#ifndef HARRIS_KERNELS_H
#define HARRIS_KERNELS_H

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <math.h>
#include <type_traits>

#include "harris_tuning.h"
#include "harris_launch.h"

namespace {

constexpr int kWave = 64;

// ---------------------------------------------------------------- small helpers

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

constexpr int gcd_c(int a, int b) { return b == 0 ? a : gcd_c(b, a % b); }
constexpr int lcm_c(int a, int b) { return a / gcd_c(a, b) * b; }

// Value of v in the lane to the right (lane + 1); lanes without one get 0.
// DPP control 0x130 is "wave shift left by 1": lane i reads lane i + 1.
__device__ __forceinline__ float from_right(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));
}

// Column I of a lane's PX columns, I < PX + 2: beyond the lane's own it is the next lane's.  Written
// at the place of its use, with the operation that takes it, the lane shift becomes a modifier of
// that operation; the compiler looks only some 20 instructions ahead for it, and leaves a move of
// its own for every shift whose use lies further away.
template <int I, int PX>
__device__ __forceinline__ float column(const float (&a)[PX]) {
    if constexpr (I < PX) return a[I];
    else if constexpr (I < 2 * PX) return from_right(a[I - PX]);
    else return from_right(from_right(a[I - 2 * PX]));
}

// ---------------------------------------------------------------- row loads and stores

// Cache policy of the accesses (the "aux" operand of the buffer instructions): bit 0 = sc0,
// bit 1 = nt (non-temporal), bit 4 = sc1.  0 is the default policy.  Results are never read
// back, so they are always stored non-temporal.  Input rows are loaded non-temporal when the
// whole problem fits the last-level cache anyway, and with the default policy otherwise: then
// the line that two neighbouring strips share, and the rows that two neighbouring
// bands share, are found in the CU's vector cache by the second wavefront of the
// same workgroup.
// The policies are compile-time constants of the instructions; the macros exist so that a build
// with other values can be timed against this one.  Measured (us, interleaved runs on one GPU):
//   stores nt + sc1 (written through at device scope) instead of nt, many small tiles whose strip
//     borders lie on 64-byte boundaries of float32 rows: 8192x8192 uint8 84.8 against 86.6, 64x1080x1920
//     354.1 / 355.6, 4096x4096 44.7 / 45.0;
//     borders and row ends inside 64-byte blocks, which then reach the memory in parts: 16x1079x1919
//     100.3 / 91.8, 8191x8191 uint8 94.1 / 89.5, to 16-bit and 8-bit results 16x1079x1919 float32 to
//     binary16 87.9 / 81.0, 8192x8192 uint8 to binary16 77.3 / 72.3 and to codes 73.0 / 69.5 -- so only
//     float32 results with moved borders take it, and those only where a row has more strips than
//     ends (one strip: 781 images of 240x160 105.0 / 86.5, 521 of 240x240 91.4 / 80.9; two: 391 of 240x320 100.3 /
//     86.9, 312 of 240x400 90.7 / 82.2, but 258 of 240x484, 480 result columns, 78.6 / 78.5), from float32 input beyond
//     400 MB more than six (480 MB of images of 720 rows: three strips 81.1 / 78.1, four 77.8 / 76.9, six 79.6 / 78.1 and 75.1 /
//     74.7, eight 76.2 / 76.2; 128 of 720x1280, six, 316 / 308; but 64 of 1080x1920, eight, 333 / 337; up to 400 MB, and
//     from uint8 input, three to eight strips are 0.98 to 1.03 of the time either way, on the whole better written through);
//     small launches gain whatever their borders: up to 16 MB from uint8 to float32 and 16 bits (17 images of
//     237x320 4.99 / 5.37, 1101x1630 5.64 / 6.21, 7 of 480x642 at 15 MB 6.36 / 6.71, but 19 of 300x401 at 16.4 MB the
//     same either way; 727x2200 to binary16 4.79 / 5.12), up to 13 MB from float32 to float32 (6 of 260x332
//     4.16 / 4.54, 9 of them 4.70 / 4.90, but 3 of 480x642 at 15 MB 5.23 / 5.13; to 16 bits and codes never;
//     nor where the strip is the row: 268 of 34x25 uint8 6.41 / 6.11, 21 of 240x240 float32 5.57 / 5.17);
//     one tile per CU, 1536x2560: 12.7 against 12.0 -- nor does that kernel (kWriteThrough is the rule);
//   default-policy stores: 13.4 (1536x2560), 97.6 (8192x8192 uint8), 39.8 (2832x4256);
//   loads nt + sc1: 12.8 on 1536x2560, no change on the large workloads; sc1 without nt, or
//     sc1 on the rows two tiles share: 4 to 22 % slower.
#ifndef HARRIS_LOAD_AUX
#define HARRIS_LOAD_AUX 2
#endif
#ifndef HARRIS_STORE_AUX
#define HARRIS_STORE_AUX 2
#endif
#ifndef HARRIS_MANY_STORE_AUX
#define HARRIS_MANY_STORE_AUX 18
#endif
constexpr int kAuxDefault = 0;
constexpr int kAuxNonTemporal = HARRIS_LOAD_AUX;
// Tile kernel only, not a hardware value: non-temporal, except that the first and the last
// four input rows of a tile, which the tile above or below reads as well, are loaded with the
// default policy.  The launches that use it are those of many small tiles; their float32 stores are
// written through (kAuxManyStore) if strips end on 64-byte boundaries.
constexpr int kAuxKeepShared = -1;
// Tile kernel only: rows that do not lie within 2 GB of each other, with the default policy and as kAuxKeepShared.
constexpr int kAuxFar = -2, kAuxFarKeepShared = -3;
constexpr int kAuxStore = HARRIS_STORE_AUX, kAuxManyStore = HARRIS_MANY_STORE_AUX;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Buffer descriptor over `bytes` bytes at p: raw (unstrided) 32-bit data.  A lane
// whose byte offset is not below `bytes` loads 0 and stores nothing.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}

// One row segment of the three planes as raw 32-bit words, PX pixels per lane.
template <typename In, int PX>
struct RawRow {
    static constexpr int NW = std::is_same<In, float>::value ? PX : (PX + 3) / 4;
    uint32_t w[3][NW];
};

// One plane's part of it: voff is the lane's byte offset and soff the wavefront's, both from where rs begins.  The
// hardware loads zeros where voff is not below the descriptor's size less soff.
template <typename In, int PX, int AUX>
__device__ __forceinline__ void load_plane_row(RawRow<In, PX>& r, int c, __amdgpu_buffer_rsrc_t rs, uint32_t voff, uint32_t soff) {
    constexpr int BYTES = PX * (int)sizeof(In);
    if constexpr (BYTES >= 16) {
#pragma unroll
        for (int j = 0; j < BYTES / 16; ++j) {
            u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, voff + 16 * j, soff, AUX);
            r.w[c][4 * j + 0] = v.x; r.w[c][4 * j + 1] = v.y; r.w[c][4 * j + 2] = v.z; r.w[c][4 * j + 3] = v.w;
        }
    } else if constexpr (BYTES == 8) {
        u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, voff, soff, AUX);
        r.w[c][0] = v.x; r.w[c][1] = v.y;
    } else if constexpr (BYTES == 4) {
        r.w[c][0] = __builtin_amdgcn_raw_buffer_load_b32(rs, voff, soff, AUX);
    } else if constexpr (BYTES == 2) {
        r.w[c][0] = __builtin_amdgcn_raw_buffer_load_b16(rs, voff, soff, AUX);
    } else {
        r.w[c][0] = __builtin_amdgcn_raw_buffer_load_b8(rs, voff, soff, AUX);
    }
}

// row points at column 0 of the row in plane 0; voff is the lane's byte offset in the row.
template <typename In, int PX, int AUX>
__device__ __forceinline__ void load_row(RawRow<In, PX>& r, const In* row, size_t plane, uint32_t row_bytes, uint32_t voff) {
#pragma unroll
    for (int c = 0; c < 3; ++c) load_plane_row<In, PX, AUX>(r, c, make_rsrc(row + c * plane, row_bytes), voff, 0);
}

// 8-bit rows that start on any byte, four pixels per lane: every lane loads the aligned 32-bit
// word at its offset from the row's address rounded down to 4 bytes, so no access is
// misaligned and none leaves the aligned words that hold the row's bytes.  With the row
// starting `shift` bytes into its first word, a lane's four pixels are the upper bytes of its
// word and the lower bytes of the word of the lane to its right (realign_row).
// voff is the lane's first column (a multiple of 4); shift[c] is kept for realign_row, which takes it modulo 4.
template <int AUX>
__device__ __forceinline__ void load_row_shifted(RawRow<uint8_t, 4>& r, uint32_t (&shift)[3], const uint8_t* row, size_t plane,
                                                 uint32_t row_bytes, uint32_t voff) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const uintptr_t a = reinterpret_cast<uintptr_t>(row + c * plane);
        shift[c] = (uint32_t)a & 3u;
        const uint32_t bytes = row_bytes ? (row_bytes + shift[c] + 3u) & ~3u : 0u;
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(reinterpret_cast<const void*>(a & ~(uintptr_t)3), bytes);
        r.w[c][0] = __builtin_amdgcn_raw_buffer_load_b32(rs, voff, 0, AUX);
    }
}

typedef uint32_t u32_any __attribute__((aligned(1)));

__device__ __forceinline__ void realign_row(RawRow<uint8_t, 4>& r, const uint32_t (&shift)[3]) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const uint32_t own = r.w[c][0];
        const uint32_t right = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)own, 0x130, 0xf, 0xf, true);
        r.w[c][0] = __builtin_amdgcn_alignbyte(right, own, shift[c] & 3u);
    }
}

// PX results of one lane to a result row described by rs (its size is the row's
// bytes, or 0 to store nothing); voff is the lane's byte offset in the row.  (No offset in a scalar register: the compiler lets the
// data of a 16-byte store that has one be overwritten by the next instruction, and wrong results were stored.)
template <int PX, int AUX = kAuxStore>
__device__ __forceinline__ void store_row(const float (&o)[PX], __amdgpu_buffer_rsrc_t rs, uint32_t voff) {
    if constexpr (PX >= 4) {
#pragma unroll
        for (int j = 0; j < PX / 4; ++j) {
            u32x4 v = {__float_as_uint(o[4 * j]), __float_as_uint(o[4 * j + 1]), __float_as_uint(o[4 * j + 2]), __float_as_uint(o[4 * j + 3])};
            __builtin_amdgcn_raw_buffer_store_b128(v, rs, voff + 16 * j, 0, AUX);
        }
    } else if constexpr (PX == 2) {
        u32x2 v = {__float_as_uint(o[0]), __float_as_uint(o[1])};
        __builtin_amdgcn_raw_buffer_store_b64(v, rs, voff, 0, AUX);
    } else {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o[0]), rs, voff, 0, AUX);
    }
}

// float32 -> bit pattern of the nearest binary16 / bfloat16 value (ties to even, overflow to
// infinity, NaN stays NaN), by the hardware conversions: round-to-nearest-even is the mode
// HIP kernels run in, and gfx950 converts two float32 values to a bfloat16 pair in one
// instruction.
__device__ __forceinline__ uint32_t to_f16_bits(float x) {
    return (uint32_t)__builtin_bit_cast(unsigned short, (_Float16)x);
}
__device__ __forceinline__ uint32_t to_bf16_bits(float x) {
    return (uint32_t)__builtin_bit_cast(unsigned short, (__bf16)x);
}
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
// Two values in one 32-bit word: lo in bits 0..15, hi in bits 16..31.
template <bool BF>
__device__ __forceinline__ uint32_t to_16bit_pair(float lo, float hi) {
    const f32x2 v = {lo, hi};
    if constexpr (BF) return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
    else return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));
}

// PX results of one lane as 16-bit values (BF: bfloat16, else binary16); voff is the lane's
// byte offset in the row (2 bytes per column).
template <int PX, bool BF, int AUX = kAuxStore>
__device__ __forceinline__ void store_row_16(const float (&o)[PX], __amdgpu_buffer_rsrc_t rs, uint32_t voff) {
    if constexpr (PX >= 4) {
#pragma unroll
        for (int j = 0; j < PX / 4; ++j) {
            const u32x2 v = {to_16bit_pair<BF>(o[4 * j], o[4 * j + 1]), to_16bit_pair<BF>(o[4 * j + 2], o[4 * j + 3])};
            __builtin_amdgcn_raw_buffer_store_b64(v, rs, voff + 8 * j, 0, AUX);
        }
    } else if constexpr (PX == 2) {
        __builtin_amdgcn_raw_buffer_store_b32(to_16bit_pair<BF>(o[0], o[1]), rs, voff, 0, AUX);
    } else {
        __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(BF ? to_bf16_bits(o[0]) : to_f16_bits(o[0])), rs, voff, 0, AUX);
    }
}

// PX results of one lane as 8-bit codes clamp(rint(fma(v, scale, offset)), 0, 255); NaN gives 0.
// The hardware's float-to-byte conversion does the rounding (to nearest, ties to even), the
// clamp and the packing into byte i of a word in one instruction per value.  voff is the
// lane's byte offset in the row (1 byte per column).
template <int PX, int AUX = kAuxStore>
__device__ __forceinline__ void store_row_8(const float (&o)[PX], float scale, float offset, __amdgpu_buffer_rsrc_t rs, uint32_t voff) {
    constexpr int WORDS = (PX + 3) / 4;
    uint32_t w[WORDS];
#pragma unroll
    for (int j = 0; j < WORDS; ++j) w[j] = 0u;
#pragma unroll
    for (int i = 0; i < PX; ++i) w[i / 4] = __builtin_amdgcn_cvt_pk_u8_f32(fmaf(o[i], scale, offset), (uint32_t)(i % 4), w[i / 4]);
    if constexpr (PX >= 4) {
#pragma unroll
        for (int j = 0; j < WORDS; ++j) __builtin_amdgcn_raw_buffer_store_b32(w[j], rs, voff + 4 * j, 0, AUX);
    } else if constexpr (PX == 2) {
        __builtin_amdgcn_raw_buffer_store_b16((unsigned short)w[0], rs, voff, 0, AUX);
    } else {
        __builtin_amdgcn_raw_buffer_store_b8((unsigned char)w[0], rs, voff, 0, AUX);
    }
}

// Grayscale.  float32 input: gray = wr*R + wg*G + wb*B.  8-bit input: 299 R + 587 G + 114 B, a whole number below 2^18, in units of
// 2^-18: exact, and so are the sums and differences of gray values that the Sobel responses are made of (whole numbers below 2^21).  The
// result is multiplied by what that leaves out, the Sobel scale and 1/255000 each to the fourth power (Params::gain), when it is complete.
constexpr float kGrayUnit = 1.0f / 262144.0f;
template <typename In, int PX>
__device__ __forceinline__ void gray_row(const RawRow<In, PX>& r, float wr, float wg, float wb, float (&g)[PX]) {
#pragma unroll
    for (int i = 0; i < PX; ++i) {
        if constexpr (std::is_same<In, float>::value) {
            g[i] = fmaf(wb, __uint_as_float(r.w[2][i]), fmaf(wg, __uint_as_float(r.w[1][i]), wr * __uint_as_float(r.w[0][i])));
        } else {
            float ch[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) ch[c] = (float)((r.w[c][i / 4] >> (8 * (i % 4))) & 0xffu);
            g[i] = fmaf(114.0f * kGrayUnit, ch[2], fmaf(587.0f * kGrayUnit, ch[1], (299.0f * kGrayUnit) * ch[0]));
        }
    }
}

// The same of float32 input in the registers of the red row.  Ten rows in flight leave a wavefront of 128 registers none for another row: the
// compiler, which does not reuse a loaded row's registers one by one, spills there.
template <int PX>
__device__ __forceinline__ void gray_row_in_place(RawRow<float, PX>& r, float wr, float wg, float wb, float (&g)[PX]) {
#pragma unroll
    for (int i = 0; i < PX; ++i) {
        asm("v_mul_f32_e32 %0, %1, %0" : "+v"(r.w[0][i]) : "s"(wr));
        g[i] = fmaf(wb, __uint_as_float(r.w[2][i]), fmaf(wg, __uint_as_float(r.w[1][i]), __uint_as_float(r.w[0][i])));
    }
}

// The same numbers for 8-bit input with four pixels per lane, on the matrix cores.  v_mfma_f32_4x4x4 multiplies sixteen pairs of 4x4
// matrices, one for every four lanes: each lane brings four values, its column of the right matrix, and gets four, its column of
// the product.  With a diagonal matrix on the left, lane l of four holding row l, every lane's four pixels of a plane are multiplied by
// the plane's weight and added to its sums, exactly: bytes and weights are exact in binary16, sums in float32.  A byte becomes
// binary16 by standing alone in 16 bits, a subnormal number of as many 2^-24; 64 times the weight makes that units of
// 2^-18.  Six byte permutes and three matrix instructions take the place of twelve conversions and twelve multiply-adds: launches that
// vector instructions bound gain, 3712x2348 to codes 11.0 us (11.4 without), 31 images of 598x300 to bfloat16 10.3 (10.6), 1580x2832 9.2 (9.5).
// (Loads that convert, buffer_load_format_d16_xyzw, save the permutes too but run at half the rate: 8192x8192 90 us against 81.)
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
struct GrayMatrix {
    u32x2 row[3];           // this lane's row of the three matrices
    uint32_t select[2];     // the permutes that put a lane's pixels 0 and 1, 2 and 3 into halves of a word
};
// drop: bits by which the lane's pixels stand further up in the loaded word than they should.
__device__ __forceinline__ GrayMatrix gray_matrix(unsigned lane, unsigned drop) {
    const uint32_t half = 0xffffu << (16u * (lane & 1u)), lo = lane & 2u ? 0u : half, hi = lane & 2u ? half : 0u;
    constexpr uint32_t kWeights[3] = {0x74ac74acu, 0x78967896u, 0x6f206f20u};       // 64 x 299, 64 x 587 and 64 x 114 in binary16, twice
    GrayMatrix a;
#pragma unroll
    for (int c = 0; c < 3; ++c) a.row[c] = u32x2{lo & kWeights[c], hi & kWeights[c]};
    a.select[0] = 0x0c010c00u + (drop >> 3) * 0x00010001u;
    a.select[1] = 0x0c030c02u + (drop >> 3) * 0x00010001u;      // may name a byte of the word again: of columns that nobody uses
    return a;
}
__device__ __forceinline__ void gray_row(const RawRow<uint8_t, 4>& r, const GrayMatrix& a, float (&g)[4]) {
    f32x4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const uint32_t w = r.w[c][0];
        const u32x2 pixels = {__builtin_amdgcn_perm(w, w, a.select[0]), __builtin_amdgcn_perm(w, w, a.select[1])};
        sum = __builtin_amdgcn_mfma_f32_4x4x4f16(__builtin_bit_cast(f16x4, a.row[c]), __builtin_bit_cast(f16x4, pixels), sum, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) g[i] = sum[i];
}

// ---------------------------------------------------------------- the pipeline state of one lane

template <int PX>
struct LineBuffers {
    float g[2][PX];       // the last two gray rows (kQuads: the last one)
    float d[2][PX];       // kDifferences: and their differences along the row, [-1 0 1]
    float q[2][PX];       // kQuads: the last row of sums over 2x2 gray values
    float x[2][PX];       // box window: Ix, Iy of the last even row
    float p[2][3][PX];    // Ix*Ix, Ix*Iy, Iy*Iy: of the last odd row (box, in p[1]), of the last two rows (binomial)
    float t[3][PX];       // box window: sums of the products of two neighbouring rows, an odd one and the even one below it
};

// One row step.  The sums that a row's results are made of are added up in an order that depends on whether the
// row's number in its band or tile is even: equal input rows may differ in their results' last bits.
// T is the row's number in its band or tile, modulo 2 at least: it fixes the slots of
// the row's values (T % 2).
// STAGE 0: gray only (first two rows of a band); 1: also Sobel and products (next
// two rows); 2: also window sums and coarsity: one result row in o, for the caller to store.
//
// Both Sobel kernels are separated, and the order of the passes is free at six operations a pixel:
//   kDifferences  takes the difference along the row first, of gray values that are close to each other: it is small and mostly
//                 exact, and what is added up afterwards rounds at that size (1536x2560 float32: error of the result
//                 against 64 bits 2.4e-7 of its norm, 3.0e-7 with the sums first).  float32 input, which pays 3 to 7
//                 registers a lane for two rows of differences and, in launches of 8 to 15 MB in tiles of 4 x 4, up to 4 % (6 images of 260x332 4.16 us,
//                 3.95 with the sums first; 4 of 480x642 5.39 / 5.31; larger ones nothing).
//   kSums         sums down the column first; for float32 instances without these registers.
//   kQuads        sums over 2x2 gray values first; their differences along the two diagonals are, added and subtracted,
//                 the responses: three lane shifts a row instead of five.  8-bit input, where every one of these numbers is exact: the
//                 result's error against 64 bits is 1.1e-7 of its norm, 4.0e-7 with gray values that are rounded.  (The window sums could be taken of the
//                 diagonal differences themselves, which are the gradient turned by 45 degrees; that saves two more operations a
//                 pixel, but an edge along the rows or columns then cancels in the determinant: up to 6.1e-7.)
//
// A row's Sobel responses can go out to the wavefront above (kSobelOut, in `sobel`) or come from the one below
// (kSobelIn; gc is not looked at then).  kQuadsIn: gc is the row's 2x2 sums.
enum SobelRow { kSobelOwn, kSobelOut, kSobelIn, kQuadsIn };
enum SobelOrder { kSums, kDifferences, kQuads };
struct Coarsity { float k, gain; };     // gain: kQuads

template <int STAGE, int T, int PX, bool BINOM, int ORDER, int SOBEL>
__device__ __forceinline__ void row_step(LineBuffers<PX>& lb, const float (&gc)[PX], const Coarsity& cs, float (&o)[PX], float (&sobel)[2][PX]) {
    constexpr int PS = T % 2;
    constexpr bool GIVEN = SOBEL == kSobelIn, DIFF = ORDER == kDifferences, QUADS = ORDER == kQuads;
    if constexpr (QUADS && SOBEL == kQuadsIn) {
#pragma unroll
        for (int i = 0; i < PX; ++i) lb.q[PS][i] = gc[i];
    } else if constexpr (QUADS && T >= 1 && !GIVEN) {
        float pair[PX];
#pragma unroll
        for (int i = 0; i < PX; ++i) pair[i] = lb.g[1 - PS][i] + gc[i];
        static_for<0, PX>([&](auto ii) {
            constexpr int i = decltype(ii)::value;
            lb.q[PS][i] = column<i + 1, PX>(pair) + pair[i];
        });
    }
    [[maybe_unused]] float dx[PX];                // DIFF: [-1 0 1] along the row
    if constexpr (DIFF && !GIVEN) {
        static_for<0, PX>([&](auto ii) {
            constexpr int i = decltype(ii)::value;
            dx[i] = column<i + 2, PX>(gc) - gc[i];
        });
    }
    [[maybe_unused]] float v[3][PX];              // [1 c 1] down the column of the three products
    if constexpr (STAGE >= 1) {
        [[maybe_unused]] float sy[PX];            // without DIFF: [1 2 1] down the column
        [[maybe_unused]] float dy[PX];            // [-1 0 1] down the column
#pragma unroll
        for (int i = 0; i < PX && !GIVEN && !QUADS; ++i) {
            dy[i] = gc[i] - lb.g[PS][i];
            if constexpr (!DIFF) sy[i] = fmaf(2.0f, lb.g[1 - PS][i], lb.g[PS][i] + gc[i]);
        }
        static_for<0, PX>([&](auto ii) {
            constexpr int i = decltype(ii)::value;
            float ix, iy;
            [[maybe_unused]] float falling, rising;
            if constexpr (QUADS && !GIVEN) {
                falling = column<i + 1, PX>(lb.q[PS]) - lb.q[1 - PS][i];
                rising = lb.q[PS][i] - column<i + 1, PX>(lb.q[1 - PS]);
            }
            if constexpr (GIVEN) ix = sobel[0][i];
            else if constexpr (QUADS) ix = falling - rising;
            else if constexpr (DIFF) ix = fmaf(2.0f, lb.d[1 - PS][i], lb.d[PS][i] + dx[i]);
            else ix = column<i + 2, PX>(sy) - sy[i];
            if constexpr (GIVEN) iy = sobel[1][i];
            else if constexpr (QUADS) iy = falling + rising;
            else iy = fmaf(2.0f, column<i + 1, PX>(dy), column<i + 2, PX>(dy) + dy[i]);   // [1 2 1] along the row
            if constexpr (SOBEL == kSobelOut) { sobel[0][i] = ix; sobel[1][i] = iy; }
            // Products and window sums down the column (the window is separated too, c = 1 for
            // the unweighted sum, 2 for the binomial window).
            const float fa[3] = {ix, ix, iy}, fb[3] = {ix, iy, iy};
            if constexpr (BINOM) {
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const float p = fa[q] * fb[q];
                    if constexpr (STAGE >= 2) v[q][i] = fmaf(2.0f, lb.p[1 - PS][q][i], lb.p[PS][q][i] + p);
                    lb.p[PS][q][i] = p;
                }
            } else if constexpr (PS == 0) {
                // Two neighbouring sums a + b + c and b + c + d share t = b + c, with b the odd
                // row: the even rows' products then occur only as the product of a multiply-add,
                // and a row costs two operations a product instead of three.
                if constexpr (STAGE >= 2) {
                    const float ea[3] = {lb.x[0][i], lb.x[0][i], lb.x[1][i]}, eb[3] = {lb.x[0][i], lb.x[1][i], lb.x[1][i]};
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        lb.t[q][i] = fmaf(fa[q], fb[q], lb.p[1][q][i]);
                        v[q][i] = fmaf(ea[q], eb[q], lb.t[q][i]);
                    }
                }
                lb.x[0][i] = ix;
                lb.x[1][i] = iy;
            } else {
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    lb.p[1][q][i] = fa[q] * fb[q];
                    if constexpr (STAGE >= 2) v[q][i] = lb.t[q][i] + lb.p[1][q][i];
                }
            }
        });
    }
#pragma unroll
    for (int i = 0; i < PX && !GIVEN && SOBEL != kQuadsIn; ++i) {
        lb.g[PS][i] = gc[i];
        if constexpr (DIFF) lb.d[PS][i] = dx[i];
    }
    if constexpr (STAGE >= 2) {
        // Along the row neighbouring results share a pair sum.
        float s[3][PX];
        static_for<0, 3>([&](auto qq) {
            constexpr int q = decltype(qq)::value;
            if constexpr (BINOM) {
                float pair[PX];                           // v[i] + v[i+1]
                static_for<0, PX>([&](auto ii) {
                    constexpr int i = decltype(ii)::value;
                    pair[i] = column<i + 1, PX>(v[q]) + v[q][i];
                });
                static_for<0, PX>([&](auto ii) {
                    constexpr int i = decltype(ii)::value;
                    s[q][i] = column<i + 1, PX>(pair) + pair[i];   // v[i] + 2 v[i+1] + v[i+2]
                });
            } else if constexpr (PX == 1) {
                s[q][0] = (column<1, PX>(v[q]) + v[q][0]) + column<2, PX>(v[q]);
            } else {
                static_for<0, PX / 2>([&](auto jj) {
                    constexpr int j = decltype(jj)::value;
                    const float pair = column<2 * j + 2, PX>(v[q]) + v[q][2 * j + 1];
                    s[q][2 * j] = v[q][2 * j] + pair;
                    s[q][2 * j + 1] = column<2 * j + 3, PX>(v[q]) + pair;
                });
            }
        });
        // Coarsity.
#pragma unroll
        for (int i = 0; i < PX; ++i) {
            float det = fmaf(s[0][i], s[2][i], -(s[1][i] * s[1][i]));
            float tr = s[0][i] + s[2][i];
            o[i] = fmaf(-(cs.k * tr), tr, det);
            if constexpr (QUADS) o[i] *= cs.gain;
        }
    }
}

template <int STAGE, int T, int PX, bool BINOM, int ORDER>
__device__ __forceinline__ void row_step(LineBuffers<PX>& lb, const float (&gc)[PX], const Coarsity& cs, float (&o)[PX]) {
    [[maybe_unused]] float none[2][PX];
    row_step<STAGE, T, PX, BINOM, ORDER, kSobelOwn>(lb, gc, cs, o, none);
}

// ---------------------------------------------------------------- the kernel

// Tiles are numbered image-major, then band, then strip.  Workgroup b of the grid is
// placed on XCD b % 8 by the hardware dispatcher; this gives XCD x the x-th contiguous
// run of workgroup-sized tile groups.
__device__ __forceinline__ unsigned xcd_contiguous(unsigned b, unsigned nb) {
    const unsigned q = nb / 8, r = nb % 8, x = b % 8, j = b / 8;
    return x * q + min(x, r) + j;       // XCDs 0..r-1 take q + 1 groups each, the others q
}

template <typename In, int PX, int D, int LAUX, bool BINOM>
__global__ __launch_bounds__(256) void harris_fused_kernel(const harris_launch::Params p) {
    constexpr int ORDER = std::is_same<In, float>::value ? kDifferences : kQuads;
    constexpr int U = lcm_c(2, D);            // row steps per loop trip: queue slots and parities stay static

    const unsigned lane = threadIdx.x % kWave;
    const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const unsigned waves_per_block = blockDim.x / kWave;
    unsigned blk = blockIdx.x;
    blk = (p.flags & HARRIS_TUNE_NO_XCD_REMAP) ? blk : xcd_contiguous(blk, p.n_blocks);

    // A workgroup of 2 or 4 wavefronts holds two vertically adjacent bands (of one strip,
    // or of two adjacent strips): band 2j walks upwards and band 2j+1 downwards, so both
    // begin on the four input rows they share, and the second request for those rows (and
    // for the cache line two adjacent strips share) is served by the CU's vector cache.
    const unsigned group_h = waves_per_block >= 2 ? 2u : 1u;
    const unsigned group_w = waves_per_block / group_h;
    const unsigned img = blk / p.blocks_per_image;
    const unsigned rem = blk % p.blocks_per_image;
    const int band = (int)((rem / p.blocks_x) * group_h + wave / group_w);
    const int strip = (int)((rem % p.blocks_x) * group_w + wave % group_w);
    if (band >= (int)p.n_bands || strip >= (int)p.n_strips) return;   // uniform per wavefront; no barrier is ever used

    const int y0 = band * p.rows_per_band;                      // first result row of the band
    const int rows = min(p.rows_per_band, p.n - y0);            // result rows of this band (>= 1)
    const int steps = rows + 4;                                 // input rows consumed
    const bool up = !(p.flags & HARRIS_TUNE_NO_ALTERNATE) && !(band & 1);

    // A strip yields p.strip_pitch result columns (at most 64*PX - 4, the same for every
    // strip so that all wavefronts carry the same load); the lanes beyond only supply halo.
    const unsigned col = (unsigned)strip * p.strip_pitch + lane * PX; // first column of this lane (input and result)
    const unsigned lcol = min(col, (unsigned)(p.W - PX));       // loads stay inside the row
    // Lanes beyond the strip's columns and its 4-column halo request nothing (out-of-range offset).
    const uint32_t load_voff = lane * PX < p.strip_pitch + 4 ? lcol * (uint32_t)sizeof(In) : 0x80000000u;
    // Halo-only lanes store nothing: an offset beyond any row.  Lanes whose columns lie
    // right of the result row are dropped by the buffer's range check.
    const uint32_t store_voff = lane * PX < p.strip_pitch ? col * 4u : 0x80000000u;
    const uint32_t in_row_bytes = (uint32_t)p.W * (uint32_t)sizeof(In);
    const uint32_t out_row_bytes = (uint32_t)p.m * 4u;

    const size_t plane = (size_t)p.in_plane_pitch;
    const In* img_in = static_cast<const In*>(p.rgb) + (size_t)img * (size_t)p.in_image_pitch;
    float* img_out = static_cast<float*>(p.out) + (size_t)img * (size_t)p.out_image_pitch;   // float32 results only

    // Input row read at step t.  Steps past the band's end (the loop runs in trips of U
    // steps, and the queue reads D rows ahead) get an empty descriptor: such a load
    // returns zeros and moves no data.
    auto in_row_ptr = [&](int t) -> const In* {
        int r = up ? y0 + rows + 3 - t : y0 + t;
        r = max(0, min(p.H - 1, r));
        return img_in + (size_t)r * (size_t)p.in_row_pitch;
    };
    auto in_row_size = [&](int t) -> uint32_t { return t < steps ? in_row_bytes : 0u; };

    RawRow<In, PX> queue[D];
    static_for<0, D>([&](auto d) {
        constexpr int dd = decltype(d)::value;
        load_row<In, PX, LAUX>(queue[dd], in_row_ptr(dd), plane, in_row_size(dd), load_voff);
        __builtin_amdgcn_sched_barrier(0);
    });

    LineBuffers<PX> lb;
    const Coarsity cs = {p.k, p.gain};
    float gc[PX], o[PX];

    // Rows 0..3 of the band fill the pipeline.
    static_for<0, 4>([&](auto tt) {
        constexpr int t = decltype(tt)::value;
        gray_row<In, PX>(queue[t % D], p.wr, p.wg, p.wb, gc);
        __builtin_amdgcn_sched_barrier(0);
        load_row<In, PX, LAUX>(queue[t % D], in_row_ptr(t + D), plane, in_row_size(t + D), load_voff);
        __builtin_amdgcn_sched_barrier(0);
        row_step<(t < 2 ? 0 : 1), t, PX, BINOM, ORDER>(lb, gc, cs, o);
    });

    for (int t0 = 4; t0 < steps; t0 += U) {
        static_for<0, U>([&](auto uu) {
            constexpr int u = decltype(uu)::value;
            const int t = t0 + u;
            // The slot's registers are free as soon as its gray row exists: refill it at
            // once, so that D rows stay in flight while the rest of the step computes.
            gray_row<In, PX>(queue[(4 + u) % D], p.wr, p.wg, p.wb, gc);
            __builtin_amdgcn_sched_barrier(0);
            load_row<In, PX, LAUX>(queue[(4 + u) % D], in_row_ptr(t + D), plane, in_row_size(t + D), load_voff);
            __builtin_amdgcn_sched_barrier(0);
            // Result row: the top row of the 5-row window that this step completes.  Steps
            // past the band's end get an empty descriptor and store nothing.
            const int orow = max(0, min(p.n - 1, up ? y0 + rows + 3 - t : y0 + t - 4));
            const __amdgpu_buffer_rsrc_t out_rs = make_rsrc(img_out + (size_t)orow * (size_t)p.out_row_pitch, t < steps ? out_row_bytes : 0u);
            row_step<2, 4 + u, PX, BINOM, ORDER>(lb, gc, cs, o);
            store_row<PX>(o, out_rs, store_voff);
        });
    }
}


// Makes the compiler finish these values here: without it the last multiply-add of a result
// is moved down to the stores, and its three operands stay in registers instead of the one
// result (the tile kernel holds RW rows of results until its store burst).
template <int PX>
__device__ __forceinline__ void pin_values(float (&v)[PX]) {
#pragma unroll
    for (int i = 0; i < PX; ++i) asm volatile("" : "+v"(v[i]));
}

// Rows of 16-bit results or 8-bit codes that may start on any byte their element type allows, four
// pixels per lane (WORDS): a lane stores its four results where they belong, with one store at any byte, which the hardware
// does; the lane that straddles the end of a row stores the one to three results it has there in one or two pieces.  Nothing is shifted
// between lanes, no descriptor is worked out, and the border between two strips stays where it is.  Against storing the aligned
// words of a row, shifted together from two lanes, and its ends element by element: 16 images of 768x1366 uint8 to codes 19.5 us
// (20.7), 4 of 1289x1121 binomial 10.9 (11.8), 776 of 64x161 13.2 (14.3), 8 of 1079x1919 uint8 to binary16 19.5 (20.2), 3 of
// 1679x1413 float32 to codes 19.9 (20.6); large float32 launches to 16 bits the same within 0.5 %.
template <int KIND>
struct PackedRow {
    static constexpr int NW = KIND == HARRIS_OUT_U8 ? 1 : 2;        // 32-bit words of four results
    uint32_t w[NW];
};
template <int KIND>
__device__ __forceinline__ PackedRow<KIND> pack_row(const float (&o)[4], float q_scale, float q_offset) {
    PackedRow<KIND> r;
    if constexpr (KIND == HARRIS_OUT_U8) {
        r.w[0] = 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) r.w[0] = __builtin_amdgcn_cvt_pk_u8_f32(fmaf(o[i], q_scale, q_offset), (uint32_t)i, r.w[0]);
    } else {
        r.w[0] = to_16bit_pair<KIND == HARRIS_OUT_BF16>(o[0], o[1]);
        r.w[1] = to_16bit_pair<KIND == HARRIS_OUT_BF16>(o[2], o[3]);
    }
    return r;
}
typedef u32x2 u32x2_any __attribute__((aligned(1)));
typedef uint16_t u16_any __attribute__((aligned(1)));
template <typename T> using in_device_memory = __attribute__((address_space(1))) T;      // or the compiler makes flat stores
// row: the strip's first column in the row; voff the lane's byte offset from there.
template <int KIND>
__device__ __forceinline__ void store_packed(const PackedRow<KIND>& r, uintptr_t row, uint32_t voff) {
    in_device_memory<char>* at = reinterpret_cast<in_device_memory<char>*>(row) + voff;
    if constexpr (KIND == HARRIS_OUT_U8) __builtin_nontemporal_store(r.w[0], reinterpret_cast<in_device_memory<u32_any>*>(at));
    else __builtin_nontemporal_store(u32x2{r.w[0], r.w[1]}, reinterpret_cast<in_device_memory<u32x2_any>*>(at));
}
// The lane's first `tail` results, 1 to 3.
template <int KIND>
__device__ __forceinline__ void store_packed_tail(const PackedRow<KIND>& r, uintptr_t row, uint32_t voff, uint32_t tail) {
    in_device_memory<char>* at = reinterpret_cast<in_device_memory<char>*>(row) + voff;
    if constexpr (KIND == HARRIS_OUT_U8) {
        if (tail & 2u) __builtin_nontemporal_store((uint16_t)r.w[0], reinterpret_cast<in_device_memory<u16_any>*>(at));
        if (tail & 1u) __builtin_nontemporal_store((uint8_t)(tail & 2u ? r.w[0] >> 16 : r.w[0]), reinterpret_cast<in_device_memory<uint8_t>*>(at + (tail & 2u)));
    } else {
        if (tail & 2u) __builtin_nontemporal_store(r.w[0], reinterpret_cast<in_device_memory<u32_any>*>(at));
        if (tail & 1u) __builtin_nontemporal_store((uint16_t)(tail & 2u ? r.w[1] : r.w[0]), reinterpret_cast<in_device_memory<u16_any>*>(at + (tail & 2u) * 2u));
    }
}

// ---------------------------------------------------------------- the tile kernel
//
// The default schedule: a
// workgroup of NW wavefronts owns a tile of NW*RW input rows of one strip, and every
// wavefront requests its RW rows (3*RW loads) at once, so no wavefront goes through a
// chain of dependent memory round trips.  Wavefront w turns its rows into gray,
// publishes its first four gray rows in LDS and, after one barrier, takes the four
// gray rows below its own from wavefront w+1 there (8-bit input: a gray row, a row of 2x2 sums and two
// of Sobel responses, below): nothing is read twice inside a tile.  Each wavefront then runs the same register pipeline as the band kernel over
// its RW+4 gray rows and stores RW result rows (the last wavefront has no neighbour
// below and stores RW-4).  A tile yields NW*RW-4 result rows; the tile below re-reads
// four rows.
//
// HANDOFF selects how a wavefront learns that the rows below its own are in LDS.  false: the
// workgroup's barrier, after every wavefront has worked through its own rows.  true: a ready
// flag per wavefront in LDS, set as soon as its first four gray rows are written; a wavefront
// waits only for the flag of the one below it, and a barrier before the store burst keeps the
// stores behind the workgroup's loads.  With one large tile per CU the last wavefront's data
// arrives long after the first's, and without the flags every wavefront's last four rows would
// wait for it and then be computed by all at once (1536x2560: 12.2 against 12.4 us); with many
// small tiles the barrier is faster (720x1280: 6.1 against 6.4 us).
//
// SHIFTED (8-bit input, four pixels per lane): rows start on any byte.  Launches that the vector ALUs or latency bound, WORDS
// and SMALL in tiles of four rows per wavefront and one tile per CU, load their pixels where they are (BYTES): the lane shifts and byte-aligns of
// whole words are 24 of some 480 vector operations per wavefront (codes; counters: 456 without), and the loads, all of one policy, stand in one
// straight line.  16 images of 768x1366 to codes 21.7 us (23.3 with words), 9 of 2442x1862 52.1 (57.1), 8 of 1079x1919 to
// binary16 21.9 (23.8), 1079x1919 to float32 5.67 (5.97), 19 of 300x401 6.50 (6.89).  Large launches to float32 are bound
// by memory and load aligned words (load_row_shifted, realign_row), non-temporal but for the rows that tiles share:
// 8191x8191 88 us (92), 4 of 2159x3839 45.7 (48.6).
//
// WORDS (16-bit results or 8-bit codes, four pixels per lane): result rows start on any byte of their
// type and are stored where they are (store_packed).  Instances of their
// own: as a branch of every four-pixel kernel this code cost the others registers (float32, 10 rows: up
// to 28 vector registers in scratch memory; 2160x3840 23.0 us, 22.2 without; 2159x3839 to binary16
// itself 21.9 and 20.8).
//
// 8-bit input with four pixels per lane hands over, instead of four gray rows, the first one, the 2x2 sums of the first two and the Sobel responses
// that the wavefront has computed from all four (six rows of LDS): the wavefront above needs exactly these, and does
// not compute them again (4 instead of 6 rows of responses for 4 result rows; 8192x8192 at 4 x 4: 390 vector
// operations per wavefront by the counters, 423 before).  8-bit launches that are not held up by memory gain: 16 images of 768x1366 to codes 22.4 us (23.0
// before), 9 of 2442x1862 to codes 51.8 (54.1), 10 of 480x640 to float32 6.80 (6.92), 600x800 3.71 (3.82); 8192x8192 to
// float32 is bound by the memory's view of its tiles (83 us, 84 without any arithmetic) and takes the same time.  At 4 x 4
// the 19 KB leave eight workgroups on a CU.  float32 input is bound by memory and keeps the gray rows.
//
// SMALL (8-bit input, shared rows kept): a launch whose tiles are all resident at once (Params::resident).
//
// Scalar work: a SIMD issues a scalar instruction every four cycles (measured: 4.5 with eight wavefronts), no faster than vector ones, so the
// address arithmetic of short-lived wavefronts can take as long as their pixels.  Rows are therefore loaded through a descriptor
// per plane and a row offset (NEAR), in one branch for a wavefront's load policy, and the result rows' descriptors take a dozen
// instructions each: 8192x8192 uint8 in 4 x 4 tiles some 190 scalar instructions per wavefront by the counters, 327 with a descriptor
// worked out for each row and plane and a branch for each row.  In us (before): 8192x8192 uint8 81.2 (83.6), 4096x4096 23.3 (24.5), 8 of 1080x1920
// 23.1 (23.9), 1536x2560 7.04 (7.47), 480x640 3.06 (3.28), 16 images of 768x1366 to codes 19.6 (20.8), 31 of 598x300 to
// bfloat16 10.6 (10.9), 64x96 float32 2.66 (2.80).  float32 tiles of 8 rows and more gain nothing and keep a descriptor per row.
//
// kAuxFar, kAuxFarKeepShared: a wavefront's rows do not lie within 2 GB of each other, pitches do not fit the compact arguments, or the factor of 8-bit results takes two
// numbers: 64-bit addresses for each row and all arguments whole (four rows per wavefront; plan() in harris_api.cpp sees to it).
// Args: compact::Params, or Params for these two.
template <typename In, int PX, int RW, int LAUX, bool BINOM, bool HANDOFF, bool SHIFTED, bool SMALL, bool WORDS, typename Args>
__device__ __forceinline__ void harris_tile(const Args& args) {
    const harris_launch::compact::Tile p = harris_launch::compact::unpack(args, sizeof(In), RW);
    // Ten rows fill the 128 vector registers that a workgroup of 16 wavefronts leaves each.  Instances that the
    // two rows of differences would push into scratch memory (none that float32 results take by default)
    // take the sums first.
    constexpr int ORDER = std::is_same<In, uint8_t>::value ? kQuads : !(RW == 10 && (LAUX == kAuxKeepShared || WORDS || (BINOM && !HANDOFF))) ? kDifferences : kSums;
    static_assert(!SHIFTED || (std::is_same<In, uint8_t>::value && PX == 4), "shifted rows: 8-bit input, four pixels per lane");
    static_assert(!WORDS || PX == 4, "result rows on any byte: four pixels per lane");
    constexpr bool FAR = LAUX == kAuxFar || LAUX == kAuxFarKeepShared;
    constexpr bool KEEP = LAUX == kAuxKeepShared || LAUX == kAuxFarKeepShared;  // the rows that two tiles share with the default policy, tiles dealt by turns
    constexpr bool MATRIX = std::is_same<In, uint8_t>::value && PX == 4;
    constexpr bool HAND_SOBEL = harris_launch::hands_sobel(std::is_same<In, uint8_t>::value, PX);
    extern __shared__ __align__(16) float halo_lds[];           // [NW][4][64][PX]; HAND_SOBEL: [1 + (NW - 1) * 6][64][PX]
    __shared__ unsigned ready[16];                              // HANDOFF: wavefront w has published its four rows

    const unsigned lane = threadIdx.x % kWave;
    const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if constexpr (HANDOFF) {
        // Every flag is cleared before any wavefront can look at one (the barrier orders the
        // clearing stores before every later access of the workgroup).  At this point the
        // wavefronts of a workgroup are a few hundred cycles apart: the barrier costs nothing measurable.
        if (lane == 0) __hip_atomic_store(&ready[wave], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __syncthreads();
    }
    const unsigned n_waves = p.waves_per_block;                 // == blockDim.x / 64
    unsigned tile = blockIdx.x;
    // The grid size is read with all other arguments, not in a branch of its own: one wait
    // for the arguments instead of two before the first load can be issued.
    unsigned n_blocks = p.n_blocks;
    if constexpr (KEEP) {
        unsigned chunk = p.chunk;
        asm volatile("" : "+s"(n_blocks), "+s"(chunk));
        if (!(p.flags & HARRIS_TUNE_NO_XCD_REMAP)) tile = harris_launch::dealt_tile(tile, blockIdx.y, chunk);
        if (tile >= n_blocks) return;                           // at the end of the last turn; a whole workgroup, before any barrier
    } else {
        asm volatile("" : "+s"(n_blocks));
        tile = (p.flags & HARRIS_TUNE_NO_XCD_REMAP) ? tile : xcd_contiguous(tile, n_blocks);
    }
    // Every workgroup that gets here has a tile, and every wavefront of it reaches the barrier.

    const unsigned img = harris_launch::compact::image_of(args, tile);
    const unsigned rem = tile - img * args.tiles_per_image;
    const int band = (int)harris_launch::compact::band_of(args, rem);
    const int strip = (int)(rem - (unsigned)band * p.n_strips);

    const int tile_rows = p.rows_per_band;                      // result rows per tile: NW*RW - 4
    const int y_wave = band * tile_rows + (int)wave * RW;       // first input row = first result row of this wavefront
    const int y_end = min(p.n, (band + 1) * tile_rows);         // result rows of this tile end here
    const int out_rows = max(0, min(RW, y_end - y_wave));       // result rows this wavefront stores

    const unsigned col = (unsigned)strip * p.strip_pitch + lane * PX;
    // Lanes right of the row load what the last lane with a column of the row loads (nobody
    // uses what they compute).  That lane may straddle the end of the row (a width that is no
    // multiple of PX): it gets zeros for the words beyond the end, since each 32-bit word of a
    // load is checked against the descriptor's size by itself.
    const unsigned lcol = min(col, ((unsigned)p.W - 1u) & ~(unsigned)(PX - 1));
    // Results are float32, 16-bit or 8-bit: esh is log2 of a result element's bytes.
    const unsigned esh = p.out_shift;
    // With aligned stores the border between this strip and the next lies, in each result row,
    // on the first 64-byte boundary of that row's address at or after the nominal border: up to
    // 12 (float32), 28 (16-bit) or 60 (8-bit) columns further right.
    const unsigned x0 = (unsigned)strip * p.strip_pitch;        // first result column of this strip
    // Lanes beyond the strip's columns, the border's reach and the 4-column halo request nothing
    // (out-of-range offset).
    const uint32_t load_voff = lane * PX < p.strip_reach ? lcol * (uint32_t)sizeof(In) : 0x80000000u;
    const uint32_t in_row_bytes = (uint32_t)p.W * (uint32_t)sizeof(In);

    const size_t plane = (size_t)p.in_plane_pitch;
    const In* img_in = static_cast<const In*>(p.rgb) + (size_t)img * (size_t)p.in_image_pitch;
    const uintptr_t img_out = reinterpret_cast<uintptr_t>(p.out) + (uintptr_t)img * p.out_image_bytes;

    // All RW rows of this wavefront at once; rows below the image get an empty descriptor.
    RawRow<In, PX> raw[RW];
    [[maybe_unused]] uint32_t shift[RW][3];                     // SHIFTED: byte offset of each row in its first word
    // Shifted rows: every lane within reach loads the word at its own column (one lane further
    // right than otherwise, which supplies the last lane's missing bytes); the descriptor's
    // size stops the lanes right of the row.
    [[maybe_unused]] const uint32_t shifted_voff = lane * PX < p.strip_reach + 4 ? col : 0x80000000u;
    constexpr bool BYTES = SHIFTED && !FAR && (LAUX == kAuxNonTemporal || (RW == 4 && (WORDS || SMALL || LAUX == kAuxDefault)));
    // BYTES: every lane takes its four pixels with one load at any byte, which the hardware does (byte_lane).  Rows below
    // the image load its last one, and nobody uses what comes of them.
    [[maybe_unused]] const harris_launch::ByteLane bytes = harris_launch::byte_lane(col, (unsigned)p.W);
    constexpr bool NEAR = !FAR && (std::is_same<In, uint8_t>::value ? !SHIFTED || BYTES || !BINOM : RW <= 6);
    if constexpr (NEAR) {
        const int last = p.H - 1 - y_wave;                      // the image's last row, counted from this wavefront's first; negative below the image
        const int y_first = min(y_wave, p.H - 1);
        const harris_launch::NearRows near = harris_launch::near_rows(p.H, y_first, (uint32_t)p.in_row_pitch * (uint32_t)sizeof(In), RW, std::is_same<In, uint8_t>::value);
        const In* first = img_in + (size_t)(unsigned)y_first * (size_t)p.in_row_pitch;
        // A plane's rows from the wavefront's first on, as far as it needs them and the image has them; rows below the image
        // load its last one again, which nobody uses, and wavefronts below it nothing.  From float32, whose lanes may straddle a row's end, every
        // row has a descriptor that ends with it.
        constexpr bool EACH = std::is_same<In, float>::value;
        const uint32_t rows = last < 0 ? 0u : min(near.last, (RW - 1) * near.pitch) + in_row_bytes;
        // SHIFTED words: a plane's rows from the aligned word that its first one begins in; as each row's descriptor ends with the
        // word of the row's last byte, no access leaves the words that hold the row's bytes.  Box window, us (a descriptor per row and plane): 8191x8191
        // 85.1 (87.0), 8 of 1079x1919 23.8 (24.6), 2831x4255 18.3 (18.9), 64 of 333x499 15.5 (16.4); with the binomial window it gains 2 %
        // or loses as much (8 of 1079x1919 25.3 (25.8), 12 of 1001x1303 25.1 (24.7)) and is left out.
        [[maybe_unused]] const uint32_t word_voff = last < 0 ? 0x80000000u : shifted_voff;
        if constexpr (SHIFTED && !BYTES) {
            static_for<0, RW>([&](auto tt) {
                constexpr int t = decltype(tt)::value;
#pragma unroll
                for (int c = 0; c < 3; ++c) shift[t][c] = ((uint32_t)reinterpret_cast<uintptr_t>(first + c * plane) & 3u) + near_row(near, t);
            });
        }
        auto load_all = [&](auto head, auto tail) {
            static_for<0, RW>([&](auto tt) {
                constexpr int t = decltype(tt)::value;
                constexpr bool SHARED = (t < 4 && decltype(head)::value) || (t >= RW - 4 && decltype(tail)::value);
                constexpr int AUX = LAUX != kAuxKeepShared ? LAUX : SHARED ? kAuxDefault : kAuxNonTemporal;
                const uint32_t off = near_row(near, t), end = EACH && last >= 0 ? off + in_row_bytes : rows;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    if constexpr (BYTES) {
                        const u32_any* at = reinterpret_cast<const u32_any*>(first + c * plane + (bytes.voff + off));
                        raw[t].w[c][0] = LAUX == kAuxNonTemporal ? __builtin_nontemporal_load(at) : *at;
                    } else if constexpr (SHIFTED) {
                        const uintptr_t word = reinterpret_cast<uintptr_t>(first + c * plane) & ~(uintptr_t)3;
                        const __amdgpu_buffer_rsrc_t rs = make_rsrc(reinterpret_cast<const void*>(word), (shift[t][c] + in_row_bytes + 3u) & ~3u);
                        raw[t].w[c][0] = __builtin_amdgcn_raw_buffer_load_b32(rs, word_voff, shift[t][c] & ~3u, AUX);
                    } else {
                        load_plane_row<In, PX, AUX>(raw[t], c, make_rsrc(first + c * plane, end), load_voff, off);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);              // row by row: the first is worked on when it is there
            });
        };
        if constexpr (LAUX != kAuxKeepShared || BYTES) load_all(std::false_type{}, std::false_type{});
        else if (wave == 0 || (RW == 4 && wave + 1 == n_waves)) load_all(std::true_type{}, std::false_type{});
        else if (RW != 4 && wave + 1 == n_waves) load_all(std::false_type{}, std::true_type{});
        else load_all(std::false_type{}, std::false_type{});
    } else {
        auto load_far = [&](auto tt, auto aux) {
            constexpr int t = decltype(tt)::value, AUX = decltype(aux)::value;
            const int r = y_wave + t;
            const In* row_in = img_in + (size_t)min(r, p.H - 1) * (size_t)p.in_row_pitch;
            const uint32_t row_bytes = r < p.H ? in_row_bytes : 0u;
            if constexpr (SHIFTED) load_row_shifted<AUX>(raw[t], shift[t], row_in, plane, row_bytes, shifted_voff);
            else load_row<In, PX, AUX>(raw[t], row_in, plane, row_bytes, load_voff);
        };
        const std::integral_constant<int, kAuxDefault> shared_aux;
        const std::integral_constant<int, kAuxNonTemporal> own_aux;
        static_assert(!FAR || RW == 4, "far rows: four per wavefront");
        if constexpr (LAUX == kAuxFar) {
            static_for<0, RW>([&](auto tt) { load_far(tt, shared_aux); });
        } else if constexpr (LAUX == kAuxFarKeepShared) {       // of four rows all are shared, or none
            if (wave == 0 || wave + 1 == n_waves) static_for<0, RW>([&](auto tt) { load_far(tt, shared_aux); });
            else static_for<0, RW>([&](auto tt) { load_far(tt, own_aux); });
        } else {
            static_for<0, RW>([&](auto tt) {
                constexpr int t = decltype(tt)::value;
                if constexpr (LAUX != kAuxKeepShared) load_far(tt, std::integral_constant<int, LAUX>{});
                else if ((t < 4 && wave == 0) || (t >= RW - 4 && wave + 1 == n_waves)) load_far(tt, shared_aux);
                else load_far(tt, own_aux);
            });
        }
    }
    __builtin_amdgcn_sched_barrier(0);

    // Descriptors of the RW result rows, worked out while the loads are in flight (scalar
    // arithmetic that would otherwise sit between the last result and the first store).
    // Result row j of this wavefront is row y_wave + j.  A descriptor covers the strip's columns in that row, from its left border, out_skip
    // bytes behind the strip's first column x0, to its right one; rows past the tile or the image get an empty descriptor,
    // whose address is never used.  A lane's offset counts from the left border and wraps to a huge value for
    // lanes left of it, so lanes outside store nothing.
    __amdgpu_buffer_rsrc_t out_rs[RW];
    [[maybe_unused]] uint32_t out_skip[RW];
    // The empty statement makes everything below depend on values defined after the loads:
    // none of this arithmetic is moved in front of them.
    unsigned sx0 = x0;
    int sy = y_wave;
    asm volatile("" : "+s"(sx0), "+s"(sy) : : "memory");
    const uintptr_t out_pitch = p.out_row_bytes;
    const uintptr_t out_first = img_out + (uintptr_t)(unsigned)sy * out_pitch;
    if constexpr (!WORDS) {
        const uintptr_t at = out_first + (uintptr_t)(sx0 << esh);
        // An image of very many strips may have one that begins behind its last column.
        const uint32_t rest = (uint32_t)max(p.m - (int)sx0, 0) << esh, width = p.strip_pitch << esh;
        int32_t size[RW];                                       // from border to border; signed, as the scalar unit has no saturating subtraction
        const bool moved = p.flags & HARRIS_TUNE_ALIGNED_STORES;
        if (RW <= 6 && !moved) {                                // (taller tiles: one way for both, whose registers they need)
#pragma unroll
            for (int j = 0; j < RW; ++j) { size[j] = (int32_t)min(rest, width); out_skip[j] = 0u; }
        } else {
            const uint32_t right = moved ? 63u : 0u, left = sx0 == 0u ? 0u : right;
            const uint32_t to_left = 0u - (uint32_t)at, to_right = to_left - width, pitch32 = (uint32_t)out_pitch;
#pragma unroll
            for (int j = 0; j < RW; ++j) {
                out_skip[j] = (to_left - (uint32_t)j * pitch32) & left;
                size[j] = (int32_t)min(rest, width + ((to_right - (uint32_t)j * pitch32) & right)) - (int32_t)out_skip[j];
            }
        }
#pragma unroll
        for (int j = 0; j < RW; ++j) {
            out_rs[j] = make_rsrc(reinterpret_cast<const void*>(at + (size_t)j * out_pitch + out_skip[j]), j < out_rows ? (uint32_t)max(size[j], 0) : 0u);
            asm volatile("" : "+s"(out_skip[j]));               // finished here, not next to the store
        }
    }
    uint32_t lane_bytes = (lane * PX) << esh;
    asm volatile("" : "+v"(lane_bytes));
    __builtin_amdgcn_sched_barrier(0);

    LineBuffers<PX> lb;
    const Coarsity cs = {p.k, p.gain};
    [[maybe_unused]] GrayMatrix gray;
    if constexpr (MATRIX) gray = gray_matrix(lane, BYTES ? bytes.drop : 0u);
    float gc[PX], none[PX];
    // The RW result rows stay in registers until the wavefront has used up all its loads and
    // are stored together at the end: bursts of reads and bursts of writes use the memory
    // better than a fine mixture (measured on 1536x2560: 13.0 us against 14.4 us).
    float results[RW][PX];
    // HAND_SOBEL: the first wavefront, which has nobody to publish for, writes its six rows over each other into
    // a row of its own.
    const unsigned my_row = !HAND_SOBEL ? wave * 4u : wave == 0 ? 0u : wave * 6u - 5u;
    const unsigned my_pitch = HAND_SOBEL && wave == 0 ? 0u : kWave * PX;
    float* my_halo = halo_lds + ((size_t)my_row * kWave + lane) * PX;
    auto publish = [&](unsigned row, const float (&v)[PX]) {
        float* at = my_halo + row * my_pitch;
#pragma unroll
        for (int i = 0; i < PX; ++i) at[i] = v[i];
    };

    static_for<0, RW>([&](auto tt) {
        constexpr int t = decltype(tt)::value;
        if constexpr (SHIFTED && !BYTES) realign_row(raw[t], shift[t]);
        if constexpr (MATRIX) gray_row(raw[t], gray, gc);
        else if constexpr (RW == 10) gray_row_in_place<PX>(raw[t], p.wr, p.wg, p.wb, gc);
        else gray_row<In, PX>(raw[t], p.wr, p.wg, p.wb, gc);
        if constexpr (HAND_SOBEL) {
            if constexpr (t == 0) publish(0, gc);
        } else if constexpr (t < 4) {
#pragma unroll
            for (int i = 0; i < PX; ++i) my_halo[(size_t)t * kWave * PX + i] = gc[i];
        }
        if constexpr (HANDOFF && t == 3) {
            // Publish.  The lanes' writes of the four rows are ordered before lane 0's release
            // store by a release fence, a barrier and an acquire fence at wavefront scope; the
            // release store at workgroup scope then carries them to whoever acquires the flag.
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (lane == 0) __hip_atomic_store(&ready[wave], 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        if constexpr (HAND_SOBEL && (t == 2 || t == 3)) {
            float sobel[2][PX];
            row_step<1, t, PX, BINOM, ORDER, kSobelOut>(lb, gc, cs, none, sobel);
            publish(2 * t - 2, sobel[0]);
            publish(2 * t - 1, sobel[1]);
        } else if constexpr (t < 4) {
            row_step<(t < 2 ? 0 : 1), t, PX, BINOM, ORDER>(lb, gc, cs, none);
            if constexpr (HAND_SOBEL && t == 1) publish(1, lb.q[1]);
        } else {
            row_step<2, t, PX, BINOM, ORDER>(lb, gc, cs, results[t - 4]);
            pin_values<PX>(results[t - 4]);
        }
        // Each row is worked through as soon as it has arrived: without this the compiler
        // gathers the arithmetic of all rows behind the wait for the last one.
        __builtin_amdgcn_sched_barrier(0);
    });

    if constexpr (!HANDOFF) __syncthreads();

    if (wave + 1 < n_waves) {
        if constexpr (HANDOFF) {
            // Acquire load of the neighbour's flag: pairs with its release store, so the rows read
            // below are the published ones.  The wait ends: all wavefronts of a workgroup are
            // resident on the CU together (a workgroup is dispatched as a whole), and wavefront
            // wave + 1 reaches its release store without waiting for anybody (every wavefront
            // runs through the code above unconditionally; its loads always return).
            while (__hip_atomic_load(&ready[wave + 1], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) == 0u)
                __builtin_amdgcn_s_sleep(4);
        }
        const float* below = halo_lds + ((size_t)(HAND_SOBEL ? wave * 6u + 1u : (wave + 1) * 4u) * kWave + lane) * PX;
        auto fetch = [&](unsigned row, float (&v)[PX]) {
#pragma unroll
            for (int i = 0; i < PX; ++i) v[i] = below[(size_t)row * kWave * PX + i];
        };
        // HAND_SOBEL: two rows are read ahead of their use where a launch's tiles are all resident at once and a CU has
        // few wavefronts to hide the reads (AHEAD).  Others hide them, and are slower with the rows in registers
        // (13 images of 277x448 to float32 4.81 us ahead, 5.00 not; 600x800 3.65 / 3.73; but 8 of 1080x1920 to binary16
        // 21.3 / 19.7, 4000x3000 to codes 15.0 / 14.3, 9 of 2442x1862 to codes on any byte 54.3 / 51.8).  SMALL launches
        // with the binomial window do without, as it gains a little here and loses a little there (1080x1920 5.01 us, ahead
        // 4.97; 1200x1600 4.96 / 4.90; 4 images of 600x800 5.37 / 5.43); one tile per CU gains (480x640 3.42 us ahead, 3.46 not).
        constexpr bool AHEAD = HAND_SOBEL && !WORDS && (LAUX == kAuxNonTemporal || (SMALL && !BINOM));
        [[maybe_unused]] float sobel[2][2][PX];
        [[maybe_unused]] float second[PX];
        if constexpr (AHEAD) {
            fetch(0, gc);
            fetch(1, second);
            __builtin_amdgcn_sched_barrier(0);
        }
        static_for<RW, RW + 4>([&](auto tt) {
            constexpr int t = decltype(tt)::value, row = t - RW;
            if constexpr (HAND_SOBEL && (AHEAD ? row % 2 == 0 : row >= 2)) {
                // The responses that the step after next takes (two steps ahead), or this step's own.
                constexpr int from = AHEAD ? row / 2 : row - 2;
                fetch(2 * from + 2, sobel[from][0]);
                fetch(2 * from + 3, sobel[from][1]);
                if constexpr (AHEAD) __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (HAND_SOBEL && row >= 2) {
                row_step<2, t, PX, BINOM, ORDER, kSobelIn>(lb, gc, cs, results[t - 4], sobel[row - 2]);
            } else if constexpr (HAND_SOBEL && row == 1) {
                [[maybe_unused]] float nobody[2][PX];
                if constexpr (!AHEAD) fetch(row, second);
                row_step<2, t, PX, BINOM, ORDER, kQuadsIn>(lb, second, cs, results[t - 4], nobody);
            } else {
                if constexpr (!AHEAD) fetch(row, gc);
                row_step<2, t, PX, BINOM, ORDER>(lb, gc, cs, results[t - 4]);
            }
            pin_values<PX>(results[t - 4]);
        });
    }

    // The second factor of 8-bit results: behind a branch of the wavefront, which images that are here for their size pass by (66000x66000 to codes
    // 4.00 ms, 4.08 multiplied by one).
    if constexpr (FAR && ORDER == kQuads) {
        if (__float_as_uint(p.more_gain) != __float_as_uint(1.0f)) {
#pragma unroll
            for (int j = 0; j < RW; ++j)
#pragma unroll
                for (int i = 0; i < PX; ++i) results[j][i] *= p.more_gain;
        }
    }
    // The last wavefront skips the four rows it has no data for.
    if constexpr (HANDOFF) __syncthreads();                     // stores only after all of the workgroup's loads
    __builtin_amdgcn_sched_barrier(0);
    constexpr int SAUX = kAuxStore;
    // The rows of this wavefront in one burst, written through or not (many-tile kernels only).
    [[maybe_unused]] auto store_all = [&](auto&& store_one) {
        if (KEEP && (p.flags & harris_launch::kWriteThrough)) {
            static_for<0, RW>([&](auto jj) {
                if (decltype(jj)::value < RW - 4 || wave + 1 < n_waves) store_one(std::integral_constant<int, kAuxManyStore>{}, jj);
            });
        } else {
            static_for<0, RW>([&](auto jj) {
                if (decltype(jj)::value < RW - 4 || wave + 1 < n_waves) store_one(std::integral_constant<int, SAUX>{}, jj);
            });
        }
    };
    if constexpr (WORDS) {
        auto store_words = [&](auto kind) {
            constexpr int KIND = decltype(kind)::value;
            constexpr uint32_t SIZE = KIND == HARRIS_OUT_U8 ? 1u : 2u;
            const uint32_t columns = (uint32_t)min(max(p.m - (int)sx0, 0), (int)p.strip_pitch), tail = columns & 3u;
            const uintptr_t at = out_first + (uintptr_t)(sx0 * SIZE);
            float q_offset = p.q_offset;
            asm volatile("" : "+v"(q_offset));                  // a multiply-add takes one scalar operand
            if (lane * 4u + 4u <= columns) {
                static_for<0, RW>([&](auto jj) {
                    constexpr int j = decltype(jj)::value;
                    uintptr_t row = at + (size_t)j * out_pitch;
                    asm volatile("" : "+s"(row));               // a scalar base for the lanes' offsets
                    if (j < out_rows) store_packed<KIND>(pack_row<KIND>(results[j], p.q_scale, q_offset), row, lane_bytes);
                });
            }
            if (tail == 0u) return;
            if (lane == columns / 4u) {
                static_for<0, RW>([&](auto jj) {
                    constexpr int j = decltype(jj)::value;
                    uintptr_t row = at + (size_t)j * out_pitch;
                    asm volatile("" : "+s"(row));
                    if (j < out_rows) store_packed_tail<KIND>(pack_row<KIND>(results[j], p.q_scale, q_offset), row, lane_bytes, tail);
                });
            }
        };
        if (p.out_kind == HARRIS_OUT_U8) store_words(std::integral_constant<int, HARRIS_OUT_U8>{});
        else if (p.out_kind == HARRIS_OUT_F16) store_words(std::integral_constant<int, HARRIS_OUT_F16>{});
        else store_words(std::integral_constant<int, HARRIS_OUT_BF16>{});
    } else if (__builtin_expect(p.out_kind == HARRIS_OUT_F32, 1)) {
        store_all([&](auto aux, auto jj) {
            constexpr int j = decltype(jj)::value;
            store_row<PX, decltype(aux)::value>(results[j], out_rs[j], lane_bytes - out_skip[j]);
        });
    } else {
        // A value of its own, or the compiler makes one switch of all kinds and moves the float32 stores behind
        // the others: small launches wait for the instruction cache then (480x640 uint8 3.51 us, 3.44 without).
        unsigned kind = p.out_kind;
        asm volatile("" : "+s"(kind));
        if (kind == HARRIS_OUT_F16) {
            store_all([&](auto aux, auto jj) {
                constexpr int j = decltype(jj)::value;
                store_row_16<PX, false, decltype(aux)::value>(results[j], out_rs[j], lane_bytes - out_skip[j]);
            });
        } else if (kind == HARRIS_OUT_BF16) {
            store_all([&](auto aux, auto jj) {
                constexpr int j = decltype(jj)::value;
                store_row_16<PX, true, decltype(aux)::value>(results[j], out_rs[j], lane_bytes - out_skip[j]);
            });
        } else {
            static_for<0, RW>([&](auto jj) {
                constexpr int j = decltype(jj)::value;
                if (j < RW - 4 || wave + 1 < n_waves) store_row_8<PX, SAUX>(results[j], p.q_scale, p.q_offset, out_rs[j], lane_bytes - out_skip[j]);
            });
        }
    }
}

template <typename In, int PX, int RW, int LAUX, bool BINOM, bool HANDOFF, bool SHIFTED = false, bool SMALL = false, bool WORDS = false>
__global__ __launch_bounds__(1024) void harris_tile_kernel(const harris_launch::compact::Params args) {
    harris_tile<In, PX, RW, LAUX, BINOM, HANDOFF, SHIFTED, SMALL, WORDS>(args);
}
template <typename In, int PX, int LAUX, bool BINOM, bool SHIFTED, bool WORDS>
__global__ __launch_bounds__(1024) void harris_far_tile_kernel(const harris_launch::Params args) {
    harris_tile<In, PX, 4, LAUX, BINOM, false, SHIFTED, false, WORDS>(args);
}

}  // namespace

#endif  // HARRIS_KERNELS_H
