// Internal to libharris: what the host-side planner hands to the kernel launcher.
#ifndef HARRIS_LAUNCH_H
#define HARRIS_LAUNCH_H

#include <math.h>
#include <stddef.h>

#include "harris_tuning.h"

namespace harris_launch {

// Lanes of a 64-lane wavefront that produce result columns when each lane holds px
// columns: the remaining lane(s) only supply the 4-column halo to the right.
constexpr int valid_lanes(int px) { return 64 - (4 + px - 1) / px; }

// Division of a 32-bit unsigned number by a divisor fixed at launch, as one multiply-high, an
// addition and two shifts (Granlund and Montgomery, "Division by invariant integers using
// multiplication", 1994, the unsigned algorithm for a run-time invariant divisor): with
// l = ceil(log2 d), mul = floor(2^32 (2^l - d) / d) + 1, sh1 = min(l, 1), sh2 = max(l - 1, 0),
// floor(x / d) = (t + ((x - t) >> sh1)) >> sh2 where t = high word of mul * x.  Exact for every
// x < 2^32 and 1 <= d < 2^32.  A workgroup decomposes its index with it before its first load
// (a hardware integer division costs some 25 dependent scalar instructions).
struct FastDiv {
    unsigned mul, sh1, sh2;
};

inline FastDiv make_fastdiv(unsigned d) {
    FastDiv f;
    unsigned l = 0;
    while (l < 32 && (1ull << l) < d) ++l;
    f.mul = (unsigned)((((1ull << l) - d) << 32) / d + 1);
    f.sh1 = l < 1 ? l : 1;
    f.sh2 = l < 1 ? 0 : l - 1;
    return f;
}

#if defined(__HIPCC__)
#define HARRIS_HOST_DEVICE __host__ __device__
#else
#define HARRIS_HOST_DEVICE
#endif
HARRIS_HOST_DEVICE inline unsigned fastdiv(unsigned x, const FastDiv& f) {
    const unsigned t = (unsigned)(((unsigned long long)f.mul * x) >> 32);
    return (t + ((x - t) >> f.sh1)) >> f.sh2;
}

// Tile of workgroup (x, y) of a launch of many tiles, 8 chunk x turns workgroups: the hardware deals workgroups out
// to the eight XCDs one by one, and XCD i takes the tiles of chunks i, i + 8, i + 16, ..., `chunk` neighbouring tiles each.  All
// XCDs together then work on one stretch of the images that moves on, instead of on eight stretches far apart;
// memory serves that faster (replayed from graphs, 64 images of 1080x1920 float32: 354 us in eight stretches, 333 by turns, called one
// after the other 350 and 340; to binary16, 28 images: 155 and 137; uint8, 64 images: 177 and 160; 4320x7680: 94.6 and 88.6).  Workgroups beyond the last
// tile, at the end of the last turn, have nothing to do.
HARRIS_HOST_DEVICE inline unsigned dealt_tile(unsigned x, unsigned y, unsigned chunk) { return (y * 8u + x % 8u) * chunk + x / 8u; }

// Bit of Params::flags beside the HARRIS_TUNE_* bits: the tile kernel stores float32 and 16-bit results
// written through (kAuxManyStore in harris_kernels.h, which says where that is faster).
constexpr unsigned kWriteThrough = 0x80000000u;

// Kernel arguments (passed by value).  What the tile kernel reads before its first load sits
// together, so that a few wide scalar loads fetch it at once.
struct Params {
    const void* rgb;        // device, [batch][3][H][W] with the pitches below
    void* out;              // device, [batch][n][m] with the pitches below; element type given by out_kind
    long long in_row_pitch, in_plane_pitch, in_image_pitch;   // in input elements
    long long out_row_pitch, out_image_pitch;                 // in result elements
    int H, W;               // input rows, columns
    int n, m;               // result rows, columns (H-4, W-4)
    int rows_per_band;      // result rows per band (BANDS) or per tile (TILES)
    unsigned n_strips;      // strips per band
    unsigned strip_pitch;   // result columns per strip (a multiple of px, at most valid_lanes(px)*px; 12 less with aligned stores)
    unsigned tiles_per_image;  // n_bands * n_strips (TILES: one workgroup each)
    FastDiv by_tiles_per_image, by_n_strips;   // TILES: division by these two, where far_rows
    unsigned n_blocks;      // workgroups of the launch (the grid size)
    unsigned waves_per_block;  // wavefronts per workgroup (the block size / 64)
    float wr, wg, wb;       // float32 input: gray weights, times the Sobel scale
    float gain, more_gain;  // 8-bit input: (Sobel scale 2^18 / 255000)^4 as two factors (split_gain), the result is that multiple of what the kernel works out
    float k;                // coarsity constant
    unsigned flags;         // HARRIS_TUNE_* bits, kWriteThrough
    unsigned long long out_row_bytes, out_image_bytes;        // TILES: the result's pitches in bytes
    unsigned out_shift;     // log2 of a result element's bytes
    unsigned strip_reach;   // TILES: columns of a strip's rows that its lanes load
    unsigned out_kind;      // a harris_out_dtype (other than float32: tile kernel only)
    float q_scale, q_offset;   // 8-bit results: code = clamp(rint(fma(v, q_scale, q_offset)), 0, 255)
    int binomial;           // 1: window [1 2 1; 2 4 2; 1 2 1], 0: unweighted 3x3 sum
    unsigned lds_bytes;     // TILES: dynamic LDS per workgroup (the tile's rows, or more to bound the resident workgroups)
    int in_shifted;         // 1: 8-bit rows that start on any byte, loaded as aligned words and shifted or where they are (tile kernel, px 4)
    unsigned n_bands;       // bands (BANDS) or tiles down the image (TILES)
    unsigned blocks_x;      // BANDS: workgroups across a row of bands
    unsigned blocks_per_image;  // BANDS: workgroups per image
    // HARRIS_TUNE_PACKED_IMAGES: lanes of an image, 65536 / that rounded up, images of a wavefront, images of the call.
    // tiles_per_image is then the number of bands down the images, rows_per_band their height.
    unsigned image_lanes, image_lanes_inverse, images, batch;
    // TILES with shared rows kept, and narrow images: tiles that an XCD takes in a row, and how often.
    unsigned chunk, turns;
    int far_rows;           // TILES: 1: the rows that a wavefront loads do not lie within 2 GB (rows_are_far), compact::fits does not hold, or more_gain is not 1
    int resident;           // TILES: 1: the chip holds all tiles of the launch at once
};

// The factor of 8-bit results as two of float32, the second 1 wherever the first holds it.  Sobel scales from 4.2e9 on have factors beyond
// float32, and scales below 3.2e-10 such as it holds in fewer than 24 bits or not at all; results of the former may still be finite, and of
// the latter normal numbers.  The first factor then is 2^96 or 2^-96, which rounds nothing that the second brings back into range.  (From 2.7e67 on it is
// clamped: every result but zero is infinite then, and zero stays zero.)
inline void split_gain(double gain, float& first, float& second) {
    constexpr double kLeast = 1.17549435082228750797e-38, kMost = 3.40282346638528859812e+38, kStep = 79228162514264337593543950336.0;
    second = 1.0f;
    if ((gain >= kLeast && gain <= kMost) || gain == 0.0) { first = (float)gain; return; }
    first = gain > 1.0 ? (float)kStep : (float)(1.0 / kStep);
    const double rest = gain > 1.0 ? gain / kStep : gain * kStep;
    second = (float)(rest < kMost ? rest : kMost);
}

// 8-bit input: k times the square of a trace of scale one, up to 2^18, has to be a finite float32 before the factor is applied to it.  A k from 2^64 on
// hands its power of two to the factor; det, at most a quarter of the trace's square, is then far below the last bit of
// the result with either k.
inline void bound_k(float& k, double& gain) {
    int e;
    const double m = frexp((double)k, &e);
    if (e <= 64) return;
    k = (float)ldexp(m, 64);
    gain = ldexp(gain, e - 64);
}

// TILES: the same in 96 bytes, which is what the kernels take.  The runtime writes a launch's arguments into memory
// that the GPU reads: an empty kernel takes 2.7 to 2.9 us a launch with 88 to 112 bytes, 3.2 to 3.6 with 120 to 240 (8000 launches one after the other, six runs in three
// processes; from some host cores all are faster and 240 bytes cost 0.1 us).
// Pitches of 2^32 elements and more, result rows of 2 GB, rows that are far apart and scales whose factor takes two numbers take Params itself (compact::fits).
namespace compact {

// Division by a divisor of at most 2^31 of numbers below 2^31: floor(x mul / 2^(31 + l)) with l = ceil(log2 d) and mul = ceil(2^(31 + l) / d), which is at
// most 2^32 - 1 and off by less than d / d, so that x times the error stays below 2^(31 + l).  (Granlund and Montgomery 1994, theorem 4.2.)
inline unsigned divide_shift(unsigned d) { return d <= 1u ? 0u : 32u - (unsigned)__builtin_clz(d - 1u); }
inline unsigned divide_mul(unsigned d) { return (unsigned)(((1ull << (31 + divide_shift(d))) + d - 1) / d); }
HARRIS_HOST_DEVICE inline unsigned divide(unsigned x, unsigned mul, unsigned l) { return (unsigned)(((unsigned long long)x * mul) >> (31u + l)); }

struct Params {
    const void* rgb;
    void* out;
    unsigned in_row_bytes, out_row_bytes;
    unsigned in_plane, in_image, out_image;     // in elements
    int H, W;
    unsigned n_strips, tiles_per_image, n_blocks, chunk;
    unsigned by_tiles_per_image, by_n_strips;   // divide_mul
    float weights[3];                           // float32 input: wr, wg, wb; 8-bit input: gain
    float k, q_scale, q_offset;
    // strip_pitch 8 bits, strip_reach - strip_pitch = 4 << e: e 3, wavefronts - 1: 4, divide_shift of tiles_per_image and n_strips 5 each,
    // out_kind 2, out_shift 2, not dealt to the XCDs 1, borders moved 1, written through 1.
    unsigned bits;
};
static_assert(sizeof(Params) == 96, "more than the runtime writes quickly");

inline bool fits(const harris_layout& lay, int batch, int out_elem) {
    const long long most = 1LL << 32;
    return lay.rgb_plane_pitch < most && (batch == 1 || (lay.rgb_image_pitch < most && lay.out_image_pitch < most)) && lay.out_row_pitch < (1LL << 31) / out_elem;
}

inline Params pack(const harris_launch::Params& p, int elem) {
    Params c;
    c.rgb = p.rgb; c.out = p.out;
    c.in_row_bytes = (unsigned)(p.in_row_pitch * elem); c.out_row_bytes = (unsigned)p.out_row_bytes;
    c.in_plane = (unsigned)p.in_plane_pitch; c.in_image = (unsigned)p.in_image_pitch; c.out_image = (unsigned)p.out_image_pitch;
    c.H = p.H; c.W = p.W;
    c.n_strips = p.n_strips; c.tiles_per_image = p.tiles_per_image; c.n_blocks = p.n_blocks; c.chunk = p.chunk;
    c.by_tiles_per_image = divide_mul(p.tiles_per_image); c.by_n_strips = divide_mul(p.n_strips);
    c.weights[0] = elem == 1 ? p.gain : p.wr; c.weights[1] = p.wg; c.weights[2] = p.wb;
    c.k = p.k; c.q_scale = p.q_scale; c.q_offset = p.q_offset;
    unsigned e = 0;
    while (e < 7 && p.strip_pitch + (4u << e) < p.strip_reach) ++e;
    c.bits = p.strip_pitch | e << 8 | (p.waves_per_block - 1u) << 11 | divide_shift(p.tiles_per_image) << 15 | divide_shift(p.n_strips) << 20 |
             p.out_kind << 25 | p.out_shift << 27 | (p.flags & HARRIS_TUNE_NO_XCD_REMAP ? 1u << 29 : 0u) | (p.flags & HARRIS_TUNE_ALIGNED_STORES ? 1u << 30 : 0u) |
             (p.flags & kWriteThrough ? 1u << 31 : 0u);
    return c;
}

// What the kernel works with; `rows` result and input rows of a wavefront.
struct Tile {
    const void* rgb;
    void* out;
    unsigned long long in_row_pitch, in_plane_pitch, in_image_pitch;    // in elements
    unsigned long long out_row_bytes, out_image_bytes;
    int H, W, n, m, rows_per_band;
    unsigned n_strips, strip_pitch, strip_reach, n_blocks, chunk, waves_per_block, flags, out_kind, out_shift;
    float wr, wg, wb, gain, more_gain, k, q_scale, q_offset;
};
HARRIS_HOST_DEVICE inline Tile unpack(const Params& c, unsigned elem, int rows) {
    Tile t;
    const unsigned waves = (c.bits >> 11 & 15u) + 1u;
    t.rgb = c.rgb; t.out = c.out;
    t.in_row_pitch = c.in_row_bytes / elem; t.in_plane_pitch = c.in_plane; t.in_image_pitch = c.in_image;
    t.out_shift = c.bits >> 27 & 3u;
    t.out_row_bytes = c.out_row_bytes; t.out_image_bytes = (unsigned long long)c.out_image << t.out_shift;
    t.H = c.H; t.W = c.W; t.n = c.H - 4; t.m = c.W - 4;
    t.rows_per_band = rows * (int)waves - 4;
    t.n_strips = c.n_strips; t.n_blocks = c.n_blocks; t.chunk = c.chunk; t.waves_per_block = waves;
    t.strip_pitch = c.bits & 255u;
    t.strip_reach = t.strip_pitch + (4u << (c.bits >> 8 & 7u));
    t.flags = (c.bits >> 29 & 1u) * HARRIS_TUNE_NO_XCD_REMAP | (c.bits >> 30 & 1u) * HARRIS_TUNE_ALIGNED_STORES | (c.bits >> 31) * kWriteThrough;
    t.out_kind = c.bits >> 25 & 3u;
    t.wr = t.gain = c.weights[0]; t.wg = c.weights[1]; t.wb = c.weights[2];
    t.more_gain = 1.0f;
    t.k = c.k; t.q_scale = c.q_scale; t.q_offset = c.q_offset;
    return t;
}
HARRIS_HOST_DEVICE inline Tile unpack(const harris_launch::Params& p, unsigned, int) {
    Tile t;
    t.rgb = p.rgb; t.out = p.out;
    t.in_row_pitch = (unsigned long long)p.in_row_pitch; t.in_plane_pitch = (unsigned long long)p.in_plane_pitch; t.in_image_pitch = (unsigned long long)p.in_image_pitch;
    t.out_shift = p.out_shift; t.out_row_bytes = p.out_row_bytes; t.out_image_bytes = p.out_image_bytes;
    t.H = p.H; t.W = p.W; t.n = p.n; t.m = p.m; t.rows_per_band = p.rows_per_band;
    t.n_strips = p.n_strips; t.n_blocks = p.n_blocks; t.chunk = p.chunk; t.waves_per_block = p.waves_per_block;
    t.strip_pitch = p.strip_pitch; t.strip_reach = p.strip_reach; t.flags = p.flags; t.out_kind = p.out_kind;
    t.wr = p.wr; t.wg = p.wg; t.wb = p.wb; t.gain = p.gain; t.more_gain = p.more_gain;
    t.k = p.k; t.q_scale = p.q_scale; t.q_offset = p.q_offset;
    return t;
}
// Image of a tile, and band of a tile of an image.
HARRIS_HOST_DEVICE inline unsigned image_of(const Params& c, unsigned tile) { return divide(tile, c.by_tiles_per_image, c.bits >> 15 & 31u); }
HARRIS_HOST_DEVICE inline unsigned band_of(const Params& c, unsigned tile) { return divide(tile, c.by_n_strips, c.bits >> 20 & 31u); }
HARRIS_HOST_DEVICE inline unsigned image_of(const harris_launch::Params& p, unsigned tile) { return fastdiv(tile, p.by_tiles_per_image); }
HARRIS_HOST_DEVICE inline unsigned band_of(const harris_launch::Params& p, unsigned tile) { return fastdiv(tile, p.by_n_strips); }

}  // namespace compact

// TILES: whether a wavefront hands the one above it Sobel responses (harris_tile_kernel says when), and the bytes of LDS
// that the wavefronts of a workgroup then need: six rows of all but the first, which has a row to write to, or
// four gray rows each.
HARRIS_HOST_DEVICE constexpr bool hands_sobel(bool from_8_bit, int px) { return from_8_bit && px == 4; }
HARRIS_HOST_DEVICE constexpr unsigned tile_lds_bytes(bool from_8_bit, int px, unsigned waves) {
    return (hands_sobel(from_8_bit, px) ? 1u + (waves - 1u) * 6u : waves * 4u) * 64u * (unsigned)px * 4u;
}

// TILES: whether the rows of a wavefront lie too far apart for the 32-bit offsets from the first one's start at which the
// kernel loads them; those from 2 GB on are for lanes that load nothing.
inline bool rows_are_far(long long row_pitch, int W, int elem, int rows) {
    const long long most = 1LL << 31;
    return row_pitch > most / elem / rows || (rows - 1) * row_pitch * elem + (long long)W * elem > most;
}

// TILES: where a wavefront of `rows` rows finds them in a plane, in bytes from the start of its first one, row y (the image's last for wavefronts below it): row t at
// near_row(r, t); the rows below the image's last are that one again.  The rows of one wavefront lie within 2 GB (rows_are_far), those of a plane need
// not: 32 bits do for the former alone, and `last` counts no further.  Only from 8-bit input a plane's rows lie within 2^32 bytes too (compact::fits), and
// the image's last row does for `last` (2427 images of 32x129 21.7 us, 22.2 with the wavefront's; 480x640 3.04 / 3.06).
struct NearRows { unsigned pitch, last; };
HARRIS_HOST_DEVICE inline NearRows near_rows(int H, int y, unsigned pitch, int rows, bool from_8_bit) {
    const int below = H - 1 - y, most = from_8_bit ? 0x7fffffff : rows - 1;
    return {pitch, (unsigned)(below < most ? below : most) * pitch};
}
HARRIS_HOST_DEVICE inline unsigned near_row(const NearRows& r, int t) {
    const unsigned at = (unsigned)t * r.pitch;
    return at < r.last ? at : r.last;
}

// TILES, 8-bit rows on any byte loaded where they are: the byte of a row of W >= 4 pixels at which the lane of column
// `col` loads four, and the bits by which it shifts them down: a lane whose columns end behind the row loads the
// row's last four.  No load leaves the row.
struct ByteLane { unsigned voff, drop; };
HARRIS_HOST_DEVICE inline ByteLane byte_lane(unsigned col, unsigned W) {
    const unsigned last = W - 4u;
    return {col < last ? col : last, col > last ? 8u * ((col - last) & 3u) : 0u};
}

// HARRIS_TUNE_PACKED_IMAGES: most wavefronts of a workgroup, each with four rows; the last one only hands its
// rows on.
constexpr int kPatchWaves = 8;

// HARRIS_TUNE_PACKED_IMAGES: what one lane of a wavefront loads of a row.  Offsets and sizes are in
// bytes from the row's first element in the first of the group's `images` images; elem is the input
// element's size.
struct PatchLane {
    unsigned image;         // which image of the group this lane works on
    unsigned col;           // its first column
    bool live;              // whether there is such an image
    unsigned in_bytes;      // from the row's start in the first image to its end in the last: loads of
                            // float32 rows end there
    unsigned in_voff;       // the lane's load, of four elements
    unsigned drop;          // 8-bit input: bits by which the loaded word is shifted down
};
HARRIS_HOST_DEVICE inline PatchLane patch_lane(const Params& p, unsigned images, unsigned lane, unsigned elem) {
    PatchLane l;
    const unsigned in_image = (unsigned)(p.in_image_pitch * elem), last_col = (unsigned)p.W - 4u;
    l.image = (lane * p.image_lanes_inverse) >> 16;             // lane / image_lanes
    l.col = (lane - l.image * p.image_lanes) * 4u;
    l.live = l.image < images;
    l.in_bytes = (images - 1u) * in_image + (unsigned)p.W * elem;
    // 8-bit lanes load the row's last four bytes where they straddle its end, and the first image's where
    // they have no image: every load lies inside a row.  float32 lanes that straddle the end of a row
    // load what follows it up to in_bytes; the planner lets them where that is another row of the call.
    const unsigned col = elem == 1u && l.col > last_col ? last_col : l.col;
    const unsigned at = l.image * in_image + col * elem;        // below 2^31 for every lane (planner)
    if (elem == 1u) l.in_voff = l.live ? at : 0u;
    else l.in_voff = at | (l.live ? 0u : 0x80000000u);          // beyond in_bytes without an image; no branch
    l.drop = l.col > last_col ? 8u * ((l.col - last_col) & 3u) : 0u;
    return l;
}

// The same, dense 8-bit images whose rows start on any byte: a lane loads the two aligned words around its four pixels.  Offsets count from the aligned
// word that the group begins in, `lead` bytes before its first: the lane's column in its image's first row (the group's first without an image), row y of plane c from
// there (the image's last for rows below it), and the end of the word that holds the group's last byte, past which nothing is loaded.
// Rows that follow each other without a gap and do not all start on words, up to the widths where pairs win (us, single words /
// pairs): 528 images of 66x11 6.27 / 5.57, 2292 of 55x14 6.38 / 5.35, 3000 of 50x21 10.66 / 7.00, 3886 of 130x14 32.0 / 28.9.
// A launch of one turn, up to twice as wide: 214 of 42x46 4.39 / 4.19, 103 of 120x51 4.58 / 4.47, but 273 of 108x73 5.51 / 5.52 and
// 179 of 25x122 4.17 / 4.26.  Between the two other things bound it: 5833 of 26x27 9.11 / 9.42, 690 of 123x47 8.18 / 8.51 (larger
// launches, from 10 million pixels on, take 0.91 to 0.97 with their images in the last-level cache, 1.0 to 1.01 without).
inline bool patch_in_pairs(const Params& p) {
    const bool dense = p.in_row_pitch == p.W && p.in_plane_pitch == p.in_row_pitch * p.H && p.in_image_pitch == 3 * p.in_plane_pitch;
    const bool on_words = p.W % 4 == 0 && (size_t)p.rgb % 4 == 0;
    return dense && !on_words && p.W <= (p.turns == 1 ? 60 : 24);
}
HARRIS_HOST_DEVICE inline unsigned patch_first_byte(const Params& p, const PatchLane& l, unsigned lead) { return lead + (l.live ? l.image * (unsigned)p.in_image_pitch + l.col : 0u); }
HARRIS_HOST_DEVICE inline unsigned patch_row(const Params& p, int y, int c) { return (unsigned)(y < p.H - 1 ? y : p.H - 1) * (unsigned)p.in_row_pitch + (unsigned)c * (unsigned)p.in_plane_pitch; }
HARRIS_HOST_DEVICE inline unsigned patch_words_end(const Params& p, unsigned images, unsigned lead) { return (lead + images * (unsigned)p.in_image_pitch + 3u) & ~3u; }

// Narrow images: the arguments of their kernel, 88 bytes (namespace compact says why).  The planner keeps an image's pitch below 2^30 elements, and with it
// those of rows and planes.
namespace compact_patch {

struct Params {
    const void* rgb;
    void* out;
    unsigned in_row, in_plane, in_image, out_row, out_image;    // in elements
    int H, W;
    unsigned bands, n_blocks, chunk, batch, by_bands;           // by_bands: compact::divide_mul
    float weights[3], k;                                        // as in compact::Params
    unsigned image_lanes_inverse;
    unsigned bits;                                              // rows_per_band 5 bits, divide_shift of bands 5, image_lanes 6, images 7
};
static_assert(sizeof(Params) <= 96, "more than the runtime writes quickly");

inline Params pack(const harris_launch::Params& p, int elem) {
    Params c;
    c.rgb = p.rgb; c.out = p.out;
    c.in_row = (unsigned)p.in_row_pitch; c.in_plane = (unsigned)p.in_plane_pitch; c.in_image = (unsigned)p.in_image_pitch;
    c.out_row = (unsigned)p.out_row_pitch; c.out_image = (unsigned)p.out_image_pitch;
    c.H = p.H; c.W = p.W;
    c.bands = p.tiles_per_image; c.n_blocks = p.n_blocks; c.chunk = p.chunk; c.batch = p.batch; c.by_bands = compact::divide_mul(p.tiles_per_image);
    c.weights[0] = elem == 1 ? p.gain : p.wr; c.weights[1] = p.wg; c.weights[2] = p.wb;
    c.k = p.k;
    c.image_lanes_inverse = p.image_lanes_inverse;
    c.bits = (unsigned)p.rows_per_band | compact::divide_shift(p.tiles_per_image) << 5 | p.image_lanes << 10 | p.images << 16;
    return c;
}
HARRIS_HOST_DEVICE inline harris_launch::Params unpack(const Params& c) {
    harris_launch::Params p;
    p.rgb = c.rgb; p.out = c.out;
    p.in_row_pitch = c.in_row; p.in_plane_pitch = c.in_plane; p.in_image_pitch = c.in_image;
    p.out_row_pitch = c.out_row; p.out_image_pitch = c.out_image;
    p.H = c.H; p.W = c.W; p.n = c.H - 4; p.m = c.W - 4;
    p.rows_per_band = (int)(c.bits & 31u);
    p.tiles_per_image = c.bands; p.n_blocks = c.n_blocks; p.chunk = c.chunk; p.batch = c.batch;
    p.wr = p.gain = c.weights[0]; p.wg = c.weights[1]; p.wb = c.weights[2];
    p.k = c.k;
    p.image_lanes = c.bits >> 10 & 63u; p.images = c.bits >> 16 & 127u; p.image_lanes_inverse = c.image_lanes_inverse;
    return p;
}
HARRIS_HOST_DEVICE inline unsigned group_of(const Params& c, unsigned tile) { return compact::divide(tile, c.by_bands, c.bits >> 5 & 31u); }

}  // namespace compact_patch

// Enqueue the fused kernel.  `shape` must come from harris_plan (all fields set).
// Returns a harris_status.
int launch(const Params& p, const harris_tuning& shape, long long n_blocks, int dtype, void* stream);

// The translation units that hold the kernels: each enqueues the instance that `shape` names
// with `grid` workgroups of `block` threads and returns the hipError_t of the launch as int
// (hipErrorInvalidValue for a shape it has no kernel for).
int launch_tiles_f32(const Params& p, const harris_tuning& shape, unsigned grid, unsigned block, void* stream);
int launch_tiles_u8(const Params& p, const harris_tuning& shape, unsigned grid, unsigned block, void* stream);
int launch_tiles_f32_words(const Params& p, const harris_tuning& shape, unsigned grid, unsigned block, void* stream);   // HARRIS_TUNE_WORD_STORES
int launch_tiles_u8_words(const Params& p, const harris_tuning& shape, unsigned grid, unsigned block, void* stream);
int launch_patches(const Params& p, int dtype, unsigned block, void* stream);
int launch_bands(const Params& p, const harris_tuning& shape, int dtype, unsigned grid, unsigned block, void* stream);

// Floats of workspace the grouped (unfused) pipelines need; 0 for an unknown grouping.
size_t grouped_workspace_floats(int grouping, int batch, int H, int W);

// Whether the kernels of a grouping take four neighbouring pixels of two rows per thread, or one pixel.
// Smaller images keep one: a launch is then bound by its latency, and eight times the wavefronts hide
// more of it (the three groupings on 600x800: 43.6 us, wide 48.5; on 720x1000 55.2 and 51.5).  So do narrower
// ones: a row of 64 threads takes 256 columns when wide, and most threads of the 3x3 stages would have
// none (wide against one pixel: 16 images of 651x64 63.4 / 53.2 us, of 651x96 68.2 / 70.9, 64 of 128x128 62.5 / 66.2; with
// workgroups dealt out one by one, 8 million pixels: 64 columns 363 / 331, 96 columns 304 / 402).
inline bool grouped_wide(int batch, int H, int W) { return (long long)batch * H * W >= 5LL << 17 && W >= 96; }

// Workgroups of `each` pixels (or rows) that cover `size` of them; size + each may lie beyond int.
inline unsigned groups_covering(int size, int each) { return ((unsigned)size + (unsigned)each - 1u) / (unsigned)each; }

// How the workgroups of a grouping's launches are dealt to the XCDs (harris_grouped.hip): a run of each image to an XCD, a run
// of images, or one by one in order.  Of images with few workgroups the first starts up to seven more than needed for each (in
// order / a run of each / a run of images, the three groupings: 500 images of 40x40 67.0 / 83.8 / 64.9 us, 20000 of 8x8 189 / 977 / 168, 200 of
// 96x96 97 / 113 / 96, 1336 of 307x7, 76 workgroups, 548 / 568 / 532); the division that the second needs is waited for in large images and in small
// launches (480x640 41.5 / 37.6 / 40.5; 4 of 1080x1920 289 / 270 / 278; 16 of 651x64, 162 workgroups, 56.7 / 53.2 / 54.7; 30 of 100x200, 100, 59.5 / 55.0 /
// 55.5; images and workspace not in the last-level cache: 30 of 25x66, 180 in all, 30.4 / 30.7 / 32.5, 1284 of 6x28 uint8, 1284, 36.7 / 83 / 39.6, 299 of
// 29x70 uint8, 4186, 68.9 / 69.7 / 62.3).
enum GroupedDealing { kRunOfEach, kRunOfImages, kInOrder };
inline GroupedDealing grouped_dealing(int batch, int H, int W, bool wide) {
    const unsigned long long each = (unsigned long long)groups_covering(W - 4, wide ? 256 : 64) * groups_covering(H - 4, wide ? 8 : 4);
    if (batch == 1 || each >= 128) return kRunOfEach;
    return each * batch >= 1536 ? kRunOfImages : kInOrder;
}

// Grid of `blocks` workgroups for an image of a grouping, 8 x chunk by turns (dealt_tile): one turn, in which each XCD
// takes one run, unless the launch's x dimension would come near the 2^32 threads that a dimension may have (images of
// few columns and more than 33 million rows).
struct GroupedGrid { unsigned chunk, turns; };
inline GroupedGrid grouped_grid(unsigned long long blocks) {
    const unsigned long long most = 1ull << 23, turns = blocks > most ? (blocks + most - 1) / most : 1;
    return {(unsigned)((blocks + 8 * turns - 1) / (8 * turns)), (unsigned)turns};
}

// Enqueue grouping 1, 2 or 3 (see harris_coarsity_grouped).  Returns a harris_status.
int launch_grouped(const void* rgb, int dtype, int batch, int H, int W, float k, float sobel_scale, int binomial,
                   int grouping, float* workspace, float* out, void* stream);

// Device address, on the current device, of the library's fixed scratch array of
// HARRIS_GROUPED_SCRATCH_BYTES bytes (see harris_coarsity_grouped_static); NULL on failure.
float* scratch_of_current_device();

// Enqueue the streaming-copy probe (see harris_probe_copy).  Returns a harris_status.
int launch_copy_probe(const void* rgb, int dtype, int batch, int H, int W, float* out, void* stream);

// Enqueue a pure read or write stream (see harris_probe_stream).  Returns a harris_status.
int launch_stream_probe(int kind, const void* src, void* dst, long long bytes, void* stream);

}  // namespace harris_launch

#endif
