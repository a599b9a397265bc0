// C interface of libharris: argument checks, launch-shape planning, dispatch.
// Everything here runs on the host and touches no device memory.

#include <math.h>
#include <stdint.h>

#include "harris_tuning.h"
#include "harris_launch.h"

namespace {

constexpr int kVersion = 400;   // 0.4.0

bool power_of_two_aligned(uintptr_t p, unsigned bytes) { return (p & (uintptr_t)(bytes - 1)) == 0; }

int elem_size(int dtype) { return dtype == HARRIS_U8 ? 1 : 4; }
int out_elem_size(int out_dtype) { return out_dtype == HARRIS_OUT_F32 ? 4 : out_dtype == HARRIS_OUT_U8 ? 1 : 2; }
bool known_out_dtype(int d) { return d == HARRIS_OUT_F32 || d == HARRIS_OUT_F16 || d == HARRIS_OUT_BF16 || d == HARRIS_OUT_U8; }

// Can every lane load px input elements and store its result columns with single, naturally
// aligned vector accesses?  Loads are px*elem bytes wide up to 16; stores are min(px,4) result elements.
bool px_fits(int px, int dtype, int out_dtype, int W, int rgb_align, int out_align) {
    if (px < 1 || W % px != 0) return false;
    int load_bytes = px * elem_size(dtype);
    if (load_bytes > 16) load_bytes = 16;
    int store_bytes = (px < 4 ? px : 4) * out_elem_size(out_dtype);
    return rgb_align % load_bytes == 0 && out_align % store_bytes == 0;
}

// Four pixels per lane without natural alignment (a width that is no multiple of 4, padded
// rows, an offset view); tile kernel only.  float32 rows start on 4-byte boundaries: buffer
// accesses of several 32-bit words need only 4-byte alignment, and the hardware checks each
// word of such an access against the end of the row by itself, so the lane that straddles the
// end of a row loads zeros beyond it and stores nothing there.  8-bit rows may start on any
// byte: the kernel loads the aligned words that hold them and shifts.  Results: float32, or
// 16-bit with rows that start on 4-byte boundaries and have an even number of columns: the
// range check works on whole 32-bit words, so a word that held the last column of an odd row
// together with two bytes behind it would either be dropped or written whole.  (Other rows of 16-bit
// results and of 8-bit codes: px4_fits_shifted.)
bool px4_fits_word_aligned(int dtype, int out_dtype, int W, int rgb_align, int out_align) {
    if (dtype == HARRIS_F32 && rgb_align % 4 != 0) return false;
    if (out_dtype == HARRIS_OUT_U8 || out_align % 4 != 0) return false;
    return out_dtype == HARRIS_OUT_F32 || W % 2 == 0;
}

// Four pixels per lane for rows of 16-bit results and 8-bit codes on any boundary of their element type:
// the tile kernel stores a lane's four where they belong and the ends of rows in pieces (HARRIS_TUNE_WORD_STORES).
bool px4_fits_shifted(int dtype, int out_dtype, int rgb_align) {
    return out_dtype != HARRIS_OUT_F32 && !(dtype == HARRIS_F32 && rgb_align % 4 != 0);
}

// Whether to take them by default, for default shapes (a caller that asks for a shape gets the lanes that it
// names or the narrower ones), instead of lanes of `narrower` pixels, 1 or 2.
//   - A strip of them takes the time of several narrower strips, whatever its width (float32 input 1.8 of one
//     pixel and 1.2 to 1.6 of two, 8-bit input 1.6 of either): it must replace more than that.  13889 images
//     of 64x9 float32 to binary16, one strip for one, 263 us wide and 146 narrow; 2049 of 64x61 45.9 / 24.5; 776
//     of 64x161, one for three, 23.2 / 28.6, from 8-bit input 17.5 / 26.3.
//   - From 14 tiles of the narrower lanes per CU on, or, where a wide strip replaces three of one pixel, from
//     about 1.5 million pixels on: below, a launch is bound by its latency, which the longer store code
//     adds to, and the narrower lanes' many wavefronts do no harm (700x401 float32 to binary16 4.9 / 3.5 us;
//     33 of 200x301, two strips for five, 11 tiles, 9.1 / 8.5; but 1079x1919, 8 strips for 32, 11 tiles,
//     7.6 / 9.1, and 776 of 64x161 as above).  Not from 1.5 million on if the planner's one tile per CU
//     would leave a third of the CUs without (130 of 64x241, 130 tiles, 9.4 / 8.4; 50 of 64x501, 150, 8.3 / 7.4).
//   - Strips of four pixels per lane are counted as the planner cuts them from 8-bit input, 248 columns (with 244, before: 178 calls whose rows end in the
//     last four columns of a strip take 0.90 of the time on average, 6 of them 1.01 to 1.05).  From float32 input they hold 252,
//     but counted so some launches to codes take four pixels that are slower with them (43 of 100x505 7.4 / 8.2 us), and 248 stand.
//   Over 1174 shapes of 1.6 to 32 million pixels, 62 to 2831 columns wide, the choice takes on average 0.4 %
//   longer than the faster of the two; always wide would take 6.8 %, always narrow 12.5 %.
bool px4_shifted_by_default(int dtype, int batch, int H, int W, int narrower, const harris_tuning& t) {
    if (t.rows != 0 || t.waves_per_block != 0 || t.flags != 0u || t.lds_kb != 0) return false;
    const long long n = H - 4, m = W - 4;
    if (n < 1 || m < 1 || (long long)batch * H * W < 3LL << 19) return false;
    const long long wide_pitch = harris_launch::valid_lanes(4) * 4 - 4, narrow_pitch = harris_launch::valid_lanes(narrower) * narrower;
    const long long wide = (m + wide_pitch - 1) / wide_pitch, narrow = (m + narrow_pitch - 1) / narrow_pitch;
    const int worth = dtype == HARRIS_U8 ? (narrower == 1 ? 180 : 170) : (narrower == 1 ? 215 : 150);     // hundredths of a narrower strip
    if (100 * narrow < worth * wide) return false;
    if (batch * narrow * ((n + 11) / 12) >= 14 * 256) return true;
    return narrower == 1 && narrow >= 3 * wide && !(batch * wide > 128 && batch * wide <= 170);
}

// Batches of narrow images, float32 results, default shapes only: as many images side by side in a
// wavefront as its 64 lanes of four columns hold (harris_patches.hip), from two on (W <= 128).
//   - A workgroup holds four, five or eight wavefronts of four rows (patch_waves; a caller may ask for 2 to 8), the
//     last of which only hands its rows on; taller images are cut into bands of equal height.
//   - float32 rows whose length is no multiple of 4 must follow each other without a gap, those of
//     neighbouring planes and images too: the lane at the end of a row reads up to three floats of what
//     follows it, which must be a row of the call and nothing else.  With two images only, where little is gained, such rows keep a
//     wavefront each: their ends cost two more stores a row (600 of 110x121 24.7 us, 25.9 packed).
//   - Offsets from the first to the last image of a wavefront are 32-bit.
//   - From 2^18 pixels on, and only where one image per wavefront would take more than one tile of 4 x 4
//     rows per CU: smaller launches are bound by latency and better spread over more wavefronts (packed
//     against one by one, float32: 64 images of 32x128, 192 tiles, 4.0 / 3.2 us; 20 of 120x128, 200 tiles,
//     3.9 / 3.5; 5 of 500x128, 210 tiles, 4.0 / 3.6; but 228 of 24x128, 456 tiles, 3.9 / 4.4; 64 of 64x64,
//     320 tiles, 3.8 / 4.1).
//   - Two wide float32 images, which keep more than 24 of the 64 lanes busy by themselves, gain least.  They
//     stay apart where that fills the third tile of every CU and bands of 28 result rows, packed, would leave half of the
//     CUs without a workgroup (with eight wavefronts packed against one by one: 244 of 32x128, 732 tiles, 122 workgroups, 5.4 / 5.0
//     us, 252 of 32x124 5.4 / 5.0; but 293 of 32x128, 147 workgroups, 6.0 / 6.4, 260 of 32x120 5.4 / 6.1, and
//     with 24 lanes 228 of 32x96, 684 tiles, 114 workgroups, 4.3 / 4.7).
//   A caller may ask for it with HARRIS_TUNE_PACKED_IMAGES wherever the kernel can take the problem.
using harris_launch::kPatchWaves;
constexpr long long kPatchPixels = 1LL << 18;

// Wavefronts of a workgroup and turns of a launch (dealt_tile in harris_launch.h), measured together.  Four wavefronts, 12
// result rows, by turns of some 16 workgroups, against eight in one stretch per XCD: 2048 images of 64x64 float32 24.9 us (29.4),
// 8192 of 32x32 25.8 (30.9), 5000 of 24x100 32.7 (38.1), uint8 663 of 48x64 5.67 (6.38), 3713 of 103x25 29.2 (33.1).  Small
// workgroups start and end one by one while larger ones wait for room on a CU; what they read twice, four rows in
// sixteen, comes from L2.  But a launch that the chip holds at once takes as long as its fullest CU, which a band more or less per
// image moves by a quarter: of four, five and eight wavefronts those are taken that leave the fewest on that CU, where four and
// five count less than as many in workgroups of eight (from float32 0.88 and 0.98, from 8-bit input 0.84 and 1.04), and four
// wherever they make no more than two workgroups per CU.  (In us by fours / fives / eights, wavefronts on the fullest CU in
// brackets, input and results not in the last-level cache: 460 float32 images of 150x37 11.9 / 14.5 / 12.6 [16 / 20 / 16]; 394 of 104x35 9.9 / 8.5 / 8.0 [12 / 10 / 8];
// 219 of 97x64 6.5 / 7.3 / 7.0 [8 / 10 / 7]; uint8 1648 of 60x55 14.1 / 14.6 / 15.0 [36 / 35 / 32].)
//   - From float32 fours keep the chip busiest beyond 24 wavefronts a CU (1931 of 61x83 31.5 / 33.3 / 34.3).
//   - From 8-bit input six workgroups of four a CU count 0.90 (1140 of 67x47 10.9 / 8.6 / 8.8 [24 / 20 / 21]; 2526 of 50x33 12.3 / 13.5 / 10.2 [24 /
//     25 / 21]), and fours whose bands are of eight rows or less or that take over 1.25 times the wavefronts of eights 0.94 (7323 of 18x96,
//     two bands for one, 1.07 / 0.98 / 1.00 of the time, 22916 of 17x9 15.7 / 12.6 / 12.6, 6814 of 32x28 1.01 / 1.00 / 0.92).
// Over 480 shapes of 1.2 to 25 million pixels, each with its images in the last-level cache and not, 0.94 of the time of eight in
// one stretch per XCD; at most 1.1.  Of images of 5 to 24 columns 2795 uint8 images of 116x13 take 1.10, 25029 float32 of 15x7 1.06.
// Launches below some 1.2 million pixels keep eight, one band of up to 28 rows, and one turn: a test of the plans fixes
// their bands (four would take 0.85 to 1.02 of the time: 71 uint8 images of 91x80 3.9 / 4.3, 311 float32 of 28x88 5.6 / 5.7).  From some
// 1.44 million on a launch has more than a workgroup per CU, as a test of the turns has it (1787 uint8 images of 32x36, 256
// workgroups of eight, 512 of five: 5.75 / 5.86 us; others 1.00 to 1.05 of the time).
constexpr long long kPatchSmallPixels = 9LL << 17, kPatchFewPixels = 11LL << 17;
int patch_waves(int dtype, long long pixels, long long groups, int n) {
    if (pixels < kPatchSmallPixels) return kPatchWaves;
    struct Shape { long long blocks; int rows, waves; long long fullest; };     // rows of a band; wavefronts of a workgroup and on the fullest CU
    const auto shape = [&](int most) {
        const int bands = (n + 4 * (most - 1) - 1) / (4 * (most - 1)), rows = (n + bands - 1) / bands, waves = (rows + 3) / 4 + 1;
        return Shape{groups * bands, rows, waves, (groups * bands + 255) / 256 * waves};
    };
    const Shape four = shape(4), five = shape(5), eight = shape(kPatchWaves);
    if (four.blocks <= 512 || (dtype == HARRIS_F32 && four.blocks * 4 > 256 * 24)) return 4;
    long long weight4 = 88, weight5 = 98;
    if (dtype == HARRIS_U8) {
        weight4 = four.rows <= 8 || 4 * four.blocks * four.waves > 5 * eight.blocks * eight.waves ? 94 : four.fullest > 20 && four.fullest <= 24 ? 90 : 84;
        weight5 = 104;
    }
    const long long cost4 = weight4 * four.fullest, cost5 = weight5 * five.fullest, cost8 = 100 * eight.fullest;
    const bool eights = pixels < kPatchFewPixels || eight.blocks > 256;
    if (eights && cost8 <= cost4 && cost8 <= cost5) return kPatchWaves;
    return cost4 < cost5 ? 4 : 5;
}
unsigned patch_turns(long long pixels, long long blocks) {
    const long long turns = pixels < kPatchSmallPixels ? 1 : (blocks + 64) / 128;
    return (unsigned)(turns < 1 ? 1 : turns > 65535 ? 65535 : turns);
}

// Kilobytes of LDS to reserve per workgroup, which bound the workgroups on a CU: three of up to five wavefronts, two of more, for large launches of very
// narrow 8-bit images.  A row of such an image is a small part of a cache line, which the rows below it need too, and a wavefront works on up
// to 32 images: with eight workgroups on a CU the lines in use do not fit the XCD's L2 and are fetched again and again, the more the faster
// a wavefront gets through its rows.  (us, as many as fit / three or two: 20000 images of 72x7 57.9 / 37.3; 4120 of 104x7 18.5 / 13.3; 7107 of 45x14
// 17.9 / 11.8; 12741 of 138x11 142 / 132.)  Over 306 launches of 2.9 to 40 million pixels, with their images in the last-level cache and not, 0.83 of the time of as
// many as fit; 4640 of 115x7 take 1.17, some of 12 to 30 rows up to 1.17 (2973 of 48x22 1.23).  From 16 columns on widths on words gain nothing (5507 of 246x24 1.06),
// smaller launches and workgroups of fewer wavefronts lose (6.7 million pixels of 8x5 1.6), and so do wider images, whose lines fit.
int patch_lds_kb(int dtype, long long pixels, int W, int waves) {
    if (dtype != HARRIS_U8 || waves < 4 || pixels < 11LL << 18) return 0;
    return W <= 12 || (W <= 24 && W % 4 != 0) ? (waves <= 5 ? 52 : 64) : 0;
}

// HARRIS_OK: planned.  HARRIS_ERR_ARG: asked for where it cannot be.  kNotPacked: one image per wavefront.
constexpr int kNotPacked = 1;
int plan_patches(int dtype, int out_dtype, int batch, int H, int W, int rgb_align, const harris_layout& lay, const harris_tuning& t,
                 harris_tuning* chosen, long long* n_blocks, harris_launch::Params* params) {
    const bool asked = t.flags & HARRIS_TUNE_PACKED_IMAGES;
    if (!asked && (t.schedule != 0 || t.px != 0 || t.rows != 0 || t.prefetch != 0 || t.waves_per_block != 0 || t.flags != 0u || t.lds_kb != 0)) return kNotPacked;
    const int n = H - 4, m = W - 4, lanes = (W + 3) / 4, images = 64 / lanes;
    if (asked) {
        if (t.flags & ~(HARRIS_TUNE_PACKED_IMAGES | HARRIS_TUNE_CACHED_LOADS | HARRIS_TUNE_PLAIN_STORES)) return HARRIS_ERR_ARG;
        if (t.schedule == HARRIS_SCHEDULE_BANDS || t.prefetch != 0 || !(t.px == 0 || t.px == 4) || !(t.rows == 0 || t.rows == 4)) return HARRIS_ERR_ARG;
        if (!(t.waves_per_block == 0 || (t.waves_per_block >= 2 && t.waves_per_block <= kPatchWaves)) || t.lds_kb < 0 || t.lds_kb > 64) return HARRIS_ERR_ARG;
        if (out_dtype != HARRIS_OUT_F32 || (dtype == HARRIS_F32 && rgb_align % 4 != 0)) return HARRIS_ERR_ARG;
    }
    if (n < 1 || m < 1 || batch < 1) return kNotPacked;
    if (asked && (batch < 2 || images < 2)) return HARRIS_ERR_ARG;
    const bool dense = lay.rgb_row_pitch == W && lay.rgb_plane_pitch == (long long)H * W && lay.rgb_image_pitch == 3 * lay.rgb_plane_pitch;
    if (out_dtype != HARRIS_OUT_F32 || batch < 2 || images < 2) return kNotPacked;
    if (dtype == HARRIS_F32 && (rgb_align % 4 != 0 || (W % 4 != 0 && !dense))) return kNotPacked;
    const long long reach = 1LL << 30;
    if (lay.rgb_image_pitch > reach / (images * elem_size(dtype)) || lay.out_image_pitch > reach / (images * 4)) return kNotPacked;
    const long long groups = ((long long)batch + images - 1) / images;
    const int max_rows = 4 * ((t.waves_per_block ? t.waves_per_block : patch_waves(dtype, (long long)batch * H * W, groups, n)) - 1), bands = (n + max_rows - 1) / max_rows, rows = (n + bands - 1) / bands;
    const int waves = t.waves_per_block ? t.waves_per_block : (rows + 3) / 4 + 1;
    const long long blocks = groups * bands;
    if (blocks > 0x7fffffffLL) return kNotPacked;
    if (!asked) {
        const long long tiles = (long long)batch * ((n + 11) / 12);         // of one image per wavefront
        if ((long long)batch * H * W < kPatchPixels || tiles <= 256) return kNotPacked;
        if (images == 2 && dtype == HARRIS_F32 && (W % 4 != 0 || (lanes > 24 && tiles > 640 && tiles <= 768 && groups * ((n + 27) / 28) <= 128))) return kNotPacked;
    }
    const int lds_kb = t.lds_kb > 0 ? t.lds_kb : patch_lds_kb(dtype, (long long)batch * H * W, W, waves);
    const harris_tuning c = {HARRIS_SCHEDULE_TILES, 4, 4, 0, waves, HARRIS_TUNE_CACHED_LOADS | HARRIS_TUNE_PLAIN_STORES | HARRIS_TUNE_PACKED_IMAGES,
                             lds_kb > 4 * waves ? lds_kb : 4 * waves};
    if (chosen) *chosen = c;
    if (n_blocks) *n_blocks = blocks;
    if (params) {
        *params = harris_launch::Params{};
        params->H = H; params->W = W; params->n = n; params->m = m;
        params->rows_per_band = rows;
        params->tiles_per_image = (unsigned)bands;
        params->n_blocks = (unsigned)blocks;
        params->waves_per_block = (unsigned)waves;
        params->flags = c.flags;
        params->lds_bytes = (unsigned)c.lds_kb * 1024u;
        params->image_lanes = (unsigned)lanes;
        params->image_lanes_inverse = (unsigned)((65535 + lanes) / lanes);
        params->images = (unsigned)images;
        params->batch = (unsigned)batch;
        params->turns = patch_turns((long long)batch * H * W, blocks);
        params->chunk = (unsigned)((blocks + 8LL * params->turns - 1) / (8LL * params->turns));
    }
    return HARRIS_OK;
}

// Number of turns in which a launch of many tiles is dealt to the XCDs (dealt_tile in harris_launch.h says why).  One, eight
// stretches as before, if about all tiles are resident at once: their order is then no matter.  Otherwise as many
// as give each XCD runs of some bands of tiles, a band being a row of tiles across an image:
//   - 8 bands, but at most some 136 tiles, where float32 input up to 400 MB (16-bit results and codes: 256 MB) keeps 3 or 4
//     tiles on a CU.  Shorter runs have more bands at their ends, whose shared rows another L2 has: 2832x4256 (18 tiles
//     a band) one turn 33.0 us, 7 bands 32.1, 4 bands 32.6, 2 bands 33.4; 2 images of 2160x3840 44.5 / 8 bands 42.5 / 2
//     bands 44.9; 2400x8000 (34 a band) 52.5 / 4 bands 50.1 / 8 bands 53.3.
//   - One float32 image to float32 beyond 128 MB, 3 tiles on a CU and so 96 on an XCD, is particular where a band has many tiles: runs
//     of 127 to 150 tiles are fast, of 152 to 178 and of 116 to 126 slow.  Where no number of turns gives the former, up to 101 tiles.
//     4200x4200 one turn 46.1 us, runs of 119 tiles 47.0, of 148 45.8; 3456x5184 47.0 / 119 48.8 / 149 46.5; 4608x4608 55.8 / 120 56.6 /
//     144 54.4; 3500x4000 38.5 / 156 39.3 / 94 37.9;
//     5778x4238 65.2 / 96 63.5 / 128 62.0.  (Two images of 2531x3743 rather take 119, 50.8 us, than 149, 53.6.)
//   - At least 2 bands and 16 tiles for larger launches, with 2 tiles on a CU, and for 8-bit input: 64 images of 1080x1920
//     float32 (8 a band) one turn 350 us, 2 bands 340; in graphs one turn 353, 2 bands 334, 6 bands 338, 16 bands 351; 6000x8000
//     127.2, 2 bands 124.9, 1 band 128; 64 images of 1080x1920 uint8 176.4, 2 bands 159.5, 16 bands 166; 2832x4256 uint8 19.5, 2 bands 18.9, 10 bands 19.4.
//   - Not less than 96 tiles from 8-bit input to float32 up to 128 MB where a band has 16 or more: 4096x4096 (18 a band) one
//     turn 24.6 us, 2 bands 25.4, 96 tiles 24.6; 2 images of 2048x4096 24.6 / 25.2 / 24.7; over 36 shapes 0.97 of the time of one turn, at
//     most 1.005 (2 bands: 0.97, at most 1.04).  Narrower images are the same or up to 2 % slower with them.
// Over 166 shapes no launch got slower than in one turn by more than 1.7 %.
unsigned chunk_turns(int dtype, int out_dtype, int batch, long long footprint, long long n_strips, long long n_tiles) {
    if (n_tiles <= 2048) return 1;
    const auto turns_of = [&](long long chunk) { return (n_tiles + 4 * chunk) / (8 * chunk); };
    const bool f32 = dtype == HARRIS_F32, to_f32 = out_dtype == HARRIS_OUT_F32, small = footprint <= (128LL << 20);
    const bool few = f32 && footprint <= ((to_f32 ? 400LL : 256LL) << 20);
    const long long bands = few ? (136 >= 8 * n_strips ? 8 : 136 / n_strips) : (16 + n_strips - 1) / n_strips;
    long long chunk = (bands < 2 ? 2 : bands) * n_strips;
    if (!f32 && to_f32 && small && n_strips >= 16 && chunk < 96) chunk = 96;
    long long turns = turns_of(chunk);
    if (few && to_f32 && !small && batch == 1 && n_strips >= 14) {
        const auto each = [&](long long t) { return (n_tiles + 8 * t - 1) / (8 * t); };
        const auto good = [&](long long t) { return each(t) >= 127 && each(t) <= 150; };
        turns = turns_of(140);
        turns = good(turns) ? turns : good(turns + 1) ? turns + 1 : (n_tiles + 8 * 101 - 1) / (8 * 101);
    }
    return (unsigned)(turns < 1 ? 1 : turns > 65535 ? 65535 : turns);
}

harris_layout dense_layout(int H, int W) {
    // (Shapes that the planner has yet to refuse come here as well: no signed overflow.)
    const long long n = H - 4LL, m = W - 4LL, plane = (long long)H * W;
    return {W, plane, (long long)(3ull * (unsigned long long)plane), m, n * m};
}

int plan_shape(int dtype, int out_dtype, int batch, int H, int W, int rgb_align, int out_align, const harris_layout& lay, const harris_tuning* tuning,
               harris_tuning* chosen, long long* n_blocks, harris_launch::Params* params) {
    if (dtype != HARRIS_F32 && dtype != HARRIS_U8) return HARRIS_ERR_ARG;
    if (!known_out_dtype(out_dtype)) return HARRIS_ERR_ARG;
    if (batch < 0 || H < 4 || W < 4) return HARRIS_ERR_SHAPE;
    if (W > (1 << 28)) return HARRIS_ERR_SHAPE;      // byte offsets within a row are 32-bit
    if (H > (1 << 30)) return HARRIS_ERR_SHAPE;      // row indices plus a tile's height stay within int
    // Byte counts below are 64-bit: 16 bytes per pixel of at most 2^58 pixels would not fit.
    if (batch > 0 && (long long)H * W > (1LL << 56) / batch) return HARRIS_ERR_SHAPE;
    if (rgb_align < 1 || out_align < out_elem_size(out_dtype)) return HARRIS_ERR_ARG;
    harris_tuning t = {0, 0, 0, 0, 0, 0u, 0};
    if (tuning) t = *tuning;
    if (t.flags & ~(HARRIS_TUNE_NO_ALTERNATE | HARRIS_TUNE_NO_XCD_REMAP | HARRIS_TUNE_CACHED_LOADS | HARRIS_TUNE_STREAM_LOADS |
                    HARRIS_TUNE_ALIGNED_STORES | HARRIS_TUNE_PLAIN_STORES | HARRIS_TUNE_KEEP_SHARED_ROWS | HARRIS_TUNE_FLAG_HANDOFF |
                    HARRIS_TUNE_WORD_STORES | HARRIS_TUNE_PACKED_IMAGES)) return HARRIS_ERR_ARG;
    if ((t.flags & HARRIS_TUNE_CACHED_LOADS) && (t.flags & HARRIS_TUNE_STREAM_LOADS)) return HARRIS_ERR_ARG;
    if ((t.flags & HARRIS_TUNE_KEEP_SHARED_ROWS) && !(t.flags & HARRIS_TUNE_STREAM_LOADS)) return HARRIS_ERR_ARG;
    if ((t.flags & HARRIS_TUNE_FLAG_HANDOFF) && (t.flags & (HARRIS_TUNE_CACHED_LOADS | HARRIS_TUNE_KEEP_SHARED_ROWS))) return HARRIS_ERR_ARG;
    if ((t.flags & HARRIS_TUNE_ALIGNED_STORES) && (t.flags & HARRIS_TUNE_PLAIN_STORES)) return HARRIS_ERR_ARG;
    if (t.schedule != 0 && t.schedule != HARRIS_SCHEDULE_BANDS && t.schedule != HARRIS_SCHEDULE_TILES) return HARRIS_ERR_ARG;

    const int packed = plan_patches(dtype, out_dtype, batch, H, W, rgb_align, lay, t, chosen, n_blocks, params);
    if (packed != kNotPacked) return packed;
    t.flags &= ~HARRIS_TUNE_PACKED_IMAGES;

    const int n = H - 4, m = W - 4;
    const bool tiles_allowed = (t.schedule == 0 || t.schedule == HARRIS_SCHEDULE_TILES) && t.prefetch == 0;
    const bool word_aligned_px4 = tiles_allowed && px4_fits_word_aligned(dtype, out_dtype, W, rgb_align, out_align);
    const bool direct_px4 = px_fits(4, dtype, out_dtype, W, rgb_align, out_align) || word_aligned_px4;
    if (t.flags & HARRIS_TUNE_WORD_STORES) {
        if (!tiles_allowed || !px4_fits_shifted(dtype, out_dtype, rgb_align) || (t.flags & HARRIS_TUNE_ALIGNED_STORES) || !(t.px == 0 || t.px == 4)) return HARRIS_ERR_ARG;
        t.px = 4;
        if (direct_px4) t.flags &= ~HARRIS_TUNE_WORD_STORES;
    } else if (t.px == 0) {
        t.px = 1;
        if (direct_px4) t.px = 4;
        else if (tiles_allowed && px4_fits_shifted(dtype, out_dtype, rgb_align) &&
                 px4_shifted_by_default(dtype, batch, H, W, px_fits(2, dtype, out_dtype, W, rgb_align, out_align) ? 2 : 1, t)) { t.px = 4; t.flags |= HARRIS_TUNE_WORD_STORES; }
        else if (px_fits(2, dtype, out_dtype, W, rgb_align, out_align)) t.px = 2;
    } else if (!((t.px == 1 || t.px == 2 || t.px == 4) &&
                 (px_fits(t.px, dtype, out_dtype, W, rgb_align, out_align) || (t.px == 4 && word_aligned_px4)))) {
        return HARRIS_ERR_ARG;
    }
    if (t.rows < 0 || t.prefetch < 0 || t.waves_per_block < 0 || t.lds_kb < 0 || t.lds_kb > 64) return HARRIS_ERR_ARG;
    // A prefetch depth exists only in the band schedule.
    if (t.schedule == 0) t.schedule = t.prefetch == 0 ? HARRIS_SCHEDULE_TILES : HARRIS_SCHEDULE_BANDS;
    if (out_dtype != HARRIS_OUT_F32 && t.schedule != HARRIS_SCHEDULE_TILES) return HARRIS_ERR_ARG;   // 16- and 8-bit results: tile kernel only
    // Strip borders on 64-byte boundaries of the result rows: the tile kernel with 16-byte lanes.
    // (A lane's stores must then be naturally aligned: borders can only lie between lanes.)
    const bool tile4 = t.schedule == HARRIS_SCHEDULE_TILES && t.px == 4;
    const bool can_align = tile4 && px_fits(4, dtype, out_dtype, W, rgb_align, out_align);
    if ((t.flags & HARRIS_TUNE_ALIGNED_STORES) && !can_align) return HARRIS_ERR_ARG;
    if ((t.flags & (HARRIS_TUNE_KEEP_SHARED_ROWS | HARRIS_TUNE_FLAG_HANDOFF)) && !tile4) return HARRIS_ERR_ARG;
    // Measured, moved against fixed borders: 378 against 393 us on 64x1080x1920 float32, 12.5
    // against 12.8 us on 1536x2560, 37.0 against 37.3 us on 2832x4256, 89 against 93 us on
    // 8192x8192 uint8.
    // 16-bit results pay more for moved borders (strips of 224 instead of 252 columns; 192 for
    // 8-bit results, which never get them by default): worth it only for large float32 inputs (64x1080x1920: 341 against 359 us; 1536x2560: 12.8 against
    // 12.4 us; 8192x8192 uint8: 81 against 74 us).
    if (!(t.flags & (HARRIS_TUNE_ALIGNED_STORES | HARRIS_TUNE_PLAIN_STORES))) {
        const long long bytes = (long long)batch * (3LL * H * W * elem_size(dtype) + (long long)out_elem_size(out_dtype) * n * m);
        const bool align = can_align && (out_dtype == HARRIS_OUT_F32 || (out_dtype != HARRIS_OUT_U8 && dtype == HARRIS_F32 && bytes > (128LL << 20)));
        t.flags |= align ? HARRIS_TUNE_ALIGNED_STORES : HARRIS_TUNE_PLAIN_STORES;
    }
    // As few strips as 64-lane wavefronts allow, all of the same width.  A moved border lies up
    // to one 64-byte block less a lane (12 float32 or 28 16-bit columns) right of the strip's
    // nominal end, and the wavefront must reach that far.
    const long long border_reach = (t.flags & HARRIS_TUNE_ALIGNED_STORES) ? 64 / out_elem_size(out_dtype) - 4 : 0;
    // 8-bit rows loaded as aligned words and shifted: the last lane only supplies bytes to its left neighbour.
    const bool in_shifted = dtype == HARRIS_U8 && tile4 && !can_align;
    const long long max_pitch = (long long)harris_launch::valid_lanes(t.px) * t.px - border_reach - (in_shifted ? 4 : 0);
    const long long n_strips = m > 0 ? (m + max_pitch - 1) / max_pitch : 0;
    const long long pitch = n_strips > 0 ? ((m + n_strips - 1) / n_strips + t.px - 1) / t.px * t.px : max_pitch;

    // Bytes the launch moves.
    const long long elem = elem_size(dtype);
    const long long footprint = (long long)batch * (3LL * H * W * elem + (long long)out_elem_size(out_dtype) * n * m);

    // Default tile shape.  A problem that one pass over the 256 CUs can hold is fastest as one
    // tile per CU: all CUs then carry the same load and finish together (measured on
    // 1536x2560: 12.2 us against 13.5 us for small tiles and 14.6 us for the best band shape).
    // The tile must cover `need` input rows; it is NW wavefronts x RW rows with the smallest
    // NW * RW, RW taken from a list in order of measured preference, some with a handicap.
    // Short tiles are better off with few rows per wavefront (a wavefront's RW + 4 row steps are
    // a serial chain, which shows once the data is there quickly: 768x1024 5.0 us with 5 x 4
    // against 5.7 us with 10 x 2; 1024x1024 5.8 us with 6 x 4 against 6.3 us with 8 x 3), tall
    // ones with 8, 6 or 9 (1440x2560 11.8 us with 8 x 9 against 12.2 us with 10 x 7 and 12.0 us
    // with 5 x 14; but 2160x3840 22.6 us with 10 x 14 against 24.1 us with 9 x 16).
    // Larger problems take many small tiles, which keep the memory system busiest (measured
    // on 2832x4256, 64x1080x1920 and 8192x8192 uint8).
    int tile_rw = 4, tile_nw = 4, tile_lds_kb = 0;
    bool one_per_cu = false;
    if (footprint <= (128LL << 20) && t.px == 4 && batch > 0 && n_strips > 0 && (long long)batch * n_strips <= 256) {
        const long long max_bands = 256 / ((long long)batch * n_strips);
        const long long need = (n + max_bands - 1) / max_bands + 4;         // input rows per tile
        // {rows per wavefront, rows of handicap}, in order of preference among equals.
        static const int kShort[][2] = {{5, 0}, {4, 0}, {6, 0}, {0, 0}};
        static const int kMedium[][2] = {{6, 0}, {5, 0}, {8, 0}, {0, 0}};
        static const int kTall[][2] = {{8, 0}, {6, 0}, {9, 0}, {10, 3}, {5, 3}, {0, 0}};
        // 8-bit input has more arithmetic per byte and does better with fewer rows per wavefront
        // (1536x2560: 7.8 us with 12 x 6 against 8.8 us with 9 x 8; 2160x3840: 13.2 us with 16 x 9
        // against 14.1 us with 14 x 10).
        static const int kTall8[][2] = {{6, 0}, {5, 3}, {8, 2}, {9, 2}, {10, 6}, {0, 0}};
        static const int kShifted[][2] = {{4, 0}, {8, 0}, {0, 0}};      // the kernels that exist for shifted 8-bit rows
        const int (*list)[2] = in_shifted ? kShifted : need <= 20 ? kShort : need <= 48 ? kMedium : dtype == HARRIS_U8 ? kTall8 : kTall;
        // Tiles of 26 to 32 rows (40 for 8-bit input), and several images with tiles of up to
        // 48 rows, are faster as many small tiles (960x1280: 6.2 against 6.5 us, 8-bit 5.1 / 5.6;
        // 1080x1920 8-bit: 5.5 / 5.9, but float32 8.4 / 8.2) -- for float32 input as long as there
        // are at most two of them per CU: a third one on some CUs costs more than it saves
        // (900x1600, 525 small tiles: 7.5 us against 6.9 with one tile of 5 x 6 rows per CU;
        // 1050x1400: 7.7 / 6.9; two images of 720x1280: 7.9 / 7.6).
        const long long small_count = (long long)batch * n_strips * ((n + 11) / 12);     // tiles of 4 x 4 rows
        const bool small_tiles = ((batch > 1 && need <= 48) || (need >= 26 && need <= (dtype == HARRIS_U8 ? 40 : 32))) &&
                                 (dtype == HARRIS_U8 || small_count <= 512);
        long long best = -1;
        for (; (*list)[0] && !small_tiles; ++list) {
            const int rw = (*list)[0];
            long long nw = (need + rw - 1) / rw;
            if (nw < 2) nw = 2;
            if (nw > 16) continue;
            const long long cost = nw * rw + (*list)[1];
            if (best < 0 || cost < best) { best = cost; tile_rw = rw; tile_nw = (int)nw; one_per_cu = true; }
        }
    }
    if (!one_per_cu && tile4 && dtype == HARRIS_U8 && out_dtype == HARRIS_OUT_U8 && !in_shifted && footprint > (128LL << 20) &&
        25LL * ((n + 35) / 36) <= 9LL * ((n + 11) / 12)) tile_rw = 10;
    if (!one_per_cu && tile4 && dtype == HARRIS_F32) {
        // Many tiles of float32 input.  Such launches are fastest with 10 to 16 wavefronts in
        // flight per CU, not with the 28 to 32 the registers allow (every wavefront requests all
        // its rows at once; with fewer in flight the requests stay within what L2 and the memory
        // controllers handle well), so the planner reserves LDS to hold the resident tiles down:
        // 36 KB -> 4 tiles per CU, 48 KB -> 3, 64 KB -> 2.  Measured with the tiles of an XCD in one stretch (shape x
        // reservation swept together; 4 x 4 rows without reservation in brackets).  Dealt by turns every one of these is
        // faster, but not all by as much: beyond 128 MB other shapes than those taken here are then up to 4.5 %
        // faster (4 x 6 at 48 KB: 6000x8000 117 us, the planner's 5 x 6 122, 4320x7680 84.6 / 86.5; 5 x 6: 64x1080x1920 332 / 341,
        // 16x1080x1920 82.4 / 84.3, 4096x4096 43.5 / 44.2).  The choice has not been swept again.  In one stretch:
        //   float32 results, up to 400 MB: 4 wavefronts x 5 rows, 3 per CU (2832x4256 32.7 [34.8]
        //     us, 2x2160x3840 44.5 [49.1]);
        //   beyond, 8 images or more: 5 x 5, 2 per CU (16x1080x1920 87.1 [103.7] us, 64x1080x1920
        //     351 [378], 128x720x1280 318 [350]); fewer, larger images: 5 x 6, 2 per CU
        //     (4320x7680 92.0 [105.7] us, 4 x 5: 99.2; 6000x8000 122.3, 4 x 5: 124.3; 8192x8192 170 to 172
        //     [191.6], 4 x 5: 172.7);
        //   16-bit results and 8-bit codes up to 256 MB: 4 x 4, 4 per CU (2832x4256 to binary16 27.8 us, 29.4
        //     with 4 x 6 and 3 per CU; 3000x3000 22.1 / 23.2, 8x1080x1920 39.0 / 40.1, 2832x4256 to codes
        //     27.3 / 29.1); above: 4 x 6, 3 per CU (16x1080x1920 75.7 [89.7] us, 64x1080x1920 331
        //     [355], 4320x7680 80.8 [94.2]); one image beyond 800 MB: 5 x 6, 2 per CU (8192x8192 161
        //     [184] us, 175 with 4 x 6);
        //   up to 128 MB (several images, too many tiles for one per CU): 4 x 4, 4 per CU
        //     (32x512x512 24.9 [25.6] us).
        // 8-bit input is the opposite: every reservation costs time (8192x8192 uint8: 93 us with
        // none, 102 us with 4 tiles per CU), so it keeps 4 x 4 and all the wavefronts that fit.  Only to
        // 8-bit codes, which leave the vector ALUs as the one limit, taller tiles gain by computing fewer rows
        // twice: above 128 MB 4 wavefronts x 10 rows (8192x8192 66.1 us, 69.4 with 4 x 4; 19x1424x1964
        // 53.0 / 55.9; but 8x1080x1920, 66 MB, 19.9 / 19.2), if the image's tiles of 36 result rows come to at
        // most 0.9 of the input rows that tiles of 12 compute: the last tile of an image is computed whole.  240
        // MB of 256-column images, 4 x 10 against 4 x 4: 40 rows high 50.9 / 53.2 us (0.83 of the rows), 240 rows
        // 57.5 / 58.0 (0.88), 96 rows 61.0 / 58.8 (0.94), 60 rows 63.3 / 59.3 (1.0), 44 rows 79.1 / 61.9 (1.25),
        // 16 rows 104 / 47 (2.5).
        if (footprint <= (128LL << 20)) { tile_rw = 4; tile_nw = 4; tile_lds_kb = 36; }
        else if (out_dtype != HARRIS_OUT_F32 && batch == 1 && footprint > (800LL << 20)) { tile_rw = 6; tile_nw = 5; tile_lds_kb = 64; }
        else if (out_dtype != HARRIS_OUT_F32 && footprint <= (256LL << 20)) { tile_rw = 4; tile_nw = 4; tile_lds_kb = 36; }
        else if (out_dtype != HARRIS_OUT_F32) { tile_rw = 6; tile_nw = 4; tile_lds_kb = 48; }
        else if (footprint <= (400LL << 20)) { tile_rw = 5; tile_nw = 4; tile_lds_kb = 48; }
        else if (batch >= 8) { tile_rw = 5; tile_nw = 5; tile_lds_kb = 64; }
        else { tile_rw = 6; tile_nw = 5; tile_lds_kb = 64; }
    }

    long long tile_rows;       // result rows per band or tile
    if (t.schedule == HARRIS_SCHEDULE_TILES) {
        if (t.rows == 0 && t.waves_per_block == 0) { t.rows = tile_rw; t.waves_per_block = tile_nw; if (t.lds_kb == 0) t.lds_kb = tile_lds_kb; }
        if (t.rows == 0) t.rows = 4;
        if (t.waves_per_block == 0) t.waves_per_block = 4;
        const bool rows_ok = t.rows == 4 || (t.px == 4 && (t.rows == 5 || t.rows == 6 || t.rows == 8 || t.rows == 9 || t.rows == 10));
        if (!rows_ok || t.waves_per_block < 2 || t.waves_per_block > 16) return HARRIS_ERR_ARG;
        if (in_shifted && !(t.rows == 4 || t.rows == 8)) return HARRIS_ERR_ARG;
        if (dtype == HARRIS_U8 && (t.flags & HARRIS_TUNE_FLAG_HANDOFF)) return HARRIS_ERR_ARG;   // ready flags: float32 input only
        if (t.prefetch != 0) return HARRIS_ERR_ARG;
        tile_rows = (long long)t.rows * t.waves_per_block - 4;
        // The reservation: at least four rows for each wavefront.  From 8-bit input a tile with 16-byte lanes takes up to
        // six (tile_lds_bytes), which the launch sees to.
        const int need_kb = (int)(((long long)t.waves_per_block * 4 * 64 * t.px * 4 + 1023) / 1024);
        if (t.lds_kb < need_kb) t.lds_kb = need_kb;
    } else {
        if (t.lds_kb != 0) return HARRIS_ERR_ARG;                       // the band schedule uses no LDS
        const bool large = footprint > (256LL << 20);
        if (t.prefetch == 0) t.prefetch = 3;
        if (t.prefetch != 3) return HARRIS_ERR_ARG;                     // the one depth the band kernels are built for
        if (t.waves_per_block == 0) t.waves_per_block = large ? 4 : 1;
        if (!(t.waves_per_block == 1 || t.waves_per_block == 2 || t.waves_per_block == 4)) return HARRIS_ERR_ARG;
        if (t.rows == 0) {
            if (large) {
                t.rows = 32;       // thousands of bands in any case: measured best trade of halo rows against run length
            } else {
                // Everything is resident at once.  Take the shortest band of 16..64 rows that
                // needs no more wavefronts than the chip has SIMDs (1024): every wavefront then
                // has a SIMD to itself, the 256 CUs hold at most 4 each, and all of them start
                // and end together.  (Measured on 1536x2560 and 2832x4256: launches whose
                // wavefront count lies just below a multiple of 256 are the fast ones.)
                const long long per_band = (long long)batch * n_strips;
                long long best_r = 64;
                for (long long r = 16; r <= 64; ++r)
                    if (((n + r - 1) / r) * per_band <= 1024) { best_r = r; break; }
                t.rows = (int)best_r;
            }
        }
        tile_rows = t.rows;
    }
    const long long n_bands = n > 0 ? ((long long)n + tile_rows - 1) / tile_rows : 0;
    const long long tiles_per_image = n_bands * n_strips;
    const long long n_tiles = tiles_per_image * batch;

    // Load policy, measured.  One tile per CU (at most 256 tiles): everything non-temporal (1536x2560:
    // 12.2 us against 12.6 us with the shared rows kept).  Many tiles: non-temporal except the rows
    // two tiles share, which the default policy keeps in L2 for the second reader (2832x4256: 34.6 us
    // against 37.1 us all-default and 39.7 us all-non-temporal; 4096x4096: 49.7 / 53.8 / 54.6 us;
    // 32x512x512: 25.7 / 27.0 / 26.8 us; 8192x8192 uint8: 91.1 / 105 / 91.8 us; 16x1080x1920 with
    // tiles of 5 x 6: 98.2 / 101.8 us all-default; 64x1080x1920 with 5 x 8: 374.4 / 378.4 us).
    // Bands and lanes narrower than 16 bytes have no mixed policy: default-policy loads from 128 MB on.
    const bool one_tile_per_cu = t.schedule == HARRIS_SCHEDULE_TILES && n_tiles <= 256;
    if (!(t.flags & (HARRIS_TUNE_CACHED_LOADS | HARRIS_TUNE_STREAM_LOADS))) {
        if (t.flags & HARRIS_TUNE_FLAG_HANDOFF) t.flags |= HARRIS_TUNE_STREAM_LOADS;
        else if (tile4 && !one_tile_per_cu) t.flags |= HARRIS_TUNE_STREAM_LOADS | HARRIS_TUNE_KEEP_SHARED_ROWS;
        else if (dtype == HARRIS_F32 && footprint > (128LL << 20)) t.flags |= HARRIS_TUNE_CACHED_LOADS;
        else t.flags |= HARRIS_TUNE_STREAM_LOADS;
        // Ready flags instead of the barrier where tiles are few and tall and the input float32
        // (measured: 1536x2560 12.1 against 12.3 us, 2048x2048 12.7 / 13.2, 2x1536x2560 22.6 / 23.3,
        // 1080x1920 8.4 / 8.4; 720x1280, 3 wavefronts per tile, 6.4 / 6.1; 2048x4096 uint8 18.1 / 15.2).
        if (one_tile_per_cu && tile4 && dtype == HARRIS_F32 && t.waves_per_block >= 5 &&
            t.flags == (t.flags & ~(HARRIS_TUNE_CACHED_LOADS | HARRIS_TUNE_KEEP_SHARED_ROWS)))
            t.flags |= HARRIS_TUNE_FLAG_HANDOFF;
    }
    // TILES: one workgroup per tile.  BANDS: one wavefront per band of a strip; a workgroup
    // of 2 or 4 wavefronts takes 2 bands x 1 or 2 strips.
    const long long group_h = t.waves_per_block >= 2 ? 2 : 1, group_w = t.waves_per_block / group_h;
    const long long blocks_x = (n_strips + group_w - 1) / group_w;
    const long long blocks_per_image = blocks_x * ((n_bands + group_h - 1) / group_h);
    const long long blocks = t.schedule == HARRIS_SCHEDULE_TILES ? n_tiles : blocks_per_image * batch;
    if (tiles_per_image > 0x7fffffffLL || n_tiles > 0x7fffffffLL || blocks > 0x7fffffffLL) return HARRIS_ERR_SHAPE;

    if (chosen) *chosen = t;
    if (n_blocks) *n_blocks = blocks;
    if (params) {
        params->H = H; params->W = W; params->n = n; params->m = m;
        params->rows_per_band = (int)tile_rows;
        params->n_strips = (unsigned)n_strips;
        params->strip_pitch = (unsigned)pitch;
        params->n_bands = (unsigned)n_bands;
        params->tiles_per_image = (unsigned)tiles_per_image;
        params->far_rows = 0;
        params->blocks_x = (unsigned)blocks_x;
        params->blocks_per_image = (unsigned)blocks_per_image;
        params->n_blocks = (unsigned)blocks;
        params->waves_per_block = (unsigned)t.waves_per_block;
        params->turns = chunk_turns(dtype, out_dtype, batch, footprint, n_strips, n_tiles);
        params->chunk = (unsigned)((n_tiles + 8LL * params->turns - 1) / (8LL * params->turns));
        // Wavefronts that a CU holds at once (64 vector registers each), or tiles that its 160 KB of LDS hold.
        const unsigned lds = harris_launch::tile_lds_bytes(dtype == HARRIS_U8, t.px, (unsigned)t.waves_per_block), reserved = (unsigned)t.lds_kb * 1024u;
        const long long by_lds = (160 << 10) / (lds > reserved ? lds : reserved), by_waves = 32 / t.waves_per_block;
        params->resident = t.schedule == HARRIS_SCHEDULE_TILES && n_tiles <= 256 * (by_lds < by_waves ? by_lds : by_waves);
        // Store policy of many-tile launches (the figures stand with kAuxManyStore): written through are
        // float32 results where a row has more strips than ends, from float32 input beyond 400 MB more than six, and
        // their borders lie on 64-byte boundaries, and small launches with two strips or more, up to 16 MB from 8-bit input and 13 from
        // float32 to float32.
        const bool aligned_strips = (t.flags & HARRIS_TUNE_ALIGNED_STORES) && n_strips > (dtype == HARRIS_F32 && footprint > (400LL << 20) ? 6 : 2);
        const bool small_launch = n_strips < 2 ? false : dtype == HARRIS_U8 ? footprint <= (16LL << 20) : out_dtype == HARRIS_OUT_F32 && footprint <= (13LL << 20);
        const bool through = small_launch || (out_dtype == HARRIS_OUT_F32 && aligned_strips);
        params->flags = t.flags | (through ? harris_launch::kWriteThrough : 0u);
        params->out_kind = (unsigned)out_dtype;
        params->in_shifted = in_shifted ? 1 : 0;
        params->out_shift = out_dtype == HARRIS_OUT_F32 ? 2u : out_dtype == HARRIS_OUT_U8 ? 0u : 1u;
        params->strip_reach = (unsigned)(pitch + 4 + border_reach);
        params->lds_bytes = (unsigned)t.lds_kb * 1024u;
    }
    return HARRIS_OK;
}

// The launch of a call: what plan_shape takes, or, whatever shape was asked for, tiles of four rows per wavefront for the kernels that address each row by
// itself and take all arguments whole.  That is for rows of hundreds of megabytes or that far apart, for images of more than 2^32 pixels, and for what the
// caller knows to need them (`far`).
int plan(int dtype, int out_dtype, int batch, int H, int W, int rgb_align, int out_align, const harris_layout& lay, const harris_tuning* tuning, bool far,
         harris_tuning* chosen, long long* n_blocks, harris_launch::Params* params) {
    harris_tuning shape;
    int rc = plan_shape(dtype, out_dtype, batch, H, W, rgb_align, out_align, lay, tuning, &shape, n_blocks, params);
    if (rc != HARRIS_OK) return rc;
    if (shape.schedule == HARRIS_SCHEDULE_TILES && !(shape.flags & HARRIS_TUNE_PACKED_IMAGES) && batch > 0 && H > 4 && W > 4)
        far = far || harris_launch::rows_are_far(lay.rgb_row_pitch, W, elem_size(dtype), shape.rows) || !harris_launch::compact::fits(lay, batch, out_elem_size(out_dtype));
    if (far) {
        // (float32: three tiles on a CU.  2 images of 40000x36000 to float32 7.97 ms, 8.66 with as many as fit, 8.13 with four, 8.54 with two.)
        const harris_tuning four = {HARRIS_SCHEDULE_TILES, shape.px == 4 ? 4 : 1, 4, 0, 4, shape.flags & HARRIS_TUNE_WORD_STORES, dtype == HARRIS_F32 && shape.px == 4 ? 48 : 0};
        rc = plan_shape(dtype, out_dtype, batch, H, W, rgb_align, out_align, lay, &four, &shape, n_blocks, params);
        if (rc != HARRIS_OK) return rc;
        if (params) {
            params->far_rows = 1;
            params->by_tiles_per_image = harris_launch::make_fastdiv(params->tiles_per_image);
            params->by_n_strips = harris_launch::make_fastdiv(params->n_strips);
        }
    }
    if (chosen) *chosen = shape;
    return HARRIS_OK;
}

unsigned pointer_alignment(const void* p) {
    uintptr_t v = (uintptr_t)p;
    unsigned a = 1;
    while (a < 256 && power_of_two_aligned(v, a * 2)) a *= 2;
    return a;
}

}  // namespace

extern "C" {

int harris_plan(int dtype, int batch, int H, int W, int rgb_align, int out_align,
                const harris_tuning* tuning, harris_tuning* chosen, long long* n_blocks) {
    return plan(dtype, HARRIS_OUT_F32, batch, H, W, rgb_align, out_align, dense_layout(H, W), tuning, false, chosen, n_blocks, nullptr);
}

int harris_plan_typed(int dtype, int out_dtype, int batch, int H, int W, int rgb_align, int out_align,
                      const harris_tuning* tuning, harris_tuning* chosen, long long* n_blocks) {
    return plan(dtype, out_dtype, batch, H, W, rgb_align, out_align, dense_layout(H, W), tuning, false, chosen, n_blocks, nullptr);
}

}  // extern "C"

namespace {

// Every entry point of the fused kernel ends here.
int run(const void* rgb, int dtype, int batch, int H, int W, const harris_layout* layout,
        float k, float sobel_scale, int window, void* out, int out_dtype, float q_scale, float q_offset,
        const harris_tuning* tuning, void* stream) {
    if (dtype != HARRIS_F32 && dtype != HARRIS_U8) return HARRIS_ERR_ARG;
    if (!known_out_dtype(out_dtype)) return HARRIS_ERR_ARG;
    if (!isfinite(q_scale) || !isfinite(q_offset)) return HARRIS_ERR_ARG;
    if (batch < 0 || H < 4 || W < 4) return HARRIS_ERR_SHAPE;
    if (!isfinite(k) || !isfinite(sobel_scale)) return HARRIS_ERR_ARG;
    if (window != HARRIS_WINDOW_BOX && window != HARRIS_WINDOW_BINOMIAL) return HARRIS_ERR_ARG;
    const long long n = H - 4, m = W - 4;
    const harris_layout lay = layout ? *layout : dense_layout(H, W);
    const long long in_rows_span = (long long)(H - 1) * lay.rgb_row_pitch + W;
    if (lay.rgb_row_pitch < W || lay.rgb_plane_pitch < in_rows_span || lay.rgb_image_pitch < 2 * lay.rgb_plane_pitch + in_rows_span)
        return HARRIS_ERR_SHAPE;
    if (lay.out_row_pitch < m || (n > 0 && lay.out_image_pitch < (n - 1) * lay.out_row_pitch + m)) return HARRIS_ERR_SHAPE;
    const bool empty = batch == 0 || H == 4 || W == 4;
    if (!empty && (rgb == nullptr || out == nullptr)) return HARRIS_ERR_NULL;
    if (!empty && (int)pointer_alignment(out) < out_elem_size(out_dtype)) return HARRIS_ERR_ARG;
    if (!empty && dtype == HARRIS_F32 && pointer_alignment(rgb) < 4) return HARRIS_ERR_ARG;

    // Alignment that every row start shares: the base pointer's and each pitch's (in bytes).
    auto common_alignment = [](unsigned a, long long pitch_bytes) {
        while (a > 1 && pitch_bytes % a != 0) a /= 2;
        return a;
    };
    unsigned rgb_align = 16, out_align = 16;
    if (!empty) {
        const long long e = elem_size(dtype);
        rgb_align = pointer_alignment(rgb);
        if (rgb_align > 16) rgb_align = 16;
        rgb_align = common_alignment(rgb_align, lay.rgb_row_pitch * e);
        rgb_align = common_alignment(rgb_align, lay.rgb_plane_pitch * e);
        rgb_align = common_alignment(rgb_align, lay.rgb_image_pitch * e);
        out_align = pointer_alignment(out);
        if (out_align > 16) out_align = 16;
        out_align = common_alignment(out_align, lay.out_row_pitch * out_elem_size(out_dtype));
        out_align = common_alignment(out_align, lay.out_image_pitch * out_elem_size(out_dtype));
    }

    harris_launch::Params p;
    harris_tuning shape;
    long long n_blocks = 0;
    // The Sobel scale multiplies Ix and Iy, which are linear in gray: fold it into the three gray weights; from 8-bit input, whose
    // weights are whole numbers, its fourth power and theirs into the factor of the result.  The kernels that take it as two numbers are those with whole
    // arguments; the others have no instruction to spare for them.
    const double unit = sobel_scale * (262144.0 / 255000.0);
    double factor = unit * unit * unit * unit;
    if (dtype == HARRIS_U8) harris_launch::bound_k(k, factor);
    float gain, more_gain;
    harris_launch::split_gain(factor, gain, more_gain);
    const bool far = dtype == HARRIS_U8 && more_gain != 1.0f && !empty;
    int rc = plan(dtype, out_dtype, batch, H, W, (int)rgb_align, (int)out_align, lay, tuning, far, &shape, &n_blocks, &p);
    if (rc != HARRIS_OK) return rc;
    if (empty) return HARRIS_OK;
    p.rgb = rgb;
    p.out = out;
    p.in_row_pitch = lay.rgb_row_pitch; p.in_plane_pitch = lay.rgb_plane_pitch; p.in_image_pitch = lay.rgb_image_pitch;
    p.out_row_pitch = lay.out_row_pitch; p.out_image_pitch = lay.out_image_pitch;
    if (batch == 1) p.in_image_pitch = p.out_image_pitch = 0;           // of no matter, and they may be long
    p.out_row_bytes = (unsigned long long)lay.out_row_pitch * out_elem_size(out_dtype);
    p.out_image_bytes = (unsigned long long)p.out_image_pitch * out_elem_size(out_dtype);
    p.wr = 0.299f * sobel_scale;
    p.wg = 0.587f * sobel_scale;
    p.wb = 0.114f * sobel_scale;
    p.gain = gain;
    p.more_gain = more_gain;
    p.k = k;
    p.binomial = window == HARRIS_WINDOW_BINOMIAL ? 1 : 0;
    p.q_scale = q_scale;
    p.q_offset = q_offset;
    return harris_launch::launch(p, shape, n_blocks, dtype, stream);
}

}  // namespace

extern "C" {

int harris_coarsity_typed(const void* rgb, int dtype, int batch, int H, int W, const harris_layout* layout,
                          float k, float sobel_scale, int window, void* out, int out_dtype,
                          const harris_tuning* tuning, void* stream) {
    if (out_dtype == HARRIS_OUT_U8) return HARRIS_ERR_ARG;          // needs a scale: harris_coarsity_quantized
    return run(rgb, dtype, batch, H, W, layout, k, sobel_scale, window, out, out_dtype, 1.0f, 0.0f, tuning, stream);
}

int harris_coarsity_quantized(const void* rgb, int dtype, int batch, int H, int W, const harris_layout* layout,
                              float k, float sobel_scale, int window, float q_scale, float q_offset,
                              uint8_t* out, const harris_tuning* tuning, void* stream) {
    return run(rgb, dtype, batch, H, W, layout, k, sobel_scale, window, out, HARRIS_OUT_U8, q_scale, q_offset, tuning, stream);
}

int harris_coarsity_pitched(const void* rgb, int dtype, int batch, int H, int W, const harris_layout* layout,
                            float k, float sobel_scale, int window, float* out,
                            const harris_tuning* tuning, void* stream) {
    return harris_coarsity_typed(rgb, dtype, batch, H, W, layout, k, sobel_scale, window, out, HARRIS_OUT_F32, tuning, stream);
}

int harris_coarsity_ex(const void* rgb, int dtype, int batch, int H, int W, float k, float sobel_scale,
                       int window, float* out, const harris_tuning* tuning, void* stream) {
    return harris_coarsity_pitched(rgb, dtype, batch, H, W, nullptr, k, sobel_scale, window, out, tuning, stream);
}

int harris_coarsity(const float* rgb, int batch, int H, int W, float k, float* out, void* stream) {
    return harris_coarsity_ex(rgb, HARRIS_F32, batch, H, W, k, 1.0f, HARRIS_WINDOW_BOX, out, nullptr, stream);
}

int harris_coarsity_u8(const uint8_t* rgb, int batch, int H, int W, float k, float* out, void* stream) {
    return harris_coarsity_ex(rgb, HARRIS_U8, batch, H, W, k, 1.0f, HARRIS_WINDOW_BOX, out, nullptr, stream);
}

long long harris_grouped_workspace_bytes(int grouping, int batch, int H, int W) {
    if (grouping < 1 || grouping > 4 || batch < 0 || H < 4 || W < 4) return -1;
    return (long long)(harris_launch::grouped_workspace_floats(grouping, batch, H, W) * sizeof(float));
}

int harris_coarsity_grouped(const void* rgb, int dtype, int batch, int H, int W, float k, float sobel_scale,
                            int window, int grouping, void* workspace, long long workspace_bytes,
                            float* out, void* stream) {
    if (grouping < 1 || grouping > 4) return HARRIS_ERR_ARG;
    if (grouping == 4) return harris_coarsity_ex(rgb, dtype, batch, H, W, k, sobel_scale, window, out, nullptr, stream);
    if (dtype != HARRIS_F32 && dtype != HARRIS_U8) return HARRIS_ERR_ARG;
    if (batch < 0 || H < 4 || W < 4) return HARRIS_ERR_SHAPE;
    if (!isfinite(k) || !isfinite(sobel_scale)) return HARRIS_ERR_ARG;
    if (window != HARRIS_WINDOW_BOX && window != HARRIS_WINDOW_BINOMIAL) return HARRIS_ERR_ARG;
    if (batch == 0 || H == 4 || W == 4) return HARRIS_OK;
    if (rgb == nullptr || out == nullptr || workspace == nullptr) return HARRIS_ERR_NULL;
    if (pointer_alignment(out) < 4 || pointer_alignment(workspace) < 4) return HARRIS_ERR_ARG;
    if (dtype == HARRIS_F32 && pointer_alignment(rgb) < 4) return HARRIS_ERR_ARG;
    if (workspace_bytes < harris_grouped_workspace_bytes(grouping, batch, H, W)) return HARRIS_ERR_ARG;
    return harris_launch::launch_grouped(rgb, dtype, batch, H, W, k, sobel_scale, window == HARRIS_WINDOW_BINOMIAL,
                                         grouping, static_cast<float*>(workspace), out, stream);
}

int harris_coarsity_grouped_static(const void* rgb, int dtype, int batch, int H, int W, float k, float sobel_scale,
                                   int window, int grouping, float* out, void* stream) {
    if (grouping < 1 || grouping > 4) return HARRIS_ERR_ARG;
    if (grouping == 4) return harris_coarsity_ex(rgb, dtype, batch, H, W, k, sobel_scale, window, out, nullptr, stream);
    if (batch < 0 || H < 4 || W < 4) return HARRIS_ERR_SHAPE;
    if (batch == 0 || H == 4 || W == 4)      // empty result: the remaining argument checks, no work, no scratch
        return harris_coarsity_grouped(rgb, dtype, batch, H, W, k, sobel_scale, window, grouping, nullptr, 0, out, stream);
    // The gray image alone is 4 bytes per pixel; checked in doubles first, since the exact count
    // below is 64-bit arithmetic and absurd shapes would not fit it.
    if (4.0 * (double)batch * (double)H * (double)W > (double)HARRIS_GROUPED_SCRATCH_BYTES) return HARRIS_ERR_SCRATCH;
    const long long need = harris_grouped_workspace_bytes(grouping, batch, H, W);
    if (need < 0 || need > (long long)HARRIS_GROUPED_SCRATCH_BYTES) return HARRIS_ERR_SCRATCH;
    if (rgb == nullptr || out == nullptr) return HARRIS_ERR_NULL;
    float* ws = harris_launch::scratch_of_current_device();
    if (ws == nullptr) return HARRIS_ERR_LAUNCH;
    return harris_coarsity_grouped(rgb, dtype, batch, H, W, k, sobel_scale, window, grouping, ws, need, out, stream);
}

int harris_probe_copy(const void* rgb, int dtype, int batch, int H, int W, float* out, void* stream) {
    if (dtype != HARRIS_F32 && dtype != HARRIS_U8) return HARRIS_ERR_ARG;
    if (batch < 0 || H < 4 || W < 4) return HARRIS_ERR_SHAPE;
    if (batch == 0 || H == 4 || W == 4) return HARRIS_OK;
    if (rgb == nullptr || out == nullptr) return HARRIS_ERR_NULL;
    const long long e = elem_size(dtype);
    if (pointer_alignment(rgb) < 16 || pointer_alignment(out) < 16) return HARRIS_ERR_ARG;
    if (((long long)H * W * e) % 16 != 0 || ((long long)(H - 4) * (W - 4) * 4) % 16 != 0) return HARRIS_ERR_ARG;
    return harris_launch::launch_copy_probe(rgb, dtype, batch, H, W, out, stream);
}

int harris_probe_stream(int kind, const void* src, void* dst, long long bytes, void* stream) {
    if (kind != HARRIS_PROBE_READ && kind != HARRIS_PROBE_WRITE && kind != HARRIS_PROBE_NONE) return HARRIS_ERR_ARG;
    if (bytes < 0) return HARRIS_ERR_SHAPE;
    if (kind == HARRIS_PROBE_NONE) return harris_launch::launch_stream_probe(kind, nullptr, nullptr, 0, stream);
    if (bytes == 0) return HARRIS_OK;
    if (dst == nullptr || (kind == HARRIS_PROBE_READ && src == nullptr)) return HARRIS_ERR_NULL;
    if (bytes % 16 != 0 || pointer_alignment(dst) < 16 || (kind == HARRIS_PROBE_READ && pointer_alignment(src) < 16)) return HARRIS_ERR_ARG;
    return harris_launch::launch_stream_probe(kind, src, dst, bytes, stream);
}

const char* harris_strerror(int status) {
    switch (status) {
        case HARRIS_OK: return "success";
        case HARRIS_ERR_NULL: return "rgb or out is NULL for a non-empty result";
        case HARRIS_ERR_SHAPE: return "invalid shape: batch < 0, H < 4, W < 4, too many tiles, or pitches smaller than the image";
        case HARRIS_ERR_ARG: return "invalid argument: non-finite k or sobel_scale, misaligned pointer, unknown dtype, window, grouping or tuning, workspace too small";
        case HARRIS_ERR_LAUNCH: return "the HIP runtime refused the kernel launch";
        case HARRIS_ERR_SCRATCH: return "the problem needs more scratch memory than the library's fixed buffer holds (HARRIS_GROUPED_SCRATCH_BYTES)";
        default: return "unknown harris_status";
    }
}

int harris_version(void) { return kVersion; }

}  // extern "C"
