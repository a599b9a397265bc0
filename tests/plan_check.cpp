// Host check of planned launches: the library's C interface (harris_api.cpp) is compiled with a
// launcher that keeps what the planner hands over instead of enqueueing it, and what the kernel's lanes
// would load is worked out from that, with the same header functions that the kernel uses.
// Built and run by tests/test_abi_host.py; prints "ok <launches checked>" or the first fault.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <vector>

#include "harris_launch.h"

namespace harris_launch {

static Params last;
static harris_tuning last_shape;
static int launches = 0;

int launch(const Params& p, const harris_tuning& shape, long long n_blocks, int, void*) {
    if (n_blocks != (long long)p.n_blocks) return HARRIS_ERR_LAUNCH;
    last = p; last_shape = shape; ++launches;
    return HARRIS_OK;
}
size_t grouped_workspace_floats(int, int, int, int) { return 0; }
int launch_grouped(const void*, int, int, int, int, float, float, int, int, float*, float*, void*) { return HARRIS_ERR_LAUNCH; }
float* scratch_of_current_device() { return nullptr; }
int launch_copy_probe(const void*, int, int, int, int, float*, void*) { return HARRIS_ERR_LAUNCH; }
int launch_stream_probe(int, const void*, void*, long long, void*) { return HARRIS_ERR_LAUNCH; }

}  // namespace harris_launch

using harris_launch::Params;

// Is byte `at` (from element 0 of the call) part of a row of the call?
static bool inside_a_row(long long at, const harris_layout& lay, int batch, int H, int W, int elem) {
    const long long e = at / elem;
    if (e < 0) return false;
    for (long long b = e / lay.rgb_image_pitch, b0 = b; b <= b0; ++b) {
        if (b >= batch) return false;
        const long long in_image = e - b * lay.rgb_image_pitch;
        for (int c = 0; c < 3; ++c) {
            const long long in_plane = in_image - c * lay.rgb_plane_pitch;
            if (in_plane < 0) continue;
            const long long row = in_plane / lay.rgb_row_pitch;
            if (row < H && in_plane - row * lay.rgb_row_pitch < W) return true;
        }
    }
    return false;
}

// Every byte that a launch of the narrow-image kernel loads: rows first and last of the planes (the others
// lie between them), every lane, full and partial groups.
static bool patch_loads_inside_rows(const Params& p, const harris_layout& lay, int batch, int elem) {
    if (!(p.flags & HARRIS_TUNE_PACKED_IMAGES)) return true;
    const unsigned groups = (p.batch + p.images - 1) / p.images;
    for (unsigned group = 0; group < groups; group += groups > 2 ? groups - 1 : 1) {
        const unsigned left = p.batch - group * p.images, images = left < p.images ? left : p.images;
        for (int row : {0, 1, p.H - 2, p.H - 1})
            for (int c = 0; c < 3; ++c)
                for (unsigned lane = 0; lane < 64; ++lane) {
                    const harris_launch::PatchLane l = harris_launch::patch_lane(p, images, lane, (unsigned)elem);
                    if (l.image != lane / p.image_lanes) { std::printf("lane %u / %u gives %u\n", lane, p.image_lanes, l.image); return false; }
                    const long long start = ((long long)group * p.images * lay.rgb_image_pitch + c * lay.rgb_plane_pitch + row * lay.rgb_row_pitch) * elem;
                    for (unsigned i = 0; i < 4u * (unsigned)elem; ++i) {
                        if (elem == 4 && (unsigned long long)l.in_voff + i >= l.in_bytes) continue;     // range check of the descriptor
                        if (!inside_a_row(start + l.in_voff + i, lay, batch, p.H, p.W, elem)) {
                            std::printf("%d images of %dx%d, elements of %d bytes, pitches %lld %lld %lld: lane %u reads byte %u of image %u, plane %d, row %d, which is in no row\n",
                                        batch, p.H, p.W, elem, lay.rgb_row_pitch, lay.rgb_plane_pitch, lay.rgb_image_pitch, lane, l.in_voff + i - l.image * (unsigned)(lay.rgb_image_pitch * elem), l.image, c, row);
                            return false;
                        }
                    }
                }
    }
    return true;
}

// The same of dense 8-bit images loaded as pairs of aligned words: first and last group, every row of a tile's wavefronts and of a workgroup without a
// tile, every lane.  No word is loaded but those that hold bytes of the group, and the pixels of the image's columns and rows are in the lane's pair.
static bool patch_pairs_inside_words(const Params& p, int batch) {
    const unsigned long long base = (size_t)p.rgb, total = (unsigned long long)batch * p.in_image_pitch;
    const unsigned groups = (p.batch + p.images - 1) / p.images;
    for (unsigned group = 0; group < groups; group += groups > 2 ? groups - 1 : 1) {
        const unsigned left = p.batch - group * p.images, images = left < p.images ? left : p.images;
        const unsigned long long first = base + (unsigned long long)group * p.images * p.in_image_pitch, from = first & ~3ull;
        const unsigned lead = (unsigned)(first & 3u), end = harris_launch::patch_words_end(p, images, lead);
        bool good = from + end <= ((base + total + 3) & ~3ull) && end >= lead + images * (unsigned)p.in_image_pitch;
        for (int y : {0, 1, 2, 3, p.H - 2, p.H - 1, p.H, p.H + 40, 1 << 30})
            for (int c = 0; c < 3; ++c)
                for (unsigned lane = 0; lane < 64; ++lane) {
                    const harris_launch::PatchLane l = harris_launch::patch_lane(p, images, lane, 1);
                    const unsigned at = harris_launch::patch_first_byte(p, l, lead) + harris_launch::patch_row(p, y, c);
                    for (unsigned i = 0; l.live && y < p.H && i < 4 && l.col + i < (unsigned)p.W; ++i) {
                        const unsigned long long pixel = (unsigned long long)l.image * p.in_image_pitch + c * p.in_plane_pitch + y * p.in_row_pitch + l.col + i;
                        good = good && from + at + i == first + pixel && at + i < end && (at & 3u) + i < 8;
                    }
                    for (unsigned word = 0; word < 2; ++word)       // the hardware drops words from the end on
                        good = good && ((at & ~3u) + 4 * word >= end || (at & ~3u) + 4 * word + 4 <= end);
                    good = good && (at & ~3u) < 0x80000000u;
                    if (!good) { std::printf("%d images of %dx%d from byte %llu: group %u, row %d, plane %d, lane %u loads at %u of %u\n", batch, p.H, p.W, base & 3, group, y, c, lane, at, end); return false; }
                }
    }
    return true;
}

int main() {
    int packed = 0, gaps_packed = 0, pairs = 0;
    for (int W = 5; W <= 128; ++W)
        for (int H : {5, 31, 64})
            for (int dtype : {HARRIS_F32, HARRIS_U8}) {
                const int n = H - 4, m = W - 4, batch = (1 << 20) / (H * W) + 3;
                // Rows, planes and images without gaps, and every combination of gaps between them.
                for (int gaps = 0; gaps < 8; ++gaps) {
                    harris_layout lay;
                    lay.rgb_row_pitch = W + (gaps & 1 ? 3 : 0);
                    lay.rgb_plane_pitch = H * lay.rgb_row_pitch + (gaps & 2 ? 2 : 0);
                    lay.rgb_image_pitch = 3 * lay.rgb_plane_pitch + (gaps & 4 ? 1 : 0);
                    lay.out_row_pitch = m; lay.out_image_pitch = (long long)n * m;
                    const int before = harris_launch::launches;
                    if (harris_coarsity_pitched((const void*)0x100000, dtype, batch, H, W, &lay, 0.04f, 1.0f, HARRIS_WINDOW_BOX, (float*)0x200000, nullptr, nullptr) != HARRIS_OK ||
                        harris_launch::launches != before + 1) {
                        std::printf("refused: %d images of %dx%d\n", batch, H, W);
                        return 1;
                    }
                    // The shape of that launch, given back, gives it again; the shape planned for images without
                    // gaps is accepted too.
                    const Params first = harris_launch::last;
                    const harris_tuning given = harris_launch::last_shape;
                    harris_tuning planned;
                    if (harris_coarsity_pitched((const void*)0x100000, dtype, batch, H, W, &lay, 0.04f, 1.0f, HARRIS_WINDOW_BOX, (float*)0x200000, &given, nullptr) != HARRIS_OK ||
                        std::memcmp(&given, &harris_launch::last_shape, sizeof given) != 0 || first.n_blocks != harris_launch::last.n_blocks ||
                        harris_plan(dtype, batch, H, W, dtype == HARRIS_U8 ? 1 : 4, 16, nullptr, &planned, nullptr) != HARRIS_OK ||
                        harris_coarsity_pitched((const void*)0x100000, dtype, batch, H, W, &lay, 0.04f, 1.0f, HARRIS_WINDOW_BOX, (float*)0x200000, &planned, nullptr) != HARRIS_OK) {
                        std::printf("planned shape not accepted, or another launch: %d images of %dx%d, dtype %d, gaps %d\n", batch, H, W, dtype, gaps);
                        return 1;
                    }
                    if (!patch_loads_inside_rows(harris_launch::last, lay, batch, dtype == HARRIS_U8 ? 1 : 4)) return 1;
                    const Params& p = first;
                    if (!(p.flags & HARRIS_TUNE_PACKED_IMAGES)) continue;
                    for (size_t lead = 0; lead < 4 && dtype == HARRIS_U8 && gaps == 0; ++lead) {
                        Params moved = first;
                        moved.rgb = (const void*)(0x100000 + lead);
                        if (harris_launch::patch_in_pairs(moved) && (++pairs, !patch_pairs_inside_words(moved, batch))) return 1;
                    }
                    ++packed;
                    if (gaps) ++gaps_packed;
                    if (!patch_loads_inside_rows(p, lay, batch, dtype == HARRIS_U8 ? 1 : 4)) return 1;
                }
            }
    // Store policy: {input type, result type, images, height, width, written through}.
    static const int store[][6] = {{HARRIS_U8, HARRIS_OUT_F32, 17, 237, 320, 1}, {HARRIS_U8, HARRIS_OUT_F32, 1, 1101, 1630, 1}, {HARRIS_U8, HARRIS_OUT_F16, 2, 700, 1200, 1},
                                   {HARRIS_U8, HARRIS_OUT_F32, 66, 237, 320, 0}, {HARRIS_U8, HARRIS_OUT_F16, 66, 237, 320, 0}, {HARRIS_F32, HARRIS_OUT_F32, 6, 260, 332, 1}, {HARRIS_U8, HARRIS_OUT_F32, 14, 240, 240, 0},
                                   {HARRIS_F32, HARRIS_OUT_F32, 21, 237, 320, 0}, {HARRIS_F32, HARRIS_OUT_F16, 8, 237, 320, 0}, {HARRIS_F32, HARRIS_OUT_F32, 781, 240, 160, 0},
                                   {HARRIS_F32, HARRIS_OUT_F32, 64, 1080, 1920, 1}, {HARRIS_U8, HARRIS_OUT_F32, 1, 8192, 8192, 1}, {HARRIS_U8, HARRIS_OUT_F32, 8, 1079, 1919, 0},
                                   {HARRIS_F32, HARRIS_OUT_F32, 128, 720, 1280, 0}, {HARRIS_F32, HARRIS_OUT_F32, 32, 720, 1280, 0}, {HARRIS_F32, HARRIS_OUT_F32, 13, 720, 1280, 1}};
    for (const auto& c : store) {
        if (harris_coarsity_typed((const void*)0x100000, c[0], c[2], c[3], c[4], nullptr, 0.04f, 1.0f, HARRIS_WINDOW_BOX, (void*)0x200000, c[1], nullptr, nullptr) != HARRIS_OK ||
            ((harris_launch::last.flags & harris_launch::kWriteThrough) != 0) != (c[5] != 0)) {
            std::printf("store policy of %d images of %dx%d, types %d and %d\n", c[2], c[3], c[4], c[0], c[1]);
            return 1;
        }
    }
    // Launches of many tiles: every tile is dealt out once, to a grid that the hardware takes; by turns from some size on.
    for (const auto& c : {std::vector<int>{1, 1080, 1920, 1}, {64, 1080, 1920, 0}, {1, 2832, 4256, 0}, {3001, 240, 161, 0}, {1, 30000, 253, 0}, {1, 12, 600000, 0}, {7, 333, 2501, 1}, {8192, 32, 32, 0}, {1501, 30, 33, 0}, {70, 120, 64, 0}})
        for (int dtype : {HARRIS_F32, HARRIS_U8})
            for (int out : {HARRIS_OUT_F32, HARRIS_OUT_F16}) {
                const harris_tuning keep = {HARRIS_SCHEDULE_TILES, 0, 0, 0, 0, HARRIS_TUNE_STREAM_LOADS | HARRIS_TUNE_KEEP_SHARED_ROWS, 0};
                if (harris_coarsity_typed((const void*)0x100000, dtype, c[0], c[1], c[2], nullptr, 0.04f, 1.0f, HARRIS_WINDOW_BOX, (void*)0x200000, out, c[3] ? &keep : nullptr, nullptr) == HARRIS_ERR_ARG) continue;
                const Params& p = harris_launch::last;
                const unsigned long long grid = 8ull * p.chunk * p.turns;
                std::vector<unsigned char> dealt(p.n_blocks, 0);
                bool good = p.turns >= 1 && p.turns <= 65535 && p.chunk >= 1 && grid < 0x7fffffffull && grid - p.n_blocks < 8ull * p.turns;
                for (unsigned y = 0; good && y < p.turns; ++y)
                    for (unsigned x = 0; x < 8 * p.chunk; ++x) {
                        const unsigned tile = harris_launch::dealt_tile(x, y, p.chunk);
                        if (tile < p.n_blocks && dealt[tile]++ != 0) good = false;
                    }
                for (unsigned char d : dealt) good = good && d == 1;
                if (!good || (p.turns > 1 && p.n_blocks <= 2048 && !(p.flags & HARRIS_TUNE_PACKED_IMAGES))) {
                    std::printf("%d images of %dx%d, types %d and %d: %u tiles, chunks of %u, %u turns\n", c[0], c[1], c[2], dtype, out, p.n_blocks, p.chunk, p.turns);
                    return 1;
                }
            }
    // Narrow images: as many wavefronts a workgroup as leave the fewest on the fullest CU, or four.
    static const int waves[][5] = {{HARRIS_F32, 460, 150, 37, 4}, {HARRIS_F32, 394, 104, 35, 8}, {HARRIS_F32, 501, 117, 44, 7}, {HARRIS_F32, 2900, 50, 26, 5}, {HARRIS_F32, 2048, 64, 64, 4},
                                   {HARRIS_F32, 8192, 32, 32, 4}, {HARRIS_F32, 1931, 61, 84, 4}, {HARRIS_U8, 1140, 67, 47, 5}, {HARRIS_U8, 2526, 50, 33, 7}, {HARRIS_U8, 2816, 26, 63, 7},
                                   {HARRIS_U8, 22916, 17, 9, 5}, {HARRIS_U8, 805, 39, 121, 4}, {HARRIS_U8, 309, 112, 52, 4}, {HARRIS_F32, 100, 60, 60, 8}};
    for (const auto& c : waves) {
        if (harris_coarsity_typed((const void*)0x100000, c[0], c[1], c[2], c[3], nullptr, 0.04f, 1.0f, HARRIS_WINDOW_BOX, (void*)0x200000, HARRIS_OUT_F32, nullptr, nullptr) != HARRIS_OK ||
            !(harris_launch::last.flags & HARRIS_TUNE_PACKED_IMAGES) || harris_launch::last_shape.waves_per_block != c[4]) {
            std::printf("%d images of %dx%d, type %d: %d wavefronts a workgroup\n", c[1], c[2], c[3], c[0], harris_launch::last_shape.waves_per_block);
            return 1;
        }
    }
    // Very narrow 8-bit images: few workgroups on a CU: {input type, images, height, width, KB reserved}.
    static const int reserved[][5] = {{HARRIS_U8, 7107, 45, 14, 52}, {HARRIS_U8, 20000, 72, 7, 52}, {HARRIS_U8, 4120, 104, 7, 52}, {HARRIS_U8, 12741, 138, 11, 64}, {HARRIS_U8, 5507, 246, 24, 16}, {HARRIS_U8, 5507, 246, 25, 16}, {HARRIS_U8, 149162, 8, 14, 8},
                                      {HARRIS_F32, 7107, 45, 14, 16}, {HARRIS_U8, 2048, 64, 14, 16}};
    for (const auto& c : reserved)
        if (harris_coarsity_typed((const void*)0x100000, c[0], c[1], c[2], c[3], nullptr, 0.04f, 1.0f, HARRIS_WINDOW_BOX, (void*)0x200000, HARRIS_OUT_F32, nullptr, nullptr) != HARRIS_OK ||
            !(harris_launch::last.flags & HARRIS_TUNE_PACKED_IMAGES) || harris_launch::last_shape.lds_kb != c[4] || (int)harris_launch::last.lds_bytes != c[4] * 1024) {
            std::printf("%d images of %dx%d, type %d: %d wavefronts, %d KB reserved\n", c[1], c[2], c[3], c[0], harris_launch::last_shape.waves_per_block, harris_launch::last_shape.lds_kb);
            return 1;
        }
    // How many tiles an XCD takes in a row, where the wrong number is slower than one turn: {input type, images, height, width, least, most}.
    static const int runs[][6] = {{HARRIS_F32, 1, 4200, 4200, 130, 150}, {HARRIS_F32, 1, 3456, 5184, 130, 150}, {HARRIS_F32, 1, 4608, 4608, 130, 150}, {HARRIS_F32, 1, 2832, 4256, 130, 150},
                                  {HARRIS_F32, 1, 4096, 4300, 130, 150}, {HARRIS_F32, 1, 5778, 4238, 127, 130}, {HARRIS_F32, 1, 3500, 4000, 70, 101}, {HARRIS_F32, 2, 2531, 3743, 110, 125}, {HARRIS_U8, 1, 4096, 4096, 90, 105},
                                  {HARRIS_U8, 2, 2048, 4096, 90, 105}, {HARRIS_U8, 8, 1080, 1920, 16, 17}, {HARRIS_U8, 1, 8192, 8192, 70, 71}};
    for (const auto& c : runs) {
        if (harris_coarsity_typed((const void*)0x100000, c[0], c[1], c[2], c[3], nullptr, 0.04f, 1.0f, HARRIS_WINDOW_BOX, (void*)0x200000, HARRIS_OUT_F32, nullptr, nullptr) != HARRIS_OK ||
            (int)harris_launch::last.chunk < c[4] || (int)harris_launch::last.chunk > c[5]) {
            std::printf("%d images of %dx%d, type %d: %u tiles in a row\n", c[1], c[2], c[3], c[0], harris_launch::last.chunk);
            return 1;
        }
    }
    // Odd result rows from 8-bit input that one strip of four pixels per lane just holds, or several: {result type, images, height, width, pixels per lane}.
    static const int odd_rows[][5] = {{HARRIS_OUT_U8, 64, 500, 250, 4}, {HARRIS_OUT_U8, 64, 500, 246, 4}, {HARRIS_OUT_U8, 64, 500, 254, 2}, {HARRIS_OUT_U8, 83, 333, 498, 4}, {HARRIS_OUT_F16, 86, 100, 251, 4},
                                      {HARRIS_OUT_BF16, 34, 100, 747, 4}, {HARRIS_OUT_F16, 86, 100, 255, 1}};
    for (const auto& c : odd_rows) {
        const int rc = c[0] == HARRIS_OUT_U8 ? harris_coarsity_quantized((const void*)0x100000, HARRIS_U8, c[1], c[2], c[3], nullptr, 0.04f, 1.0f, HARRIS_WINDOW_BOX, 1.0f, 0.0f, (uint8_t*)0x200000, nullptr, nullptr)
                                             : harris_coarsity_typed((const void*)0x100000, HARRIS_U8, c[1], c[2], c[3], nullptr, 0.04f, 1.0f, HARRIS_WINDOW_BOX, (void*)0x200000, c[0], nullptr, nullptr);
        const harris_tuning& s = harris_launch::last_shape;
        if (rc != HARRIS_OK || s.px != c[4] || (s.px == 4 && (long long)harris_launch::last.n_strips * 248 < c[3] - 4)) {
            std::printf("%d images of %dx%d, result type %d: %d pixels per lane, %u strips\n", c[1], c[2], c[3], c[0], s.px, harris_launch::last.n_strips);
            return 1;
        }
    }
    // Whether the chip holds all tiles of a launch at once: {images, height, width, wavefronts a workgroup or 0, KB reserved, it does}.
    static const int at_once[][6] = {{1, 1080, 1920, 0, 0, 1}, {1, 2457, 2400, 0, 0, 1}, {2, 2160, 3840, 0, 0, 0}, {1, 12, 600000, 0, 0, 0}, {8, 1079, 1919, 0, 0, 0},
                                     {1, 1500, 1900, 16, 0, 1}, {1, 8000, 1900, 16, 0, 0}, {1, 1080, 1920, 4, 48, 1}, {1, 1200, 1920, 4, 48, 0}, {1, 700, 960, 8, 0, 1}};
    for (const auto& c : at_once) {
        const harris_tuning t = {HARRIS_SCHEDULE_TILES, 4, 4, 0, c[3], 0u, c[4]};
        if (harris_coarsity_typed((const void*)0x100000, HARRIS_U8, c[0], c[1], c[2], nullptr, 0.04f, 1.0f, HARRIS_WINDOW_BOX, (void*)0x200000, HARRIS_OUT_F32, c[3] ? &t : nullptr, nullptr) != HARRIS_OK ||
            harris_launch::last.resident != c[5]) {
            std::printf("%d images of %dx%d, %d wavefronts, %d KB: %u tiles resident at once: %d\n", c[0], c[1], c[2], c[3], c[4], harris_launch::last.n_blocks, harris_launch::last.resident);
            return 1;
        }
    }
    // 8-bit rows on any byte loaded where they are: every lane, also beyond the row, loads inside it, and has the pixels
    // of its columns that the row has.
    for (unsigned W = 5; W <= 600; ++W)
        for (unsigned col = 0; col < W + 300; col += 4) {
            const harris_launch::ByteLane l = harris_launch::byte_lane(col, W);
            bool good = l.voff + 4 <= W && l.drop <= 24 && l.drop % 8 == 0;
            for (unsigned i = 0; i < 4 && col + i < W; ++i) good = good && l.drop / 8 + i < 4 && l.voff + l.drop / 8 + i == col + i;
            if (!good) { std::printf("lane of column %u of %u loads at %u, shifted by %u\n", col, W, l.voff, l.drop); return 1; }
        }
    // What a tile needs of LDS: rows of 64 lanes.
    for (unsigned w = 2; w <= 16; ++w)
        if (harris_launch::tile_lds_bytes(true, 4, w) != (1 + 6 * (w - 1)) * 1024 || harris_launch::tile_lds_bytes(false, 4, w) != w * 4096 || harris_launch::tile_lds_bytes(true, 2, w) != w * 2048) {
            std::printf("LDS of %u wavefronts\n", w);
            return 1;
        }
    // Grids of the groupings: fewer than 2^32 threads in x, one turn for all but huge launches, every workgroup once.
    for (unsigned long long blocks : {1ull, 7ull, 8ull, 9ull, 8100ull, (1ull << 23), (1ull << 23) + 1, 17500001ull, (1ull << 29) - 1}) {
        const harris_launch::GroupedGrid g = harris_launch::grouped_grid(blocks);
        const unsigned long long grid = 8ull * g.chunk * g.turns;
        bool good = 8ull * g.chunk * 256 < (1ull << 32) && g.turns >= 1 && g.turns <= 65535 && grid >= blocks && grid - blocks < 8ull * g.turns && (blocks > (1ull << 23) || g.turns == 1);
        std::vector<unsigned char> dealt(grid < (1ull << 25) ? grid : 0, 0);
        for (unsigned y = 0; good && !dealt.empty() && y < g.turns; ++y)
            for (unsigned x = 0; x < 8 * g.chunk; ++x) {
                const unsigned b = harris_launch::dealt_tile(x, y, g.chunk);
                if (b >= grid || dealt[b]++ != 0) good = false;
            }
        if (!good) { std::printf("%llu workgroups of a grouping: chunks of %u, %u turns\n", blocks, g.chunk, g.turns); return 1; }
    }
    // Groupings: batches of small images in runs of images, small batches of them in order.
    for (const auto& c : {std::vector<int>{500, 40, 40, 1}, {20000, 8, 8, 1}, {65535, 6, 6, 1}, {200, 96, 96, 1}, {2, 64, 96, 2}, {1, 64, 96, 0}, {4, 1080, 1920, 0}, {16, 651, 64, 0}, {3, 300000, 8, 0}})
        if (harris_launch::grouped_dealing(c[0], c[1], c[2], harris_launch::grouped_wide(c[0], c[1], c[2])) != c[3]) {
            std::printf("dealing of %d images of %dx%d\n", c[0], c[1], c[2]);
            return 1;
        }
    // Groupings: four pixels of two rows per thread only for images that give a row of threads work.
    for (const auto& c : {std::vector<int>{500, 40, 40}, {20000, 8, 8}, {3, 300000, 8}, {16, 7812, 64}, {1, 600, 800}})
        if (harris_launch::grouped_wide(c[0], c[1], c[2])) { std::printf("wide groupings of %d images of %dx%d\n", c[0], c[1], c[2]); return 1; }
    for (const auto& c : {std::vector<int>{1, 1080, 1920}, {64, 128, 128}, {16, 651, 96}, {1, 720, 1000}})
        if (!harris_launch::grouped_wide(c[0], c[1], c[2])) { std::printf("narrow groupings of %d images of %dx%d\n", c[0], c[1], c[2]); return 1; }
    // The widest images: the number of workgroups across them.
    for (int each : {4, 8, 64, 256})
        for (int size : {1, each, each + 1, 0x7fffffff - 256, 0x7fffffff - 64, 0x7fffffff - 4, 0x7fffffff})
            if (harris_launch::groups_covering(size, each) != (unsigned)(((long long)size + each - 1) / each)) { std::printf("workgroups for %d by %d\n", size, each); return 1; }
    if (packed == 0 || gaps_packed == 0 || pairs < 100) { std::printf("the narrow-image kernel was never planned\n"); return 1; }
    std::printf("ok %d\n", harris_launch::launches);
    return 0;
}
