// Host check of the compact kernel arguments (namespaces compact and compact_patch of harris_launch.h): over random calls of
// the C interface, what a kernel unpacks is what the planner decided, or the launch takes the kernels with whole
// arguments; and the division they use is exact.  Built and run by tests/test_abi_host.py; prints "ok ..." or the first fault.
#include <array>
#include <cfloat>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <initializer_list>

#include "harris_launch.h"

namespace harris_launch {

static long long tiles = 0, patches = 0, far = 0;
static int far_px = 0;
static long long far_blocks = 0;
static bool wrong = false;

#define SAME(a, b) do { if ((a) != (b)) { std::printf("%s is not %s\n", #a, #b); wrong = true; } } while (0)
template <typename T>
static void same_bits(const T& a, const T& b, const char* what) {
    if (std::memcmp(&a, &b, sizeof(T)) != 0) { std::printf("%s differs\n", what); wrong = true; }
}

static void check_tile(const Params& p, const harris_tuning& shape, int dtype) {
    const unsigned elem = dtype == HARRIS_U8 ? 1u : 4u;
    const compact::Params c = compact::pack(p, (int)elem);
    const compact::Tile t = compact::unpack(c, elem, shape.rows), w = compact::unpack(p, elem, shape.rows);
    SAME(t.rgb, w.rgb); SAME(t.out, w.out);
    SAME(t.in_row_pitch, w.in_row_pitch); SAME(t.in_plane_pitch, w.in_plane_pitch); SAME(t.in_image_pitch, w.in_image_pitch);
    SAME(t.out_row_bytes, w.out_row_bytes); SAME(t.out_image_bytes, w.out_image_bytes);
    SAME(t.H, w.H); SAME(t.W, w.W); SAME(t.n, w.n); SAME(t.m, w.m); SAME(t.rows_per_band, w.rows_per_band);
    SAME(t.n_strips, w.n_strips); SAME(t.strip_pitch, w.strip_pitch); SAME(t.strip_reach, w.strip_reach);
    SAME(t.n_blocks, w.n_blocks); SAME(t.chunk, w.chunk); SAME(t.waves_per_block, w.waves_per_block);
    SAME(t.flags, w.flags & (HARRIS_TUNE_NO_XCD_REMAP | HARRIS_TUNE_ALIGNED_STORES | kWriteThrough));
    SAME(t.out_kind, w.out_kind); SAME(t.out_shift, w.out_shift);
    if (dtype == HARRIS_U8) { same_bits(t.gain, w.gain, "gain"); same_bits(t.more_gain, w.more_gain, "more_gain"); }
    else { same_bits(t.wr, w.wr, "wr"); same_bits(t.wg, w.wg, "wg"); same_bits(t.wb, w.wb, "wb"); }
    same_bits(t.k, w.k, "k"); same_bits(t.q_scale, w.q_scale, "q_scale"); same_bits(t.q_offset, w.q_offset, "q_offset");
    for (unsigned tile : {0u, 1u, p.n_strips - 1u, p.n_strips, p.tiles_per_image - 1u, p.tiles_per_image, p.n_blocks / 2u, p.n_blocks - 1u}) {
        SAME(compact::image_of(c, tile), tile / p.tiles_per_image);
        SAME(compact::band_of(c, tile % p.tiles_per_image), tile % p.tiles_per_image / p.n_strips);
    }
}

// The rows that a wavefront loads at 32-bit offsets are the image's, wherever it lies in a plane of any size: wavefronts at either end of the image, and where
// what is left of the plane comes to just less and just more than a multiple of 4 GB.
static void check_rows(const Params& p, const harris_tuning& shape, int dtype) {
    const unsigned elem = dtype == HARRIS_U8 ? 1u : 4u;
    const long long pitch = p.in_row_pitch * elem;
    const auto rows_of = [&](long long y) {
        if (y < 0 || y > p.H + shape.rows * 16LL) return;
        const NearRows r = near_rows(p.H, (int)(y < p.H ? y : p.H - 1), (unsigned)pitch, shape.rows, dtype == HARRIS_U8);
        const long long left = p.H - 1 - y;
        for (int t = 0; t < shape.rows; ++t) {
            const long long at = (left < 0 ? 0 : left < t ? left : t) * pitch;
            if (near_row(r, t) != (unsigned long long)at || at + (long long)p.W * elem > 1LL << 31) {
                std::printf("%d rows of %lld bytes: row %d of the wavefront at %lld loaded at %u, not %lld\n", p.H, pitch, t, y, near_row(r, t), at);
                wrong = true;
                return;
            }
        }
    };
    for (long long y : {0LL, (long long)shape.rows, p.H / 2LL, p.H - 11LL, p.H - 5LL, p.H - 2LL, p.H - 1LL, (long long)p.H, p.H + 5LL}) rows_of(y);
    for (long long end = 1LL << 32; end / pitch < p.H && end <= 16LL << 32; end += 1LL << 32)
        for (int o = -2; o <= 12; ++o) rows_of(p.H - 1 - end / pitch - o);
}

static void check_patch(const Params& p, int dtype) {
    const compact_patch::Params c = compact_patch::pack(p, dtype == HARRIS_U8 ? 1 : 4);
    const Params t = compact_patch::unpack(c);
    SAME(t.rgb, p.rgb); SAME(t.out, p.out);
    SAME(t.in_row_pitch, p.in_row_pitch); SAME(t.in_plane_pitch, p.in_plane_pitch); SAME(t.in_image_pitch, p.in_image_pitch);
    SAME(t.out_row_pitch, p.out_row_pitch); SAME(t.out_image_pitch, p.out_image_pitch);
    SAME(t.H, p.H); SAME(t.W, p.W); SAME(t.n, p.n); SAME(t.m, p.m); SAME(t.rows_per_band, p.rows_per_band);
    SAME(t.tiles_per_image, p.tiles_per_image); SAME(t.n_blocks, p.n_blocks); SAME(t.chunk, p.chunk); SAME(t.batch, p.batch);
    SAME(t.image_lanes, p.image_lanes); SAME(t.image_lanes_inverse, p.image_lanes_inverse); SAME(t.images, p.images);
    if (dtype == HARRIS_U8) same_bits(t.gain, p.gain, "gain");
    else { same_bits(t.wr, p.wr, "wr"); same_bits(t.wg, p.wg, "wg"); same_bits(t.wb, p.wb, "wb"); }
    same_bits(t.k, p.k, "k");
    for (unsigned tile : {0u, p.tiles_per_image - 1u, p.tiles_per_image, p.n_blocks / 2u, p.n_blocks - 1u}) SAME(compact_patch::group_of(c, tile), tile / p.tiles_per_image);
}

int launch(const Params& p, const harris_tuning& shape, long long n_blocks, int dtype, void*) {
    if (n_blocks != (long long)p.n_blocks) return HARRIS_ERR_LAUNCH;
    if (shape.schedule != HARRIS_SCHEDULE_TILES) return HARRIS_OK;
    if (shape.flags & HARRIS_TUNE_PACKED_IMAGES) { ++patches; check_patch(p, dtype); return HARRIS_OK; }
    if (p.far_rows) {
        ++far; far_px = shape.px; far_blocks = n_blocks;
        if (shape.rows != 4 || !(shape.px == 4 || shape.px == 1) || (shape.flags & HARRIS_TUNE_FLAG_HANDOFF) || ((shape.flags & HARRIS_TUNE_WORD_STORES) && shape.px != 4)) { std::printf("no such far kernel\n"); wrong = true; }
        return HARRIS_OK;
    }
    ++tiles;
    const harris_layout lay = {p.in_row_pitch, p.in_plane_pitch, p.in_image_pitch, p.out_row_pitch, p.out_image_pitch};
    if (!compact::fits(lay, 0, 1 << p.out_shift) || rows_are_far(p.in_row_pitch, p.W, dtype == HARRIS_U8 ? 1 : 4, shape.rows)) { std::printf("does not fit\n"); wrong = true; }
    check_tile(p, shape, dtype);
    check_rows(p, shape, dtype);
    return HARRIS_OK;
}
size_t grouped_workspace_floats(int, int, int, int) { return 0; }
int launch_grouped(const void*, int, int, int, int, float, float, int, int, float*, float*, void*) { return HARRIS_ERR_LAUNCH; }
float* scratch_of_current_device() { return nullptr; }
int launch_copy_probe(const void*, int, int, int, int, float*, void*) { return HARRIS_ERR_LAUNCH; }
int launch_stream_probe(int, const void*, void*, long long, void*) { return HARRIS_ERR_LAUNCH; }

}  // namespace harris_launch

static uint64_t state = 0x9e3779b97f4a7c15ull;
static uint32_t next_u32() {
    state ^= state << 13; state ^= state >> 7; state ^= state << 17;
    return (uint32_t)(state >> 16);
}
static long long below(long long n) { return (long long)(next_u32() % (uint64_t)n); }
static long long spread(int bits) { return 1 + below(1LL << below(bits + 1)); }      // over the logarithm

static bool divides(uint32_t x, uint32_t d) {
    namespace c = harris_launch::compact;
    if (c::divide(x, c::divide_mul(d), c::divide_shift(d)) == x / d) return true;
    std::printf("mismatch: %u / %u\n", x, d);
    return false;
}

int main() {
    for (uint32_t d = 1; d <= 1024; ++d) {
        for (uint32_t x = 0; x <= 3072; ++x) if (!divides(x, d)) return 1;
        for (uint32_t q = 0x7fffffffu / d, i = 0; i < 3; ++i, --q) for (uint32_t o = 0; o < 2; ++o) if (q * d + o >= 1u && q * d + o - 1u <= 0x7fffffffu && !divides(q * d + o - 1u, d)) return 1;
    }
    for (int l = 1; l <= 31; ++l)
        for (int o = -2; o <= 2; ++o) {
            const uint32_t d = (uint32_t)((1ull << l) + o);
            if (d == 0u || d > 0x80000000u) continue;
            for (uint32_t x : {0u, 1u, d - 1u, d, d + 1u, 0x7ffffffeu, 0x7fffffffu}) if (x <= 0x7fffffffu && !divides(x, d)) return 1;
            for (int i = 0; i < 4000; ++i) if (!divides(next_u32() >> 1, d)) return 1;
        }
    for (int i = 0; i < 2000000; ++i) {
        uint32_t d = next_u32() >> (1 + next_u32() % 31);
        if (!divides(next_u32() >> 1, d == 0u ? 1u : d)) return 1;
    }

    // The factor of 8-bit results: one float32 where that holds it, else two of which neither is subnormal while the result may be a normal number.
    for (int e = -700; e <= 700; ++e)
        for (double x : {1.0, 1.25, 1.9999999}) {
            const double gain = std::ldexp(x, e);
            float a, b;
            harris_launch::split_gain(gain, a, b);
            const bool held = gain >= FLT_MIN && gain <= FLT_MAX;
            if ((held && (a != (float)gain || b != 1.0f)) || !(a >= FLT_MIN && a <= FLT_MAX) || !(b <= FLT_MAX) || (e >= -200 && b < FLT_MIN) ||
                (e >= -200 && e <= 200 && std::fabs((double)a * (double)b - gain) > std::ldexp(gain, -24))) { std::printf("factor %g: %g and %g\n", gain, a, b); return 1; }
        }

    // Large constants k: the same product with the factor, and small enough for the square of any trace.
    for (float k : {0.0f, 0.04f, -1e19f, 1.8e19f, 1.9e19f, -1e30f, FLT_MAX, -FLT_MAX, FLT_MIN}) {
        float bounded = k;
        double gain = 1e-20;
        harris_launch::bound_k(bounded, gain);
        if (std::fabs(bounded) > std::ldexp(1.0, 64) || (std::fabs(k) < 1.8e19f && (bounded != k || gain != 1e-20)) ||
            std::fabs((double)bounded * gain - (double)k * 1e-20) > 1e-15 * std::fabs((double)k * 1e-20) || (std::fabs(k) > 2e19f && std::fabs(bounded) < std::ldexp(1.0, 63))) {
            std::printf("k %g: %g, factor %g\n", k, bounded, gain);
            return 1;
        }
    }

    void *rgb = reinterpret_cast<void*>(4096), *out = reinterpret_cast<void*>(1 << 20);
    for (int i = 0; i < 400000 && !harris_launch::wrong; ++i) {
        const int dtype = (int)below(2), kind = (int)below(4), batch = (int)(below(3) ? spread(12) : 1);
        const int H = 4 + (int)spread(below(8) ? 13 : 24), W = 4 + (int)spread(below(8) ? 13 : 27);
        harris_layout lay = {W, (long long)H * W, 3LL * H * W, W - 4, (long long)(H - 4) * (W - 4)};
        if (below(3) == 0) {
            lay.rgb_row_pitch += below(2) ? below(64) : spread(31);
            lay.rgb_plane_pitch = lay.rgb_row_pitch * H + (below(2) ? 0 : spread(34));
            lay.rgb_image_pitch = 3 * lay.rgb_plane_pitch + (below(2) ? 0 : spread(34));
            lay.out_row_pitch += below(2) ? below(64) : spread(32);
            lay.out_image_pitch = lay.out_row_pitch * H + (below(2) ? 0 : spread(34));
        }
        harris_tuning t = {(int)below(2) * HARRIS_SCHEDULE_TILES, (int)below(2) * 4, 0, 0, 0, 0u, 0};
        if (below(3) == 0) { static const int rows[] = {0, 4, 5, 6, 8, 9, 10}; t.rows = rows[below(7)]; t.waves_per_block = 2 + (int)below(15); t.flags = (unsigned)below(1024); }
        const harris_tuning* tuning = below(2) ? &t : nullptr;
        const char* at = static_cast<const char*>(rgb) + (dtype == HARRIS_U8 ? below(4) : 4 * below(4));
        if (kind == HARRIS_OUT_U8) harris_coarsity_quantized(at, dtype, batch, H, W, &lay, 0.04f, 0.5f, (int)below(2), 1.5f, 90.0f, static_cast<uint8_t*>(out), tuning, nullptr);
        else harris_coarsity_typed(at, dtype, batch, H, W, &lay, 0.04f, 2.0f, (int)below(2), out, kind, tuning, nullptr);
    }
    // Images of more than 2^32 pixels: as many pixels per lane as smaller ones have, {input, result, images, height, width, pixels per lane}.
    for (const auto& c : {std::array<int, 6>{HARRIS_U8, HARRIS_OUT_F16, 1, 66001, 66001, 4}, {HARRIS_F32, HARRIS_OUT_BF16, 1, 66001, 66001, 4}, {HARRIS_U8, HARRIS_OUT_U8, 2, 40001, 36001, 4},
                          {HARRIS_U8, HARRIS_OUT_F32, 2, 40001, 36001, 4}, {HARRIS_F32, HARRIS_OUT_F32, 2, 40000, 36000, 4}}) {
        const int before = (int)harris_launch::far;
        const int rc = c[1] == HARRIS_OUT_U8 ? harris_coarsity_quantized(rgb, c[0], c[2], c[3], c[4], nullptr, 0.04f, 1.0f, 0, 1.0f, 0.0f, static_cast<uint8_t*>(out), nullptr, nullptr)
                                             : harris_coarsity_typed(rgb, c[0], c[2], c[3], c[4], nullptr, 0.04f, 1.0f, 0, out, c[1], nullptr, nullptr);
        // The plan says so too, and is accepted.
        harris_tuning planned, again;
        long long blocks = 0;
        const int rp = harris_plan_typed(c[0], c[1], c[2], c[3], c[4], c[0] == HARRIS_U8 ? 1 : 4, c[1] == HARRIS_OUT_U8 ? 1 : c[1] == HARRIS_OUT_F32 ? 4 : 2, nullptr, &planned, &blocks) |
                       harris_plan_typed(c[0], c[1], c[2], c[3], c[4], c[0] == HARRIS_U8 ? 1 : 4, c[1] == HARRIS_OUT_U8 ? 1 : c[1] == HARRIS_OUT_F32 ? 4 : 2, &planned, &again, nullptr);
        if (c[4] % 2 != 0 && (rp != HARRIS_OK || planned.rows != 4 || planned.waves_per_block != 4 || blocks != harris_launch::far_blocks || std::memcmp(&planned, &again, sizeof again) != 0)) {
            std::printf("%d images of %dx%d, types %d and %d: planned %lld tiles of %d rows, launched %lld\n", c[2], c[3], c[4], c[0], c[1], blocks, planned.rows, harris_launch::far_blocks);
            return 1;
        }
        if (rc != HARRIS_OK || harris_launch::far != before + 1 || harris_launch::far_px != c[5]) {
            std::printf("%d images of %dx%d, types %d and %d: %d pixels per lane\n", c[2], c[3], c[4], c[0], c[1], harris_launch::far_px);
            return 1;
        }
    }
    // Scales whose factor takes two numbers: the kernels that multiply by both, whatever shape was asked for.
    for (float scale : {5e9f, 3e38f, 3e-10f, 1e-45f})
        for (int shape = 0; shape < 8 && !harris_launch::wrong; ++shape) {
            const harris_tuning t = {shape == 1 ? HARRIS_SCHEDULE_BANDS : shape ? HARRIS_SCHEDULE_TILES : 0, shape == 4 ? 2 : 0, shape == 2 ? 5 : 0, 0, 0, shape == 3 ? (unsigned)HARRIS_TUNE_PACKED_IMAGES : 0u, 0};
            const int kind = shape < 5 ? HARRIS_OUT_F32 : HARRIS_OUT_F16, before = (int)harris_launch::far;
            if (harris_coarsity_typed(rgb, HARRIS_U8, 40, 41, shape == 6 ? 71 : 72, nullptr, 0.04f, scale, 0, out, kind, shape < 6 ? &t : nullptr, nullptr) != HARRIS_OK || harris_launch::far != before + 1) {
                std::printf("scale %g, shape %d: not the kernel with two factors\n", scale, shape);
                return 1;
            }
        }
    if (harris_launch::wrong) return 1;
    if (harris_launch::tiles < 50000 || harris_launch::patches < 1000 || harris_launch::far < 1000) { std::printf("too few: %lld %lld %lld\n", harris_launch::tiles, harris_launch::patches, harris_launch::far); return 1; }
    std::printf("ok %lld tiles, %lld patches, %lld far\n", harris_launch::tiles, harris_launch::patches, harris_launch::far);
    return 0;
}
