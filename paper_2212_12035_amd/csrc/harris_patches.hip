// The tile schedule for batches of narrow images (patches): several images side by side in a wavefront.
//
// harris_tile_kernel gives every strip of an image a wavefront of its own, 64 lanes of four
// columns; an image of 64 columns keeps 16 of them busy.  Here a wavefront's lanes are cut into
// groups of W / 4 (rounded up), one image each, as many as fit.  All groups work on the same rows of
// their images, so rows stay uniform per wavefront and only the lanes' offsets differ.  The lane
// shift between neighbouring columns crosses from one group into the next, but only into a
// group's last lane, whose columns are halo: every result column c takes input columns up to c + 4
// < W, all of its own group.
//
// A workgroup of at most kPatchWaves wavefronts, four in large launches, holds whole images or bands of equal height: the
// four rows that two of its tiles would both read are read once.  Everything else is
// the tile kernel's barrier form (harris_kernels.h): all rows requested at once, four gray rows handed
// to the wavefront above through LDS, results stored in one burst.
//
// Bound by memory, at 4.5 to 5.6 TB/s for float32.  Input is loaded with the default policy: rows of a
// narrow image share their cache lines with the rows above and below, which other wavefronts of the
// workgroup load.  Results are stored non-temporal, not written through, for the same reason.  Default loads
// / non-temporal ones / results written through (us): 2048 images of 64x64 float32 26.9 / 28.5 / 30.9, uint8
// 12.1 / 14.7 / 17.2; 1000 of 65x65 float32 13.5 / 17.4 / 16.6; 300 of 128x128 13.8 / 16.6 / 15.6; 600 of 110x124
// uint8 11.5 / 14.6 / 15.0 (non-temporal loads gain with 1343 of 80x27 uint8, 9.1 / 7.9, and 5000 of 24x100
// float32, 37.8 / 36.9).
// Measured against one image per wavefront (harris_tile_kernel), then with eight wavefronts a workgroup: 2048 images of 64x64
// float32 26.9 us (38.4), 8192 of 32x32 27.9 (82.3), 1000 of 65x65 13.5 (24.0), 300 of 128x128 13.8 (16.0), 2048 of
// 64x64 uint8 12.1 (30.0), 1343 of 80x27 uint8 9.1 (30.2).  With four, dealt to the XCDs by turns: 2048 of 64x64 float32
// 22.4 us, 5.8 TB/s (24.9 where nothing is left in the last-level cache).
#include "harris_kernels.h"

namespace {

// One row of the three planes of a lane's image.  rows[c] is the row's first element in the group's
// first image, `bytes` what lies from there to the row's end in the group's last image; voff the
// lane's offset (patch_lane).  Loads beyond the end give zeros.  A float32 lane that straddles the end of its
// row reads the start of the row that follows it in memory, of whichever plane or image: the planner lets it
// where the images are dense, so that all of this belongs to the call.  Nobody uses it.
// 8-bit rows start on any byte: a lane loads its four bytes where they are, the last lane of a row the
// row's last four, which gray_row takes from where they stand.
__device__ __forceinline__ void load_patch_row(RawRow<float, 4>& r, const float* row, size_t plane, uint32_t bytes, uint32_t voff) {
    load_row<float, 4, kAuxDefault>(r, row, plane, bytes, voff);
}
__device__ __forceinline__ void load_patch_row(RawRow<uint8_t, 4>& r, const uint8_t* row, size_t plane, uint32_t, uint32_t voff) {
#pragma unroll
    for (int c = 0; c < 3; ++c) r.w[c][0] = *reinterpret_cast<const u32_any*>(row + c * plane + voff);
}

// Compiled as for workgroups of 1024 threads, twice what the planner launches: within the 64 vector registers that
// eight wavefronts per SIMD leave it needs no more, and the bound of 512 measures slower (673 images of 33x75
// uint8 5.23 us, 5.15 with 1024; 291 of 123x77 6.58 / 6.51; float32 the same).
//
// TURNS: a launch of several turns.  Smaller ones, which one latency bounds, have a workgroup per tile and less to
// work out before the first load (259 uint8 images of 49x30 4.39 us, dealt as turns are 4.48; 569 float32 of 68x20 4.68 / 4.76).
//
// PAIRS: narrow 8-bit images on any byte.  A load of four bytes that starts between words costs an access per half lane, a
// wavefront's 32 instead of one or a few, and these launches are bound by that: 1296 images of 111x17 took 9.80 us.  Here a
// lane loads the two aligned words around its four pixels and shifts them together: 6.43 us.
template <typename In, bool BINOM, bool TURNS, bool PAIRS>
__global__ __launch_bounds__(2 * kWave * harris_launch::kPatchWaves) void harris_patch_kernel(const harris_launch::compact_patch::Params args) {
    const harris_launch::Params p = harris_launch::compact_patch::unpack(args);
    constexpr int PX = 4, RW = 4;
    constexpr bool F32 = std::is_same<In, float>::value;
    extern __shared__ __align__(16) float halo_lds[];           // [NW][4][64][PX]

    const unsigned lane = threadIdx.x % kWave;
    const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    // At the end of the last turn there may be workgroups without a tile: they go through the last one's motions with
    // rows below the image, storing nothing (and loading nothing from float32; the last row again from 8-bit input).  (A
    // branch here would part the loads of the arguments in two, one behind the other: 256 images of 64x64 6.77 us, 6.3 without.)
    unsigned tile;
    int idle = 0;
    if constexpr (TURNS) {
        unsigned n_blocks = p.n_blocks, chunk = p.chunk;
        asm volatile("" : "+s"(n_blocks), "+s"(chunk));
        const unsigned dealt = harris_launch::dealt_tile(blockIdx.x, blockIdx.y, chunk);
        tile = min(dealt, n_blocks - 1);
        idle = dealt < n_blocks ? 0 : 1 << 30;
    } else {
        tile = xcd_contiguous(blockIdx.x, p.n_blocks);
    }
    const unsigned group = harris_launch::compact_patch::group_of(args, tile);      // of p.images images
    const int band = (int)(tile - group * p.tiles_per_image);

    const int tile_rows = p.rows_per_band;
    const int y_wave = band * tile_rows + (int)wave * RW + idle;
    const int y_end = min(p.n, (band + 1) * tile_rows);
    const int out_rows = max(0, min(RW, y_end - y_wave));

    const unsigned images = min(p.images, p.batch - group * p.images);   // of this group
    const harris_launch::PatchLane l = harris_launch::patch_lane(p, images, lane, sizeof(In));
    const unsigned col = l.col;
    const bool live = l.live;

    const size_t first = (size_t)group * p.images;
    const In* in = static_cast<const In*>(p.rgb) + first * (size_t)p.in_image_pitch;
    float* out = static_cast<float*>(p.out) + first * (size_t)p.out_image_pitch;
    const uint32_t out_image = (uint32_t)(p.out_image_pitch * sizeof(float));
    const uint32_t out_bytes = (images - 1) * out_image + (uint32_t)p.m * 4u;

    RawRow<In, PX> raw[RW];
    const size_t plane = (size_t)p.in_plane_pitch;
    [[maybe_unused]] u32x2 pair[RW][3];
    [[maybe_unused]] uint32_t first_byte;                       // the lane's column in its image's first row, from the aligned word at or before the group
    const auto row_offset = [&](int t, int c) { return harris_launch::patch_row(p, y_wave + t, c); };
    if constexpr (PAIRS) {
        const uintptr_t at = reinterpret_cast<uintptr_t>(in);
        const uint32_t lead = (uint32_t)at & 3u;
        // The end is the end of the word that holds the group's last byte; a word that begins past it is dropped by itself.
        // Columns past W and rows past H hold other pixels of the group, and no stored result depends on them.
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(reinterpret_cast<const void*>(at - lead), harris_launch::patch_words_end(p, images, lead));
        first_byte = harris_launch::patch_first_byte(p, l, lead);
        static_for<0, RW>([&](auto tt) {
            constexpr int t = decltype(tt)::value;
#pragma unroll
            for (int c = 0; c < 3; ++c) pair[t][c] = __builtin_amdgcn_raw_buffer_load_b64(rs, (first_byte + row_offset(t, c)) & ~3u, 0, kAuxDefault);
        });
    } else {
        static_for<0, RW>([&](auto tt) {
            constexpr int t = decltype(tt)::value;
            const int r = y_wave + t;
            load_patch_row(raw[t], in + (size_t)min(r, p.H - 1) * (size_t)p.in_row_pitch, plane, r < p.H ? l.in_bytes : 0u, l.in_voff);
        });
    }
    __builtin_amdgcn_sched_barrier(0);

    constexpr int ORDER = F32 ? kDifferences : kQuads;
    LineBuffers<PX> lb;
    const Coarsity cs = {p.k, p.gain};
    [[maybe_unused]] GrayMatrix gray;
    if constexpr (!F32) gray = gray_matrix(lane, PAIRS ? 0u : l.drop);
    float gc[PX], none[PX], results[RW][PX];
    float* my_halo = halo_lds + ((size_t)wave * 4 * kWave + lane) * PX;
    static_for<0, RW>([&](auto tt) {
        constexpr int t = decltype(tt)::value;
        if constexpr (PAIRS) {
#pragma unroll
            for (int c = 0; c < 3; ++c) raw[t].w[c][0] = __builtin_amdgcn_alignbyte(pair[t][c].y, pair[t][c].x, (first_byte + row_offset(t, c)) & 3u);
        }
        if constexpr (F32) gray_row<In, PX>(raw[t], p.wr, p.wg, p.wb, gc);
        else gray_row(raw[t], gray, gc);
#pragma unroll
        for (int i = 0; i < PX; ++i) my_halo[(size_t)t * kWave * PX + i] = gc[i];
        row_step<(t < 2 ? 0 : 1), t, PX, BINOM, ORDER>(lb, gc, cs, none);
        __builtin_amdgcn_sched_barrier(0);
    });
    __syncthreads();
    if (out_rows <= 0) return;                                  // the last wavefront only supplies rows; no barrier follows
    const float* below = my_halo + (size_t)4 * kWave * PX;      // out_rows > 0: there is a wavefront below (planner)
    static_for<RW, RW + 4>([&](auto tt) {
        constexpr int t = decltype(tt)::value;
#pragma unroll
        for (int i = 0; i < PX; ++i) gc[i] = below[(size_t)(t - RW) * kWave * PX + i];
        row_step<2, t, PX, BINOM, ORDER>(lb, gc, cs, results[t - 4]);
        pin_values<PX>(results[t - 4]);
    });
    __builtin_amdgcn_sched_barrier(0);

    const unsigned m = (unsigned)p.m, rest = m & 3u;
    const uint32_t at = l.image * out_image + col * 4u;
    const uint32_t whole_voff = live && col + 4u <= m ? at : 0x80000000u;
    const bool straddles = live && col < m && col + 4u > m;     // the row's last `rest` columns
    const uint32_t pair_voff = straddles && rest >= 2u ? at : 0x80000000u;
    const uint32_t single_voff = straddles && (rest & 1u) ? at + (rest & 2u) * 4u : 0x80000000u;
    static_for<0, RW>([&](auto jj) {
        constexpr int j = decltype(jj)::value;
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(out + (size_t)(y_wave + j) * (size_t)p.out_row_pitch, j < out_rows ? out_bytes : 0u);
        store_row<PX, kAuxStore>(results[j], rs, whole_voff);
        if (rest != 0u) {
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(results[j][0]), __float_as_uint(results[j][1])}, rs, pair_voff, 0, kAuxStore);
            const uint32_t r0 = __float_as_uint(results[j][0]), r2 = __float_as_uint(results[j][2]);
            __builtin_amdgcn_raw_buffer_store_b32((rest & 2u) ? r2 : r0, rs, single_voff, 0, kAuxStore);
        }
    });
}

}  // namespace

namespace {

template <typename In, bool PAIRS>
void enqueue(const harris_launch::Params& p, dim3 block, hipStream_t stream) {
    const dim3 one(p.n_blocks), turns(8 * p.chunk, p.turns);
    const harris_launch::compact_patch::Params c = harris_launch::compact_patch::pack(p, sizeof(In));
    if (p.turns == 1 && p.binomial) hipLaunchKernelGGL((harris_patch_kernel<In, true, false, PAIRS>), one, block, p.lds_bytes, stream, c);
    else if (p.turns == 1) hipLaunchKernelGGL((harris_patch_kernel<In, false, false, PAIRS>), one, block, p.lds_bytes, stream, c);
    else if (p.binomial) hipLaunchKernelGGL((harris_patch_kernel<In, true, true, PAIRS>), turns, block, p.lds_bytes, stream, c);
    else hipLaunchKernelGGL((harris_patch_kernel<In, false, true, PAIRS>), turns, block, p.lds_bytes, stream, c);
}

}  // namespace

namespace harris_launch {

int launch_patches(const Params& p, int dtype, unsigned block, void* stream_) {
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    if (dtype != HARRIS_U8) enqueue<float, false>(p, dim3(block), stream);
    else if (patch_in_pairs(p)) enqueue<uint8_t, true>(p, dim3(block), stream);
    else enqueue<uint8_t, false>(p, dim3(block), stream);
    return (int)hipGetLastError();
}

}  // namespace harris_launch
