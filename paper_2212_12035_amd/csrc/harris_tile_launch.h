// Host-side selection of a tile-kernel instance from a planned launch; included by the
// translation units that instantiate harris_tile_kernel (two per input type, one of them for result
// rows on any byte, so that they compile in parallel).
#ifndef HARRIS_TILE_LAUNCH_H
#define HARRIS_TILE_LAUNCH_H

#include "harris_kernels.h"

namespace {

// Enqueues the instance that the other arguments and the call's flags name.
template <typename In, int PX, int RW, int LAUX, bool HANDOFF, bool SHIFTED, bool WORDS>
hipError_t launch_tile_kernel(const harris_launch::Params& p, dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
    const harris_launch::compact::Params c = harris_launch::compact::pack(p, sizeof(In));
    if constexpr (std::is_same<In, uint8_t>::value && PX == 4 && RW == 4 && LAUX == kAuxKeepShared && !WORDS) {
        if (p.resident) {
            if (p.binomial) hipLaunchKernelGGL((harris_tile_kernel<In, PX, RW, LAUX, true, HANDOFF, SHIFTED, true, WORDS>), grid, block, lds, stream, c);
            else hipLaunchKernelGGL((harris_tile_kernel<In, PX, RW, LAUX, false, HANDOFF, SHIFTED, true, WORDS>), grid, block, lds, stream, c);
            return hipGetLastError();
        }
    }
    if (p.binomial) hipLaunchKernelGGL((harris_tile_kernel<In, PX, RW, LAUX, true, HANDOFF, SHIFTED, false, WORDS>), grid, block, lds, stream, c);
    else hipLaunchKernelGGL((harris_tile_kernel<In, PX, RW, LAUX, false, HANDOFF, SHIFTED, false, WORDS>), grid, block, lds, stream, c);
    return hipGetLastError();
}

// Rows too far apart for 32-bit offsets, pitches too long for the compact arguments, or a factor of two numbers (Params::far_rows).
// Four pixels per lane keep the shared rows and are dealt by turns, like near ones; to 8-bit codes, which the vector and scalar units bound, 8-bit
// images are faster with one policy and one run per XCD (ms, by turns / one run: 66000x66000 to codes 4.40 / 4.25, to
// float32 5.58 / 5.77; 2 of 40000x36000 float32 7.85 / 8.53), as long as the grid stays below 2^32 threads.
template <typename In, int PX, int LAUX, bool SHIFTED, bool WORDS>
hipError_t launch_far_tiles(const harris_launch::Params& p, dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
    if (LAUX == kAuxFarKeepShared) grid = dim3(8 * p.chunk, p.turns);
    if (p.binomial) hipLaunchKernelGGL((harris_far_tile_kernel<In, PX, LAUX, true, SHIFTED, WORDS>), grid, block, lds, stream, p);
    else hipLaunchKernelGGL((harris_far_tile_kernel<In, PX, LAUX, false, SHIFTED, WORDS>), grid, block, lds, stream, p);
    return hipGetLastError();
}

// WORDS: result rows on any byte, four pixels per lane.  Rows of 8-bit input
// are then always loaded that way too (the planner takes them so wherever a row is not naturally aligned).
template <typename In, int PX, int RW, bool WORDS>
hipError_t launch_tiles(const harris_launch::Params& p, dim3 grid, dim3 block, hipStream_t stream) {
    constexpr bool U8 = std::is_same<In, uint8_t>::value;
    // The rows that the wavefronts publish; the planner may reserve more to bound the number of workgroups resident
    // on a CU.
    const size_t lds_needed = harris_launch::tile_lds_bytes(U8, PX, block.x / kWave);
    const size_t lds = p.lds_bytes > lds_needed ? p.lds_bytes : lds_needed;
    if (p.far_rows) {
        if constexpr (RW == 4 && PX == 1) return launch_far_tiles<In, PX, kAuxFar, false, false>(p, grid, block, lds, stream);
        if constexpr (RW == 4 && PX == 4 && U8) {
            if (p.in_shifted) return launch_far_tiles<In, PX, kAuxFarKeepShared, true, WORDS>(p, grid, block, lds, stream);
            if constexpr (!WORDS) {
                if (p.out_kind == HARRIS_OUT_U8 && p.n_blocks < (1u << 23)) return launch_far_tiles<In, PX, kAuxFar, false, false>(p, grid, block, lds, stream);
            }
        }
        if constexpr (RW == 4 && PX == 4 && !(U8 && WORDS)) return launch_far_tiles<In, PX, kAuxFarKeepShared, false, WORDS>(p, grid, block, lds, stream);
        return hipErrorInvalidValue;
    }
    // Many tiles with shared rows kept: dealt to the XCDs by turns (dealt_tile).
    if ((p.flags & HARRIS_TUNE_KEEP_SHARED_ROWS) && !(p.flags & HARRIS_TUNE_NO_XCD_REMAP)) grid = dim3(8 * p.chunk, p.turns);
    const bool cached = p.flags & HARRIS_TUNE_CACHED_LOADS, keep = p.flags & HARRIS_TUNE_KEEP_SHARED_ROWS, handoff = p.flags & HARRIS_TUNE_FLAG_HANDOFF;
    if constexpr (U8 && PX == 4 && (RW == 4 || RW == 8)) {
        // 8-bit rows on any byte: kernels for 4 and 8 rows per wavefront, barrier hand-over.
        if (p.in_shifted) {
            if (handoff) return hipErrorInvalidValue;
            if (keep) return launch_tile_kernel<In, PX, RW, kAuxKeepShared, false, true, WORDS>(p, grid, block, lds, stream);
            if (cached) return launch_tile_kernel<In, PX, RW, kAuxDefault, false, true, WORDS>(p, grid, block, lds, stream);
            return launch_tile_kernel<In, PX, RW, kAuxNonTemporal, false, true, WORDS>(p, grid, block, lds, stream);
        }
    }
    if (p.in_shifted) return hipErrorInvalidValue;
    if constexpr (!(U8 && WORDS)) {
        // The hand-over by ready flags (float32 input only) and the mixed load policy exist for 16-byte
        // lanes only (the planner asks for them nowhere else).
        if constexpr (PX == 4) {
            if (handoff) {
                if constexpr (!U8) return launch_tile_kernel<In, PX, RW, kAuxNonTemporal, true, false, WORDS>(p, grid, block, lds, stream);
                else return hipErrorInvalidValue;
            }
            if (keep) return launch_tile_kernel<In, PX, RW, kAuxKeepShared, false, false, WORDS>(p, grid, block, lds, stream);
        }
        if (cached) return launch_tile_kernel<In, PX, RW, kAuxDefault, false, false, WORDS>(p, grid, block, lds, stream);
        return launch_tile_kernel<In, PX, RW, kAuxNonTemporal, false, false, WORDS>(p, grid, block, lds, stream);
    } else {
        return hipErrorInvalidValue;
    }
}

// Tile kernels exist for 4 rows per wavefront at every lane width, and for 5, 6, 8, 9 and 10
// rows with four pixels per lane.
template <typename In, bool WORDS>
hipError_t launch_tiles_any(const harris_launch::Params& p, const harris_tuning& t, dim3 grid, dim3 block, hipStream_t stream) {
    if constexpr (!WORDS) {
        if (t.rows == 4 && t.px == 1) return launch_tiles<In, 1, 4, false>(p, grid, block, stream);
        if (t.rows == 4 && t.px == 2) return launch_tiles<In, 2, 4, false>(p, grid, block, stream);
    }
    if (t.px != 4) return hipErrorInvalidValue;
    switch (t.rows) {
        case 4: return launch_tiles<In, 4, 4, WORDS>(p, grid, block, stream);
        case 5: return launch_tiles<In, 4, 5, WORDS>(p, grid, block, stream);
        case 6: return launch_tiles<In, 4, 6, WORDS>(p, grid, block, stream);
        case 8: return launch_tiles<In, 4, 8, WORDS>(p, grid, block, stream);
        case 9: return launch_tiles<In, 4, 9, WORDS>(p, grid, block, stream);
        case 10: return launch_tiles<In, 4, 10, WORDS>(p, grid, block, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

#endif  // HARRIS_TILE_LAUNCH_H
