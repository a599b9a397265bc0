// Unfused and partly fused Harris pipelines: the kernel groupings of the thesis's chapter 3,
// section "Explicit Kernel Execution", subsection "Evaluating the Boilerplate Avoided through
// Kernel Execution" (table "Four different kernel groupings"), as plain HIP kernels that keep
// every intermediate image in device memory.
//
//   grouping 1: [gray] [Sx] [Sy] [x] [x] [x] [+] [+] [+] [coarsity]
//   grouping 2: [gray] [Sx, Sy, x]  [+, coarsity]
//   grouping 3: [gray] [Sx, Sy]     [x, +, coarsity]
//   grouping 4: everything in one kernel: that is harris_coarsity_ex itself
//
// (The thesis's table starts from a grayscale image; the grayscale stage is a kernel
// of its own here.)  They exist to measure what fusion buys on this GPU with the same
// harness, and as a second GPU implementation that shares no code with the fused
// kernels: no LDS, no lane exchange, no separation of the 3x3 kernels.  What bounds them is what
// they are compared for, the intermediate images' way through memory and one launch per kernel, so
// a thread takes four neighbouring pixels (16-byte accesses; rows of width W-2 and W-4 start on 4-byte
// boundaries, which is all that global accesses of several words need) and, where it reads a 3x3
// neighbourhood, two rows of them, so that a tap is loaded 1.5 x 2 times instead of 9.
// One 1080x1920 float32 image, groupings 1, 2 and 3 together: 90.4 us (one pixel per thread and one row: 119 us with
// workgroups dealt out one by one).

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>
#include <mutex>

#include "harris_launch.h"

// Intermediate images for harris_coarsity_grouped_static: callers that cannot allocate (code
// under stream capture, serving loops) get the groupings' workspace from here.  Each GPU the
// library runs on holds its own copy of the array, at its own address, until the process ends.
// Host code never uses this name as an address: it asks for the device's address once per
// device (scratch_of_current_device) and hands that pointer to the kernels.
static __device__ __align__(256) float scratch[HARRIS_GROUPED_SCRATCH_BYTES / sizeof(float)];

namespace {

using harris_launch::groups_covering;

// Kernels are templates over a thread's neighbouring pixels PX (4 or 1), and rows ROWS in the 3x3 stages
// (2 or 1); grouped_wide says which.
constexpr int kTileX = 64, kTileY = 4, kThreads = kTileX * kTileY;      // 64 PX columns of 4 ROWS rows

// Where a workgroup works.  Grids are 8 x chunk workgroups an image (grouped_grid): the hardware deals them out to the
// eight XCDs one by one, and each XCD takes one run of neighbours.  The rows that two of its workgroups both read, and
// most of what the kernel before has just written, are then behind the same L2; with two-dimensional grids dealt out one
// by one the three groupings of 1600x2400 took 151 us, now 138, 1080x1920 98.2 / 90.4, 480x640 41.5 / 37.6, 4
// images of 1080x1920 289 / 270.  Workgroups beyond the last have nothing to do.
//
// That is kRunOfEach, for images of many workgroups: runs end in workgroups without work, up to seven an image.  Batches of
// smaller images take a run of images to an XCD, and a workgroup divides for its own (kRunOfImages), or are left in
// order (kInOrder); grouped_dealing says when.
using harris_launch::GroupedDealing;
using harris_launch::kInOrder;
using harris_launch::kRunOfEach;
using harris_launch::kRunOfImages;
template <GroupedDealing DEALING>
struct Blocks {
    unsigned chunk;                         // workgroups of an XCD
    unsigned across;                        // workgroups across an image (3x3 stages)
    harris_launch::FastDiv by_across;
};
template <>
struct Blocks<kRunOfImages> : Blocks<kRunOfEach> {
    unsigned total, per_image;              // workgroups that have something to do, and of an image
    harris_launch::FastDiv by_image;
};
// Image and workgroup of it, or false.
template <GroupedDealing DEALING>
__device__ __forceinline__ bool place(const Blocks<DEALING>& blocks, unsigned& image, unsigned& b) {
    b = DEALING == kInOrder ? blockIdx.x : harris_launch::dealt_tile(blockIdx.x, blockIdx.y, blocks.chunk);
    image = blockIdx.z;
    if constexpr (DEALING == kRunOfImages) {
        if (b >= blocks.total) return false;
        image = harris_launch::fastdiv(b, blocks.by_image);
        b -= image * blocks.per_image;
    }
    return true;
}

typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float f2 __attribute__((ext_vector_type(2), aligned(4)));
typedef uint32_t word_any __attribute__((aligned(1)));

// N values from p on, of which the first `left` (>= 1) exist; the others are 0.  One value, and the three of a
// row that one pixel takes, always exist: a check of each would put every tap behind a branch (the three
// groupings on 729x776: 60.1 us with it).
template <int N>
__device__ __forceinline__ void load_values(const float* p, int left, float (&v)[N]) {
    if constexpr (N < 4) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = p[i];
    } else if (left >= N) {
        const f4 a = *reinterpret_cast<const f4*>(p);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        if constexpr (N == 6) {
            const f2 b = *reinterpret_cast<const f2*>(p + 4);
            v[4] = b.x; v[5] = b.y;
        }
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = i < left ? p[i] : 0.0f;
    }
}
template <int N>
__device__ __forceinline__ void load_values(const uint8_t* p, int left, float (&v)[N]) {
    if constexpr (N == 1) {
        v[0] = (float)p[0];
    } else if (N == 4 && left >= N) {
        const uint32_t w = *reinterpret_cast<const word_any*>(p);
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = (float)((w >> (8 * i)) & 0xffu);
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = i < left ? (float)p[i] : 0.0f;
    }
}
// LAST: results, which no kernel reads again: four at a time they are stored non-temporal (the three groupings of 1080x1920
// 90.4 us, 93.4 without; uint8 1079x1919 81.2 / 86.6; 1600x2400 137.2 / 136.0).
template <bool LAST, int N>
__device__ __forceinline__ void store_values(float* p, int left, const float (&v)[N]) {
    if constexpr (N == 1) {
        p[0] = v[0];
    } else if (N == 4 && left >= N) {
        const f4 all = f4{v[0], v[1 % N], v[2 % N], v[3 % N]};
        if constexpr (LAST) __builtin_nontemporal_store(all, reinterpret_cast<f4*>(p));
        else *reinterpret_cast<f4*>(p) = all;
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) if (i < left) p[i] = v[i];
    }
}

// First value of this thread in a flat array of `count`, or false.  The last thread of an array or a
// row takes its last four values, some of which its neighbour computes and stores as well (the same
// ones): a path of its own for what is left would cost its wavefront a second memory latency
// (1431x970, the three groupings: 73.8 against 74.5 us).
template <GroupedDealing DEALING, int PX>
__device__ __forceinline__ bool flat(const Blocks<DEALING>& blocks, size_t count, unsigned& image, size_t& at, int& left) {
    unsigned b;
    if (!place<DEALING>(blocks, image, b)) return false;
    at = ((size_t)b * kThreads + threadIdx.x) * PX;
    left = 1;
    if (at >= count) return false;
    if constexpr (PX > 1) {
        at = min(at, max(count, (size_t)PX) - PX);
        left = (int)min(count - at, (size_t)PX);
    }
    return true;
}

// First pixel of this thread in a w x h image, or false.
template <GroupedDealing DEALING, int PX, int ROWS>
__device__ __forceinline__ bool pixel(const Blocks<DEALING>& blocks, int w, int h, unsigned& image, int& x, int& y) {
    unsigned b;
    if (!place<DEALING>(blocks, image, b)) return false;
    const unsigned by = harris_launch::fastdiv(b, blocks.by_across), bx = b - by * blocks.across;
    const unsigned ux = (bx * kTileX + threadIdx.x % kTileX) * PX, uy = (by * kTileY + threadIdx.x / kTileX) * ROWS;
    if (ux >= (unsigned)w || uy >= (unsigned)h) return false;
    x = min((int)ux, max(w - PX, 0));
    y = (int)uy;
    return true;
}

// The input rows of ROWS result rows from (y, x) on, of an h x w result; in is (h+2) x (w+2).  Rows below
// the image repeat its last one (their results are not stored).
template <int PX, int ROWS>
struct Taps {
    float v[ROWS + 2][PX + 2];
    __device__ __forceinline__ void load(const float* in, int w, int h, int y, int x) {
#pragma unroll
        for (int r = 0; r < ROWS + 2; ++r) load_values<PX + 2>(in + (size_t)(ROWS == 1 ? y + r : min(y + r, h + 1)) * (w + 2) + x, w + 2 - x, v[r]);
    }
};
template <bool LAST, int PX, int ROWS>
__device__ __forceinline__ void store_rows(float* out, int w, int h, int y, int x, const float (&v)[ROWS][PX]) {
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
        if (ROWS == 1 || y + r < h) store_values<LAST>(out + (size_t)(y + r) * w + x, w - x, v[r]);
}

// Conversion and grayscale.  rgb[b][3][H][W] -> gray[b][H][W]; in_scale is 1 (float32) or 1/255 (uint8).
template <GroupedDealing DEALING, int PX, typename In>
__global__ void gray_kernel(const Blocks<DEALING> blocks, const In* rgb, float* gray, size_t plane, float in_scale) {
    unsigned nth;
    size_t at;
    int left;
    if (!flat<DEALING, PX>(blocks, plane, nth, at, left)) return;
    const In* p = rgb + (size_t)nth * 3 * plane + at;
    float r[PX], g[PX], b[PX], o[PX];
    load_values(p, left, r);
    load_values(p + plane, left, g);
    load_values(p + 2 * plane, left, b);
#pragma unroll
    for (int i = 0; i < PX; ++i) o[i] = 0.299f * (r[i] * in_scale) + 0.587f * (g[i] * in_scale) + 0.114f * (b[i] * in_scale);
    store_values<false>(gray + (size_t)nth * plane + at, left, o);
}

// The two Sobel responses at row r, column i of a thread's pixels.
template <int PX, int ROWS>
__device__ __forceinline__ void sobel_at(const Taps<PX, ROWS>& t, int r, int i, float s, float& ix, float& iy) {
    const float *r0 = t.v[r] + i, *r1 = t.v[r + 1] + i, *r2 = t.v[r + 2] + i;
    ix = s * ((r0[2] - r0[0]) + 2.0f * (r1[2] - r1[0]) + (r2[2] - r2[0]));
    iy = s * ((r2[0] - r0[0]) + 2.0f * (r2[1] - r0[1]) + (r2[2] - r0[2]));
}

// Sobel stage: one response per launch (Sx or Sy), both, or their three products.  in[b][h+2][w+2] ->
// out_i[b][h][w].
enum Stage { kSx, kSy, kSobelPair, kSobelProducts };
template <GroupedDealing DEALING, int PX, int ROWS, int STAGE>
__global__ void sobel_kernel(const Blocks<DEALING> blocks, const float* in, float* out0, float* out1, float* out2, int h, int w, float s) {
    unsigned nth;
    int x, y;
    if (!pixel<DEALING, PX, ROWS>(blocks, w, h, nth, x, y)) return;
    Taps<PX, ROWS> t;
    t.load(in + (size_t)nth * (h + 2) * (w + 2), w, h, y, x);
    float a[ROWS][PX], b[ROWS][PX], c[ROWS][PX];
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int i = 0; i < PX; ++i) {
            float ix, iy;
            sobel_at(t, r, i, s, ix, iy);
            a[r][i] = STAGE == kSobelProducts ? ix * ix : STAGE == kSy ? iy : ix;
            b[r][i] = STAGE == kSobelProducts ? ix * iy : iy;
            c[r][i] = iy * iy;
        }
    const size_t image = (size_t)nth * h * w;
    store_rows<false>(out0 + image, w, h, y, x, a);
    if constexpr (STAGE >= kSobelPair) store_rows<false>(out1 + image, w, h, y, x, b);
    if constexpr (STAGE == kSobelProducts) store_rows<false>(out2 + image, w, h, y, x, c);
}

// Products, one per launch.
template <int PX>
__global__ void mul_kernel(const Blocks<kRunOfEach> blocks, const float* a, const float* b, float* out, size_t count) {
    unsigned nth;
    size_t at;
    int left;
    if (!flat<kRunOfEach, PX>(blocks, count, nth, at, left)) return;
    float u[PX], v[PX], o[PX];
    load_values(a + at, left, u);
    load_values(b + at, left, v);
#pragma unroll
    for (int i = 0; i < PX; ++i) o[i] = u[i] * v[i];
    store_values<false>(out + at, left, o);
}

// 3x3 window weights: all ones, or [1 2 1; 2 4 2; 1 2 1].
__device__ __forceinline__ float window_weight(int i, int j, int binomial) {
    return binomial ? (float)((2 - (i > 1 ? i - 1 : 1 - i)) * (2 - (j > 1 ? j - 1 : 1 - j))) : 1.0f;
}

// Window sum at row r, column i of a thread's pixels.
template <int PX, int ROWS>
__device__ __forceinline__ float window_at(const Taps<PX, ROWS>& t, int r, int i, int binomial) {
    float acc = 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) acc += window_weight(a, b, binomial) * t.v[r + a][i + b];
    return acc;
}

// Window sums, one per launch.  in[b][h+2][w+2] -> out[b][h][w].
template <GroupedDealing DEALING, int PX, int ROWS>
__global__ void window_kernel(const Blocks<DEALING> blocks, const float* in, float* out, int h, int w, int binomial) {
    unsigned nth;
    int x, y;
    if (!pixel<DEALING, PX, ROWS>(blocks, w, h, nth, x, y)) return;
    Taps<PX, ROWS> t;
    t.load(in + (size_t)nth * (h + 2) * (w + 2), w, h, y, x);
    float o[ROWS][PX];
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int i = 0; i < PX; ++i) o[r][i] = window_at(t, r, i, binomial);
    store_rows<false>(out + (size_t)nth * h * w, w, h, y, x, o);
}

__device__ __forceinline__ float coarsity_of(float sxx, float sxy, float syy, float k) {
    const float det = sxx * syy - sxy * sxy, tr = sxx + syy;
    return det - k * tr * tr;
}

// Coarsity.
template <int PX>
__global__ void coarsity_kernel(const Blocks<kRunOfEach> blocks, const float* sxx, const float* sxy, const float* syy, float* out, size_t count, float k) {
    unsigned nth;
    size_t at;
    int left;
    if (!flat<kRunOfEach, PX>(blocks, count, nth, at, left)) return;
    float a[PX], b[PX], c[PX], o[PX];
    load_values(sxx + at, left, a);
    load_values(sxy + at, left, b);
    load_values(syy + at, left, c);
#pragma unroll
    for (int i = 0; i < PX; ++i) o[i] = coarsity_of(a[i], b[i], c[i], k);
    store_values<true>(out + at, left, o);
}

// Window sums and coarsity from the three product images.
template <GroupedDealing DEALING, int PX, int ROWS>
__global__ void window_coarsity_kernel(const Blocks<DEALING> blocks, const float* ixx, const float* ixy, const float* iyy, float* out, int h, int w, float k, int binomial) {
    unsigned nth;
    int x, y;
    if (!pixel<DEALING, PX, ROWS>(blocks, w, h, nth, x, y)) return;
    const size_t image = (size_t)nth * (h + 2) * (w + 2);
    Taps<PX, ROWS> a, b, c;
    a.load(ixx + image, w, h, y, x);
    b.load(ixy + image, w, h, y, x);
    c.load(iyy + image, w, h, y, x);
    float o[ROWS][PX];
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int i = 0; i < PX; ++i) o[r][i] = coarsity_of(window_at(a, r, i, binomial), window_at(b, r, i, binomial), window_at(c, r, i, binomial), k);
    store_rows<true>(out + (size_t)nth * h * w, w, h, y, x, o);
}

// Products, window sums and coarsity from the two Sobel images.
template <GroupedDealing DEALING, int PX, int ROWS>
__global__ void products_window_coarsity_kernel(const Blocks<DEALING> blocks, const float* ix, const float* iy, float* out, int h, int w, float k, int binomial) {
    unsigned nth;
    int x, y;
    if (!pixel<DEALING, PX, ROWS>(blocks, w, h, nth, x, y)) return;
    const size_t image = (size_t)nth * (h + 2) * (w + 2);
    Taps<PX, ROWS> gx, gy;
    gx.load(ix + image, w, h, y, x);
    gy.load(iy + image, w, h, y, x);
    float o[ROWS][PX];
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int i = 0; i < PX; ++i) {
            float sxx = 0.0f, sxy = 0.0f, syy = 0.0f;
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const float wt = window_weight(p, q, binomial), u = gx.v[r + p][i + q], v = gy.v[r + p][i + q];
                    sxx += wt * u * u;
                    sxy += wt * u * v;
                    syy += wt * v * v;
                }
            o[r][i] = coarsity_of(sxx, sxy, syy, k);
        }
    store_rows<true>(out + (size_t)nth * h * w, w, h, y, x, o);
}

// Every launch of grouping 1, 2 or 3.
template <GroupedDealing DEALING, int PX, int ROWS>
void enqueue(const void* rgb, int dtype, int batch, int H, int W, float k, float s, int binomial, int grouping, float* ws, float* out, hipStream_t st) {
    const int h2 = H - 2, w2 = W - 2, h4 = H - 4, w4 = W - 4;
    const size_t n0 = (size_t)batch * H * W, n2 = (size_t)batch * h2 * w2, n4 = (size_t)batch * h4 * w4, plane = (size_t)H * W;
    const dim3 threads(kThreads);
    auto launch = [](auto dealing, unsigned long long each, unsigned across, int images) {
        constexpr GroupedDealing D = decltype(dealing)::value;
        const harris_launch::GroupedGrid grid = harris_launch::grouped_grid(D == kRunOfImages ? each * images : each);
        Blocks<D> blocks;
        blocks.chunk = grid.chunk; blocks.across = across; blocks.by_across = harris_launch::make_fastdiv(across);
        if constexpr (D == kRunOfImages) { blocks.total = (unsigned)(each * images); blocks.per_image = (unsigned)each; blocks.by_image = harris_launch::make_fastdiv((unsigned)each); }
        struct { Blocks<D> blocks; dim3 grid; } l = {blocks, D == kInOrder ? dim3((unsigned)each, 1, images) : dim3(8 * grid.chunk, grid.turns, D == kRunOfImages ? 1 : images)};
        return l;
    };
    constexpr std::integral_constant<GroupedDealing, DEALING> dealing;
    constexpr std::integral_constant<GroupedDealing, kRunOfEach> whole;             // products and coarsity: one array for all images
    auto area = [&](int w, int h) { const unsigned across = groups_covering(w, kTileX * PX); return launch(dealing, (unsigned long long)across * groups_covering(h, kTileY * ROWS), across, batch); };
    auto line = [&](size_t count) { return (count + kThreads * PX - 1) / (kThreads * PX); };
    const auto gray_l = launch(dealing, line(plane), 1, batch), l2 = area(w2, h2), l4 = area(w4, h4);
    const auto f2 = launch(whole, line(n2), 1, 1), f4 = launch(whole, line(n4), 1, 1);
    float* gray = ws;
    if (dtype == HARRIS_U8) hipLaunchKernelGGL((gray_kernel<DEALING, PX, uint8_t>), gray_l.grid, threads, 0, st, gray_l.blocks, static_cast<const uint8_t*>(rgb), gray, plane, 1.0f / 255.0f);
    else hipLaunchKernelGGL((gray_kernel<DEALING, PX, float>), gray_l.grid, threads, 0, st, gray_l.blocks, static_cast<const float*>(rgb), gray, plane, 1.0f);
    if (grouping == 1) {
        float *ix = gray + n0, *iy = ix + n2, *ixx = iy + n2, *ixy = ixx + n2, *iyy = ixy + n2, *sxx = iyy + n2, *sxy = sxx + n4, *syy = sxy + n4;
        hipLaunchKernelGGL((sobel_kernel<DEALING, PX, ROWS, kSx>), l2.grid, threads, 0, st, l2.blocks, gray, ix, nullptr, nullptr, h2, w2, s);
        hipLaunchKernelGGL((sobel_kernel<DEALING, PX, ROWS, kSy>), l2.grid, threads, 0, st, l2.blocks, gray, iy, nullptr, nullptr, h2, w2, s);
        hipLaunchKernelGGL(mul_kernel<PX>, f2.grid, threads, 0, st, f2.blocks, ix, ix, ixx, n2);
        hipLaunchKernelGGL(mul_kernel<PX>, f2.grid, threads, 0, st, f2.blocks, ix, iy, ixy, n2);
        hipLaunchKernelGGL(mul_kernel<PX>, f2.grid, threads, 0, st, f2.blocks, iy, iy, iyy, n2);
        hipLaunchKernelGGL((window_kernel<DEALING, PX, ROWS>), l4.grid, threads, 0, st, l4.blocks, ixx, sxx, h4, w4, binomial);
        hipLaunchKernelGGL((window_kernel<DEALING, PX, ROWS>), l4.grid, threads, 0, st, l4.blocks, ixy, sxy, h4, w4, binomial);
        hipLaunchKernelGGL((window_kernel<DEALING, PX, ROWS>), l4.grid, threads, 0, st, l4.blocks, iyy, syy, h4, w4, binomial);
        hipLaunchKernelGGL(coarsity_kernel<PX>, f4.grid, threads, 0, st, f4.blocks, sxx, sxy, syy, out, n4, k);
    } else if (grouping == 2) {
        float *ixx = gray + n0, *ixy = ixx + n2, *iyy = ixy + n2;
        hipLaunchKernelGGL((sobel_kernel<DEALING, PX, ROWS, kSobelProducts>), l2.grid, threads, 0, st, l2.blocks, gray, ixx, ixy, iyy, h2, w2, s);
        hipLaunchKernelGGL((window_coarsity_kernel<DEALING, PX, ROWS>), l4.grid, threads, 0, st, l4.blocks, ixx, ixy, iyy, out, h4, w4, k, binomial);
    } else {
        float *ix = gray + n0, *iy = ix + n2;
        hipLaunchKernelGGL((sobel_kernel<DEALING, PX, ROWS, kSobelPair>), l2.grid, threads, 0, st, l2.blocks, gray, ix, iy, nullptr, h2, w2, s);
        hipLaunchKernelGGL((products_window_coarsity_kernel<DEALING, PX, ROWS>), l4.grid, threads, 0, st, l4.blocks, ix, iy, out, h4, w4, k, binomial);
    }
}

}  // namespace

namespace harris_launch {

size_t grouped_workspace_floats(int grouping, int batch, int H, int W) {
    const size_t n0 = (size_t)H * W, n2 = (size_t)(H - 2) * (W - 2), n4 = (size_t)(H - 4) * (W - 4);
    switch (grouping) {
        case 1: return (size_t)batch * (n0 + 5 * n2 + 3 * n4);   // gray, Ix, Iy, Ixx, Ixy, Iyy, Sxx, Sxy, Syy
        case 2: return (size_t)batch * (n0 + 3 * n2);            // gray, Ixx, Ixy, Iyy
        case 3: return (size_t)batch * (n0 + 2 * n2);            // gray, Ix, Iy
        default: return 0;
    }
}

int launch_grouped(const void* rgb, int dtype, int batch, int H, int W, float k, float sobel_scale, int binomial,
                   int grouping, float* ws, float* out, void* stream_) {
    hipStream_t st = static_cast<hipStream_t>(stream_);
    if (batch > 65535) return HARRIS_ERR_SHAPE;        // images ride on gridDim.z
    const bool wide = grouped_wide(batch, H, W);
    const auto run = [&](auto dealing) {
        constexpr GroupedDealing D = decltype(dealing)::value;
        if (wide) enqueue<D, 4, 2>(rgb, dtype, batch, H, W, k, sobel_scale, binomial, grouping, ws, out, st);
        else enqueue<D, 1, 1>(rgb, dtype, batch, H, W, k, sobel_scale, binomial, grouping, ws, out, st);
    };
    switch (grouped_dealing(batch, H, W, wide)) {
        case kRunOfEach: run(std::integral_constant<GroupedDealing, kRunOfEach>()); break;
        case kRunOfImages: run(std::integral_constant<GroupedDealing, kRunOfImages>()); break;
        case kInOrder: run(std::integral_constant<GroupedDealing, kInOrder>()); break;
    }
    return hipGetLastError() == hipSuccess ? HARRIS_OK : HARRIS_ERR_LAUNCH;
}

// Device address of `scratch` on the current device, looked up once per device (with that
// device current, as now) and kept.  NULL if the runtime cannot say.
float* scratch_of_current_device() {
    constexpr int kMaxDevices = 64;
    static std::mutex lock;
    static float* known[kMaxDevices] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> hold(lock);
    if (known[dev] == nullptr) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        known[dev] = static_cast<float*>(ptr);
    }
    return known[dev];
}

}  // namespace harris_launch
