// Aggregation regions and the gather (normalisation) of Algorithm 1, and the tiling of the
// reference grid for the filter kernel (filter_mfma.hip).
//
// The filter processes the references of a T x T tile in one workgroup and adds every
// reconstructed patch into an LDS copy of the image region those references' groups can reach
// (their search windows plus the patch extent).  The region is written, without atomics, to the
// tile's own slot of a global buffer as C + 1 planes: the channel sums and the number of patches
// covering each pixel.  The gather kernel then sums, for every pixel, the (at most a few)
// regions covering it and divides (uniform weights, "average" aggregation); a pixel no patch
// covers keeps its noisy value.
#include <algorithm>

#include "common.h"

namespace htsvd {
namespace {

// out = (sum of the regions covering the pixel) / (their count); noisy value where no patch landed.
template <int C>
__device__ __forceinline__ void gather_px(const ImageGeom &g, const TileGeom &tg, const float *__restrict__ regions,
                                          float *__restrict__ out, int64_t out_stride, int64_t e) {
    constexpr int CH = C + 1;
    const int y = (int)(e / g.w), x = (int)(e % g.w);
    const int span_y = tg.TY * g.s, span_x = tg.TX * g.s;
    const int ty_lo = max(0, (y - tg.R - PS - span_y) / span_y - 1);
    const int ty_hi = min(tg.tiles_y - 1, (y + tg.R) / span_y + 1);
    const int tx_lo = max(0, (x - tg.R - PS - span_x) / span_x - 1);
    const int tx_hi = min(tg.tiles_x - 1, (x + tg.R) / span_x + 1);
    float acc[CH];
#pragma unroll
    for (int k = 0; k < CH; ++k) acc[k] = 0.f;
    const int plane = region_plane(tg), elems = region_elems(tg, C);
    for (int ty = ty_lo; ty <= ty_hi; ++ty) {
        int r0, r1;
        region_rows(g, tg, ty, &r0, &r1);
        if (y < r0 || y > r1) continue;
        for (int tx = tx_lo; tx <= tx_hi; ++tx) {
            int c0, c1;
            region_cols(g, tg, tx, &c0, &c1);
            if (x < c0 || x > c1) continue;
            const float *src = regions + (int64_t)(ty * tg.tiles_x + tx) * elems;
            const int e0 = (y - r0) * tg.RP + (x - c0);
#pragma unroll
            for (int k = 0; k < C; ++k) acc[k] += src[e0 * C + k];
            acc[C] += src[C * plane + e0];
        }
    }
    float *o = out + (int64_t)y * out_stride + (int64_t)x * C;
    const uint8_t *px = g.img + (int64_t)y * g.stride + (int64_t)x * C;
#pragma unroll
    for (int ch = 0; ch < C; ++ch) o[ch] = acc[C] > 0.f ? acc[ch] / acc[C] : (float)px[ch];
}

template <int C>
__global__ void gather_kernel(ImageGeom g, TileGeom tg, const float *__restrict__ regions, float *__restrict__ out,
                              int64_t out_stride) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)g.h * g.w) return;
    gather_px<C>(g, tg, regions, out, out_stride, e);
}

// All pixels of all images of a batch; pix_start holds the prefix sums of the pixel counts.
template <int C>
__global__ void gather_kernel_batched(const BatchItem *__restrict__ items, int n_items,
                                      const int *__restrict__ pix_start) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= pix_start[n_items]) return;
    const int i = find_unit(pix_start, n_items, e);
    const BatchItem &it = items[i];
    const bool alt = it.ksel && *it.ksel == it.k_alt;
    gather_px<C>(it.g, alt ? it.tg_alt : it.tg, it.regions, it.out, it.out_stride, e - pix_start[i]);
}

// Tiling with T x T references per tile (tight: no padding of the region's rows).
TileGeom tiles_of(const ImageGeom &g, int W, int T, bool tight) {
    TileGeom tg;
    tg.FS = 0;
    tg.R = (W - 1) / 2;
    tg.TY = tg.TX = T;
    tg.RH = min((T - 1) * g.s + 2 * tg.R + PS, g.h);
    tg.RW = min((T - 1) * g.s + 2 * tg.R + PS, g.w);
    tg.RP = tight ? tg.RW : region_pitch(tg.RW);
    tg.tiles_y = (g.ny + T - 1) / T;
    tg.tiles_x = (g.nx + T - 1) / T;
    return tg;
}

size_t region_bytes(const TileGeom &tg, int c) {
    return (size_t)tg.tiles_y * tg.tiles_x * region_elems(tg, c) * sizeof(float);
}

}  // namespace

int filter_lds_budget() { return 160 * 1024 - filter_mfma_static_bytes() - 64; }

bool padded_region_fits(int planes, int rows, int cols) {
    return (int64_t)planes * rows * (cols + (24 - cols % 16) % 16) * 4 + 65 * 1024 <= filter_lds_budget();
}

// Fixed-point shift of the region sums: a pixel of a tile's region receives at most T^2 K
// contributions (every member of every group of the tile), each clamped to |v| <= 1024, so
// T^2 K 1024 2^FS must stay below 2^31.  Tiles are capped so that FS >= 9: a contribution
// is rounded by at most 2^-10, and so is the average of a pixel's contributions.  FS <= 12
// keeps every scaled contribution below 2^22, the range of the filter's rounding by
// addition of 1.5 * 2^23.
constexpr double FX_CLAMP = 1024.0;
constexpr int FX_MIN_SHIFT = 9;
constexpr int FX_MAX_SHIFT = 12;

int accumulation_shift(int T, int K) {
    const double worst = (double)T * T * K * FX_CLAMP;
    int fs = 0;
    while (fs < FX_MAX_SHIFT && worst * (double)(1 << (fs + 1)) < 2147483647.0) ++fs;
    return fs;
}

// Estimated microseconds of the filter over n_tiles tiles of refs references (K members each), on `share` of
// the GPU's 256 CUs (asked of no device: a plan is the same wherever it is made, and a partition with fewer
// CUs only gets tiles that suit the whole GPU): one workgroup of 8 waves per CU takes whole tiles, a wave takes
// 32 patches per step, and a tile costs a fixed time besides (clearing and writing its region, the first loads
// of its patches, waves that wait for the last one).  Whole steps that every wave takes are counted, not the
// last one of some.  The constants come from two shapes, with the tile side forced: 512 x 512 RGB, stride 4,
// window 31, K 32: 187, 188, 164, 146, 203 us at side 4, 5, 6, 8, 10, rounds (steps 14.5 + 18) = 188, 185, 152,
// 134, 192; 1536 x 2048 gray, K 16: 538, 412, 332, 320 us at side 4, 6, 8, 11, rounds (steps 4.6 + 9).
double filter_tiles_cost(int c, int K, int64_t n_tiles, int refs, double share) {
    const int64_t cu = std::max<int64_t>(1, (int64_t)(256 * share + 0.5));
    const int64_t steps = std::max(1, refs * K / (32 * 8));
    return (double)((n_tiles + cu - 1) / cu) * (c == 3 ? 14.5 * steps + 18.0 : 4.6 * steps + 9.0);
}

// Shift that a tiling's sums keep at least: that of the largest tile whose region, rows padded to 8 modulo
// 16 words, fits in LDS beside 65 KB.  The choice by time alone takes larger tiles where the LDS allows,
// with sums in coarser units (RGB, K 8, window 21, step 3: side 16 and 2^-9 instead of 15 and 2^-10).
int least_shift(const ImageGeom &g, int W, int K, int max_side) {
    int T = max_side > 0 ? min(max_side, 16) : 16;
    for (; T > 1; --T) {
        const int reach = (T - 1) * g.s + (W - 1) + PS;
        if (accumulation_shift(T, K) >= FX_MIN_SHIFT && padded_region_fits(g.c + 1, min(reach, g.h), min(reach, g.w)))
            break;
    }
    return accumulation_shift(T, K);
}

// The tile side with the lowest estimated time among those whose region fits in LDS beside the
// tables and whose sums keep least_shift: small images take small tiles, so that every CU has
// one, large ones the largest, whose regions overlap least.  The regions' way through memory
// (written and read once, about 2.5 bytes per nanosecond and direction over the whole GPU at
// these sizes) is added.  64 x 72 RGB at K 16: 108 us at the largest side (one tile), 29 at side 4;
// 256 x 256 gray: 49 against 20.  For the fixed scratch of the no-allocation call, SMALL: the side whose
// regions, without padding, take the least memory instead; SMALLEST: the same with the shifts down to
// FX_MIN_SHIFT.
TileGeom plan_filter_tiles(const ImageGeom &g, int W, int K, int max_side, double share, FilterTiles pick) {
    const bool compact = pick != FilterTiles::FASTEST;
    const int least = pick == FilterTiles::SMALLEST ? FX_MIN_SHIFT : least_shift(g, W, K, max_side);
    TileGeom best = tiles_of(g, W, 1, compact);
    double best_cost = 0.0;
    const int top = min(max_side > 0 ? min(max_side, 16) : 16, max(g.ny, g.nx));
    for (int T = 1; T <= top; ++T) {
        const TileGeom tg = tiles_of(g, W, T, compact);
        if (T > 1 && (accumulation_shift(T, K) < least || filter_mfma_lds_bytes(tg, g.c) > filter_lds_budget()))
            break;
        const double bytes = (double)region_bytes(tg, g.c);
        const double cost = compact ? bytes
                                    : filter_tiles_cost(g.c, K, (int64_t)tg.tiles_y * tg.tiles_x, T * T, share) +
                                          bytes / 2.5e6;
        if (T == 1 || cost <= best_cost) {
            best = tg;
            best_cost = cost;
        }
    }
    best.FS = accumulation_shift(best.TY, K);
    return best;
}

size_t filter_region_bytes(const TileGeom &tg, int c) { return region_bytes(tg, c); }

hipError_t launch_gather_batched(int C, const BatchItem *items, int n_items, const int *pix_start, int total_px,
                                 hipStream_t st) {
    const unsigned grid = (unsigned)((total_px + 255) / 256);
    if (C == 3)
        hipLaunchKernelGGL(gather_kernel_batched<3>, dim3(grid), dim3(256), 0, st, items, n_items, pix_start);
    else
        hipLaunchKernelGGL(gather_kernel_batched<1>, dim3(grid), dim3(256), 0, st, items, n_items, pix_start);
    return hipGetLastError();
}

hipError_t launch_gather(const ImageGeom &g, const TileGeom &tg, const float *regions, float *out, int64_t out_stride,
                         hipStream_t st) {
    const int64_t n = (int64_t)g.h * g.w;
    if (g.c == 3)
        hipLaunchKernelGGL(gather_kernel<3>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, g, tg, regions, out,
                           out_stride);
    else
        hipLaunchKernelGGL(gather_kernel<1>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, g, tg, regions, out,
                           out_stride);
    return hipGetLastError();
}

}  // namespace htsvd
