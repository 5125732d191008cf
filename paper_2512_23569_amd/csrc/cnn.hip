// Learned noise-level network: a 6-layer 3x3 convolutional net that predicts log(sigma)
// for every 8x8 block (the paper's estimator is a CNN, Sec. III-E-1 and Fig. 5; its data
// and weights are not available, so this network is trained here on synthetic crops).
//
//   x0 = (u8 - 128) / 64 (NHWC, C = 1 or 3)
//   L1 3x3 C->32 stride 2 ReLU | L2 32->32 s2 ReLU | L3 32->32 s2 ReLU
//   L4 32->32 s1 ReLU | L5 32->32 s1 ReLU | L6 32->1 s1 (linear) -> z = log(sigma)
//   loss = mean |z - log(sigma_target)|
//
// Storage: activations NHWC bf16 (round to nearest even), weights bf16 for the forward pass
// with FP32 master copies, FP32 accumulation everywhere.  Parameters are one flat array in
// layer order, each layer w[co][ky][kx][ci] then b[co].
//
// Kernels: the 32->32 convolutions are implicit GEMMs on v_mfma_f32_16x16x32_bf16 (16 output
// pixels x 16 output channels per instruction, k = the 32 input channels of one tap, 9 taps);
// layer 1 (3 input channels) and layer 6 (1 output channel) run on the vector ALUs.  The
// backward pass stays in FP32: weight gradients and the input gradients of the 32-channel layers
// are contractions on v_mfma_f32_32x32x2_f32 (FP32 operands, products and sums).
#include <math.h>

#include <algorithm>

#include "common.h"

namespace htsvd {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

namespace {

__device__ __host__ inline uint16_t f2bf(float f) {
    uint32_t u;
    __builtin_memcpy(&u, &f, 4);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __host__ inline float bf2f(uint16_t h) {
    uint32_t u = (uint32_t)h << 16;
    float f;
    __builtin_memcpy(&f, &u, 4);
    return f;
}

struct ConvShape {
    int N, H, W, Ci;    // input
    int Ho, Wo, Co;     // output
    int s;              // stride
};

// ---- layer 1: u8 image -> 32 channels, vector ALU ----
// One thread per output pixel; the 9 C input taps stay in registers, the weights are uniform
// across the wavefront (scalar loads), the 32 outputs leave as four 16-byte stores.  Image n
// starts at img + n img_batch_stride with row stride img_stride, or, with a table, at
// img_tab[n] with row stride stride_tab[n] (images of one size in separate buffers).
template <int C>
__global__ __launch_bounds__(256) void l1_fwd_kernel(const uint8_t *__restrict__ img, int64_t img_stride,
                                                     int64_t img_batch_stride,
                                                     const uint8_t *const *__restrict__ img_tab,
                                                     const int64_t *__restrict__ stride_tab, ConvShape cs,
                                                     const float *__restrict__ wq, const float *__restrict__ bias,
                                                     uint16_t *__restrict__ out) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t total = (int64_t)cs.N * cs.Ho * cs.Wo;
    if (p >= total) return;
    const int n = (int)(p / ((int64_t)cs.Ho * cs.Wo));
    const int rem = (int)(p % ((int64_t)cs.Ho * cs.Wo));
    const int yo = rem / cs.Wo, xo = rem % cs.Wo;
    const uint8_t *ibase = img_tab ? img_tab[n] : img + n * img_batch_stride;
    const int64_t rs = img_tab ? stride_tab[n] : img_stride;
    float x[9 * C];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const int yi = cs.s * yo + t / 3 - 1, xi = cs.s * xo + t % 3 - 1;
        const bool ok = yi >= 0 && yi < cs.H && xi >= 0 && xi < cs.W;
#pragma unroll
        for (int ci = 0; ci < C; ++ci) x[t * C + ci] = 0.f;
        if (ok) {
            const uint8_t *src = ibase + (int64_t)yi * rs + (int64_t)xi * C;
#pragma unroll
            for (int ci = 0; ci < C; ++ci) x[t * C + ci] = ((float)src[ci] - 128.f) * 0.015625f;
        }
    }
    uint32_t packed[16];
#pragma unroll
    for (int co = 0; co < 32; ++co) {
        float acc = bias[co];
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int ci = 0; ci < C; ++ci) acc += wq[(co * 9 + t) * C + ci] * x[t * C + ci];
        const uint32_t h = f2bf(acc > 0.f ? acc : 0.f);
        packed[co >> 1] = (co & 1) ? (packed[co >> 1] | (h << 16)) : h;
    }
    uint4 *o = reinterpret_cast<uint4 *>(out + p * 32);
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = make_uint4(packed[4 * q], packed[4 * q + 1], packed[4 * q + 2], packed[4 * q + 3]);
}

// ---- 32 -> 32 convolution on the matrix cores ----
// One wavefront computes 16 output pixels x 32 output channels per tile; weights live in
// registers (9 taps x 2 channel tiles of 8 bf16 per lane).
__global__ __launch_bounds__(256) void conv32_fwd_kernel(const uint16_t *__restrict__ in, ConvShape cs,
                                                         const uint16_t *__restrict__ wbf,
                                                         const float *__restrict__ bias,
                                                         uint16_t *__restrict__ out, int relu) {
    const int lane = threadIdx.x & 63;
    const int wave_global = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int n_waves = (gridDim.x * blockDim.x) >> 6;
    const int i16 = lane & 15, kq = lane >> 4;
    v8bf bw[9][2];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            const uint4 raw = *reinterpret_cast<const uint4 *>(wbf + ((16 * nt + i16) * 9 + t) * 32 + 8 * kq);
            bw[t][nt] = __builtin_bit_cast(v8bf, raw);
        }
    const float b0 = bias[i16], b1 = bias[16 + i16];
    const int64_t total = (int64_t)cs.N * cs.Ho * cs.Wo;
    const int64_t n_tiles = (total + 15) / 16;
    for (int64_t tile = wave_global; tile < n_tiles; tile += n_waves) {
        const int64_t p = tile * 16 + i16;
        const bool pv = p < total;
        const int64_t pp = pv ? p : 0;
        const int n = (int)(pp / ((int64_t)cs.Ho * cs.Wo));
        const int rem = (int)(pp % ((int64_t)cs.Ho * cs.Wo));
        const int yo = rem / cs.Wo, xo = rem % cs.Wo;
        v4f acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const int yi = cs.s * yo + t / 3 - 1, xi = cs.s * xo + t % 3 - 1;
            uint4 raw = {0u, 0u, 0u, 0u};
            if (pv && yi >= 0 && yi < cs.H && xi >= 0 && xi < cs.W)
                raw = *reinterpret_cast<const uint4 *>(in + (((int64_t)n * cs.H + yi) * cs.W + xi) * 32 + 8 * kq);
            const v8bf a = __builtin_bit_cast(v8bf, raw);
            acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bw[t][0], acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bw[t][1], acc1, 0, 0, 0);
        }
        // lane holds pixels 4*kq + r of the tile, channel i16 (and 16 + i16)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t q = tile * 16 + 4 * kq + r;
            if (q < total) {
                float v0 = acc0[r] + b0, v1 = acc1[r] + b1;
                if (relu) { v0 = v0 > 0.f ? v0 : 0.f; v1 = v1 > 0.f ? v1 : 0.f; }
                out[q * 32 + i16] = f2bf(v0);
                out[q * 32 + 16 + i16] = f2bf(v1);
            }
        }
    }
}

// ---- layer 6: 32 -> 1, vector ALU, FP32 output ----
__global__ void l6_fwd_kernel(const uint16_t *__restrict__ in, ConvShape cs, const float *__restrict__ wq,
                              const float *__restrict__ bias, float *__restrict__ z) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t total = (int64_t)cs.N * cs.Ho * cs.Wo;
    if (p >= total) return;
    const int n = (int)(p / ((int64_t)cs.Ho * cs.Wo));
    const int rem = (int)(p % ((int64_t)cs.Ho * cs.Wo));
    const int yo = rem / cs.Wo, xo = rem % cs.Wo;
    float acc = bias[0];
    for (int t = 0; t < 9; ++t) {
        const int yi = yo + t / 3 - 1, xi = xo + t % 3 - 1;
        if (yi < 0 || yi >= cs.H || xi < 0 || xi >= cs.W) continue;
        const uint16_t *a = in + (((int64_t)n * cs.H + yi) * cs.W + xi) * 32;
        for (int ci = 0; ci < 32; ++ci) acc += wq[t * 32 + ci] * bf2f(a[ci]);
    }
    z[p] = acc;
}

// ---- loss: mean |z - t|, dz = sign(z - t) / count ----
__global__ void l1loss_kernel(const float *__restrict__ z, const float *__restrict__ t, int64_t count,
                              float *__restrict__ dz, double *__restrict__ loss_sum) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double v = 0.0;
    if (i < count) {
        const float d = z[i] - t[i];
        dz[i] = (d > 0.f ? 1.f : (d < 0.f ? -1.f : 0.f)) / (float)count;
        v = fabs((double)d);
    }
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((threadIdx.x & 63) == 0) atomicAdd(loss_sum, v);
}

// Steps (yo, xo) of image n by d output pixels.
__device__ inline void advance(int &n, int &yo, int &xo, int d, const ConvShape &cs) {
    xo += d;
    while (xo >= cs.Wo) {
        xo -= cs.Wo;
        if (++yo == cs.Ho) {
            yo = 0;
            ++n;
        }
    }
}

// dW[co][tap][ci] += sum_p dY[p][co] * X[in(p, tap)][ci];  db[co] += sum_p dY[p][co].
//
// A contraction over the output pixels p: M = co (32, rows past Co are zero), N = 32 columns, two
// pixels per v_mfma_f32_32x32x2_f32 (lane = row or column, lane half = pixel).  NACC = 9: input of
// 32 bf16 channels, one accumulator per tap, columns ci; NACC = 1: the u8 image, columns tap * Ci + ci
// (9 Ci <= 27).  A wave takes `chunk` consecutive pixels, with the operands of the next four pairs
// loaded ahead of the products of these; the four waves of a workgroup add up in LDS and the sums go
// to global memory by float atomics.  Against one thread per (tap, ci) walking 256 pixels with a
// division, two loads and a multiply-add each, 32 crops of 128 x 128: all layers 1,641 -> 209 us.
constexpr int WG_WAVES = 4;
constexpr int WG_AHEAD = 4;   // pixel pairs loaded together, one group ahead
template <int NACC>
__global__ __launch_bounds__(64 * WG_WAVES) void wgrad_mfma_kernel(const uint16_t *__restrict__ act,
                                                                   const uint8_t *__restrict__ img,
                                                                   int64_t img_stride, int64_t img_batch_stride,
                                                                   ConvShape cs, const float *__restrict__ dy,
                                                                   int chunk, float *__restrict__ dw,
                                                                   float *__restrict__ db) {
    extern __shared__ __align__(16) float wsum[];   // [wave][NACC * 1024]
    __shared__ float bsum[WG_WAVES][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 31, h = lane >> 5;
    const int64_t total = (int64_t)cs.N * cs.Ho * cs.Wo;
    const int64_t p0 = ((int64_t)blockIdx.x * WG_WAVES + wave) * chunk, p1 = min(total, p0 + chunk);
    v16f acc[NACC];
#pragma unroll
    for (int t = 0; t < NACC; ++t) acc[t] = (v16f){};
    float bias = 0.f;
    const int tap1 = col / cs.Ci, ci1 = col - tap1 * cs.Ci;   // column of the image form
    int n = 0, yo = 0, xo = 0;
    if (p0 < total) {
        const int64_t hw = (int64_t)cs.Ho * cs.Wo;
        n = (int)(p0 / hw);
        const int rem = (int)(p0 - n * hw);
        yo = rem / cs.Wo;
        xo = rem - yo * cs.Wo;
    }
    // operands of pixel p + h: dy of row `col`, and the input value of every accumulator's column
    auto load = [&](int64_t p, float &g, float (&x)[NACC]) {
        int nn = n, y = yo, xx = xo;
        if (h) advance(nn, y, xx, 1, cs);
        const bool valid = p + h < p1;
        const float gv = dy[valid && col < cs.Co ? (p + h) * cs.Co + col : 0];
        g = valid && col < cs.Co ? gv : 0.f;
        const int yb = cs.s * y - 1, xb = cs.s * xx - 1;
#pragma unroll
        for (int t = 0; t < NACC; ++t) {
            const int tap = NACC == 9 ? t : tap1;
            const int yi = yb + tap / 3, xi = xb + tap % 3;
            const bool ok = valid && yi >= 0 && yi < cs.H && xi >= 0 && xi < cs.W && tap < 9;
            if constexpr (NACC == 9) {
                const uint16_t v = act[ok ? (((int64_t)nn * cs.H + yi) * cs.W + xi) * 32 + col : 0];
                x[t] = ok ? bf2f(v) : 0.f;
            } else {
                const uint8_t v = img[ok ? nn * img_batch_stride + (int64_t)yi * img_stride + (int64_t)xi * cs.Ci + ci1 : 0];
                x[t] = ok ? ((float)v - 128.f) * 0.015625f : 0.f;
            }
        }
    };
    if (p0 < p1) {
        float g[WG_AHEAD], x[WG_AHEAD][NACC];
        auto load_group = [&](int64_t p, float (&gg)[WG_AHEAD], float (&xx)[WG_AHEAD][NACC]) {
#pragma unroll
            for (int u = 0; u < WG_AHEAD; ++u) {
                load(p + 2 * u, gg[u], xx[u]);
                advance(n, yo, xo, 2, cs);
            }
        };
        load_group(p0, g, x);
        for (int64_t p = p0; p < p1; p += 2 * WG_AHEAD) {
            float gn[WG_AHEAD], xn[WG_AHEAD][NACC];
            load_group(p + 2 * WG_AHEAD, gn, xn);   // past the end: zeros, from index 0
#pragma unroll
            for (int u = 0; u < WG_AHEAD; ++u) {
                bias += g[u];
#pragma unroll
                for (int t = 0; t < NACC; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(g[u], x[u][t], acc[t], 0, 0, 0);
            }
#pragma unroll
            for (int u = 0; u < WG_AHEAD; ++u) {
                g[u] = gn[u];
#pragma unroll
                for (int t = 0; t < NACC; ++t) x[u][t] = xn[u][t];
            }
        }
    }
    float *mine = wsum + wave * NACC * 1024;
#pragma unroll
    for (int t = 0; t < NACC; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) mine[t * 1024 + (8 * (r >> 2) + 4 * h + (r & 3)) * 32 + col] = acc[t][r];
    bsum[wave][lane] = bias;
    __syncthreads();
    for (int e = threadIdx.x; e < NACC * 1024; e += 64 * WG_WAVES) {
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < WG_WAVES; ++w) v += wsum[w * NACC * 1024 + e];
        const int t = e >> 10, co = (e >> 5) & 31, c = e & 31;
        if (co >= cs.Co) continue;
        if constexpr (NACC == 9)
            atomicAdd(dw + (co * 9 + t) * 32 + c, v);
        else if (c < 9 * cs.Ci)
            atomicAdd(dw + co * 9 * cs.Ci + c, v);
    }
    if (threadIdx.x < cs.Co) {
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < WG_WAVES; ++w) v += bsum[w][threadIdx.x] + bsum[w][threadIdx.x + 32];
        atomicAdd(db + threadIdx.x, v);
    }
}

// dX[q][ci] = sum_{tap, co} dY[out(q, tap)][co] * W[co][tap][ci], times (act[q][ci] > 0): the ReLU
// backward of the layer below, whose output act is (post-ReLU bf16).
//
// 32 -> 32 channels: a contraction over (tap, co) with M = 32 input pixels, N = ci.  At stride 2 a
// pixel meets only the taps of its row and column parity (1, 2, 2 or 4 of the 9), so a tile holds
// pixels of one parity class.  A lane reads 16 consecutive co of its pixel's dY per tap (lane half
// h: co 16 h ..), and the weights lie in LDS in the order of the products.  FP32 throughout.
// Against one thread per (q, ci) over all taps and channels, 32 crops of 128 x 128: all layers with
// the masks 481 -> 104 us.
constexpr int DG_WAVES = 4;
__global__ __launch_bounds__(64 * DG_WAVES) void dgrad32_kernel(const float *__restrict__ dy, ConvShape cs,
                                                                const float *__restrict__ wq,
                                                                const uint16_t *__restrict__ act,
                                                                float *__restrict__ dx) {
    __shared__ __align__(16) float wl[9 * 4 * 64 * 4];   // [tap][co quad of the half][lane][4]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane & 31, h = lane >> 5;
    for (int e = threadIdx.x; e < 9 * 4 * 64 * 4; e += 64 * DG_WAVES) {
        const int j = e & 3, l = (e >> 2) & 63, k4 = (e >> 8) & 3, tap = e >> 10;
        wl[e] = wq[((16 * (l >> 5) + 4 * k4 + j) * 9 + tap) * 32 + (l & 31)];
    }
    __syncthreads();
    const int ncls = cs.s == 2 ? 4 : 1;
    int64_t first = 0;   // tiles before this class
    for (int cls = 0; cls < ncls; ++cls) {
        const int py = cls >> 1, px = cls & 1;
        const int Hc = cs.s == 2 ? (cs.H - py + 1) / 2 : cs.H, Wc = cs.s == 2 ? (cs.W - px + 1) / 2 : cs.W;
        const int64_t count = (int64_t)cs.N * Hc * Wc, tiles = (count + 31) / 32;
        const int64_t step = (int64_t)gridDim.x * DG_WAVES, me = (int64_t)blockIdx.x * DG_WAVES + wave;
        // tiles of all classes are dealt to the waves in turn
        int64_t tile = (me - first % step + step) % step;
        first += tiles;
        for (; tile < tiles; tile += step) {
            const int64_t q = tile * 32 + m;
            const bool qv = q < count;
            int n = 0, yi = 0, xi = 0;
            if (qv) {
                n = (int)(q / ((int64_t)Hc * Wc));
                const int rem = (int)(q - n * ((int64_t)Hc * Wc));
                yi = rem / Wc;
                xi = rem - yi * Wc;
                if (cs.s == 2) {
                    yi = 2 * yi + py;
                    xi = 2 * xi + px;
                }
            }
            v16f acc = {};
#pragma unroll
            for (int tap = 0; tap < 9; ++tap) {
                const int ky = tap / 3, kx = tap % 3;
                if (cs.s == 2 && (((py + 1 - ky) & 1) || ((px + 1 - kx) & 1))) continue;   // uniform
                const int ny = yi + 1 - ky, nx = xi + 1 - kx;     // = s * (yo, xo)
                const int yo = cs.s == 2 ? ny >> 1 : ny, xo = cs.s == 2 ? nx >> 1 : nx;
                const bool ok = qv && ny >= 0 && nx >= 0 && yo < cs.Ho && xo < cs.Wo;
                const float4 *src = reinterpret_cast<const float4 *>(
                    dy + (ok ? (((int64_t)n * cs.Ho + yo) * cs.Wo + xo) * 32 : 0) + 16 * h);
#pragma unroll
                for (int k4 = 0; k4 < 4; ++k4) {
                    float4 g = src[k4];
                    if (!ok) g = make_float4(0.f, 0.f, 0.f, 0.f);
                    const float4 w4 = *reinterpret_cast<const float4 *>(wl + ((tap * 4 + k4) * 64 + lane) * 4);
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(g.x, w4.x, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(g.y, w4.y, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(g.z, w4.z, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(g.w, w4.w, acc, 0, 0, 0);
                }
            }
            // lane holds channel m of pixels 8(r/4) + 4h + r%4 of the tile, whose indices those lanes have
            const int lin = (n * cs.H + yi) * cs.W + xi;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int pm = 8 * (r >> 2) + 4 * h + (r & 3);
                const int64_t e = (int64_t)__shfl(lin, pm) * 32 + m;
                if (tile * 32 + pm < count) dx[e] = bf2f(act[e]) > 0.f ? acc[r] : 0.f;
            }
        }
    }
}

// The same for one output channel (layer 6); one thread per (q, ci).
__global__ void dgrad_kernel(const float *__restrict__ dy, ConvShape cs, const float *__restrict__ wq,
                             const uint16_t *__restrict__ act, float *__restrict__ dx) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t total = (int64_t)cs.N * cs.H * cs.W * cs.Ci;
    if (e >= total) return;
    const int ci = (int)(e % cs.Ci);
    const int64_t q = e / cs.Ci;
    const int n = (int)(q / ((int64_t)cs.H * cs.W));
    const int rem = (int)(q % ((int64_t)cs.H * cs.W));
    const int yi = rem / cs.W, xi = rem % cs.W;
    float acc = 0.f;
    for (int t = 0; t < 9; ++t) {
        const int yo = yi + 1 - t / 3, xo = xi + 1 - t % 3;   // stride 1
        if (yo < 0 || xo < 0 || yo >= cs.Ho || xo >= cs.Wo) continue;
        acc += dy[((int64_t)n * cs.Ho + yo) * cs.Wo + xo] * wq[t * cs.Ci + ci];
    }
    dx[e] = bf2f(act[e]) > 0.f ? acc : 0.f;
}

__global__ void adam_kernel(float *__restrict__ w, float *__restrict__ m, float *__restrict__ v,
                            const float *__restrict__ g, int n, float lr, float b1, float b2, float eps, float c1,
                            float c2, float *__restrict__ wq, uint16_t *__restrict__ wbf) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    w[i] = wi;
    const uint16_t hb = f2bf(wi);
    wbf[i] = hb;
    wq[i] = bf2f(hb);
}

__global__ void quantize_kernel(const float *__restrict__ w, int n, float *__restrict__ wq, uint16_t *__restrict__ wbf) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint16_t hb = f2bf(w[i]);
    wbf[i] = hb;
    wq[i] = bf2f(hb);
}

inline unsigned blocks_for(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

// Offsets of each layer's weights and bias in the flat parameter array.
void cnn_layout(int c, int *w_off, int *b_off, int *total) {
    const int ci[6] = {c, 32, 32, 32, 32, 32}, co[6] = {32, 32, 32, 32, 32, 1};
    int off = 0;
    for (int l = 0; l < 6; ++l) {
        w_off[l] = off;
        off += co[l] * 9 * ci[l];
        b_off[l] = off;
        off += co[l];
    }
    *total = off;
}

static ConvShape shape_of(int l, int N, int H, int W, int c) {
    // l = 0..5: the layer; its input size is the output size of the layers before it
    // spatial size entering layer l
    int h = H, w = W;
    const int strides[6] = {2, 2, 2, 1, 1, 1};
    for (int k = 0; k < l; ++k) {
        h = (h + strides[k] - 1) / strides[k];
        w = (w + strides[k] - 1) / strides[k];
    }
    ConvShape cs;
    cs.N = N; cs.H = h; cs.W = w;
    cs.Ci = l == 0 ? c : 32;
    cs.Co = l == 5 ? 1 : 32;
    cs.s = strides[l];
    cs.Ho = (h + cs.s - 1) / cs.s;
    cs.Wo = (w + cs.s - 1) / cs.s;
    return cs;
}

// Activation sizes (elements) for a batch: a[1..5] bf16 (32 channels), z FP32.
size_t cnn_act_elems(int l, int N, int H, int W, int c) {
    ConvShape cs = shape_of(l - 1, N, H, W, c);
    return (size_t)cs.N * cs.Ho * cs.Wo * cs.Co;
}

static hipError_t forward_impl(const CnnBuffers &b, const uint8_t *img, int64_t img_stride,
                               int64_t img_batch_stride, const uint8_t *const *img_tab, const int64_t *stride_tab,
                               int N, int H, int W, int c, hipStream_t st) {
    int wo[6], bo[6], tot;
    cnn_layout(c, wo, bo, &tot);
    ConvShape cs = shape_of(0, N, H, W, c);
    int64_t np = (int64_t)cs.N * cs.Ho * cs.Wo;
    if (c == 3)
        hipLaunchKernelGGL(l1_fwd_kernel<3>, dim3(blocks_for(np, 256)), dim3(256), 0, st, img, img_stride,
                           img_batch_stride, img_tab, stride_tab, cs, b.wq + wo[0], b.wq + bo[0], b.act[1]);
    else if (c == 1)
        hipLaunchKernelGGL(l1_fwd_kernel<1>, dim3(blocks_for(np, 256)), dim3(256), 0, st, img, img_stride,
                           img_batch_stride, img_tab, stride_tab, cs, b.wq + wo[0], b.wq + bo[0], b.act[1]);
    else
        return hipErrorInvalidValue;
    for (int l = 1; l < 5; ++l) {
        cs = shape_of(l, N, H, W, c);
        np = (int64_t)cs.N * cs.Ho * cs.Wo;
        const int64_t tiles = (np + 15) / 16;
        const int64_t want = (tiles + 3) / 4;
        const unsigned grid = (unsigned)(want < 4096 ? want : 4096);
        hipLaunchKernelGGL(conv32_fwd_kernel, dim3(grid), dim3(256), 0, st, b.act[l], cs, b.wbf + wo[l],
                           b.wq + bo[l], b.act[l + 1], 1);
    }
    cs = shape_of(5, N, H, W, c);
    np = (int64_t)cs.N * cs.Ho * cs.Wo;
    hipLaunchKernelGGL(l6_fwd_kernel, dim3(blocks_for(np, 256)), dim3(256), 0, st, b.act[5], cs, b.wq + wo[5],
                       b.wq + bo[5], b.z);
    return hipGetLastError();
}

hipError_t cnn_forward(const CnnBuffers &b, const uint8_t *img, int64_t img_stride, int64_t img_batch_stride,
                       int N, int H, int W, int c, hipStream_t st) {
    return forward_impl(b, img, img_stride, img_batch_stride, nullptr, nullptr, N, H, W, c, st);
}

hipError_t cnn_forward_tab(const CnnBuffers &b, const uint8_t *const *img_tab, const int64_t *stride_tab, int N,
                           int H, int W, int c, hipStream_t st) {
    if (!img_tab || !stride_tab) return hipErrorInvalidValue;
    return forward_impl(b, nullptr, 0, 0, img_tab, stride_tab, N, H, W, c, st);
}

// Backward pass: grads (FP32, zeroed here) of mean |z - target|; d0/d1 are FP32 scratch
// buffers large enough for the largest activation.
hipError_t cnn_backward(const CnnBuffers &b, const uint8_t *img, int64_t img_stride, int64_t img_batch_stride,
                        int N, int H, int W, int c, const float *target, float *grads, float *d0, float *d1,
                        double *loss_sum, hipStream_t st) {
    int wo[6], bo[6], tot;
    cnn_layout(c, wo, bo, &tot);
    hipError_t e = launch_zero(grads, sizeof(float) * tot, st);
    if (e != hipSuccess) return e;
    e = launch_zero(loss_sum, sizeof(double), st);
    if (e != hipSuccess) return e;
    ConvShape cs = shape_of(5, N, H, W, c);
    const int64_t nz = (int64_t)cs.N * cs.Ho * cs.Wo;
    float *dy = d0, *dx = d1;
    hipLaunchKernelGGL(l1loss_kernel, dim3(blocks_for(nz, 256)), dim3(256), 0, st, b.z, target, nz, dy, loss_sum);
    for (int l = 5; l >= 0; --l) {
        cs = shape_of(l, N, H, W, c);
        const int64_t np = (int64_t)cs.N * cs.Ho * cs.Wo;
        // pixels per wave: at least two groups of loads, at most 256 workgroups (each adds its sums
        // to the whole gradient)
        const int64_t want = (np + 256 * WG_WAVES - 1) / (256 * WG_WAVES);
        const int chunk = (int)std::max<int64_t>(4 * WG_AHEAD, (want + 2 * WG_AHEAD - 1) / (2 * WG_AHEAD) * 2 * WG_AHEAD);
        const unsigned grid = (unsigned)((np + (int64_t)chunk * WG_WAVES - 1) / ((int64_t)chunk * WG_WAVES));
        if (l == 0) {
            const int lds = WG_WAVES * 1024 * 4;
            hipLaunchKernelGGL(wgrad_mfma_kernel<1>, dim3(grid), dim3(64 * WG_WAVES), lds, st, nullptr, img, img_stride,
                               img_batch_stride, cs, dy, chunk, grads + wo[l], grads + bo[l]);
        } else {
            const int lds = WG_WAVES * 9 * 1024 * 4;
            if ((e = prepare_dynamic_lds((const void *)wgrad_mfma_kernel<9>, lds, 64 * WG_WAVES * 4)) != hipSuccess)
                return e;
            hipLaunchKernelGGL(wgrad_mfma_kernel<9>, dim3(grid), dim3(64 * WG_WAVES), lds, st, b.act[l], nullptr,
                               (int64_t)0, (int64_t)0, cs, dy, chunk, grads + wo[l], grads + bo[l]);
        }
        if (l > 0) {   // with the ReLU backward of layer l - 1
            const int64_t nq = (int64_t)cs.N * cs.H * cs.W;
            if (cs.Co == 1) {
                hipLaunchKernelGGL(dgrad_kernel, dim3(blocks_for(nq * cs.Ci, 256)), dim3(256), 0, st, dy, cs,
                                   b.wq + wo[l], b.act[l], dx);
            } else {
                const int64_t tiles = nq / 32 + 4;
                const unsigned wgs = (unsigned)std::min<int64_t>(1024, (tiles + DG_WAVES - 1) / DG_WAVES);
                hipLaunchKernelGGL(dgrad32_kernel, dim3(wgs), dim3(64 * DG_WAVES), 0, st, dy, cs, b.wq + wo[l],
                                   b.act[l], dx);
            }
            float *t = dy; dy = dx; dx = t;
        }
    }
    return hipGetLastError();
}

hipError_t cnn_adam(float *w, float *m, float *v, const float *g, int n, float lr, int64_t step, float *wq,
                    uint16_t *wbf, hipStream_t st) {
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    hipLaunchKernelGGL(adam_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, w, m, v, g, n, lr, b1, b2, eps, c1, c2,
                       wq, wbf);
    return hipGetLastError();
}

hipError_t cnn_quantize(const float *w, int n, float *wq, uint16_t *wbf, hipStream_t st) {
    hipLaunchKernelGGL(quantize_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, w, n, wq, wbf);
    return hipGetLastError();
}

uint16_t host_f2bf(float f) { return f2bf(f); }

}  // namespace htsvd
