// Hyperspectral tube patches (Sec. IV-D): Haar-tSVD on an h x w x B cube with 8 x 8 x B patches.
//
// Grouping runs on a gray guide, the band mean rounded half up (the block matcher of the other
// paths, Eq. 9 on one channel).  The transform runs in FP64 (so that keep/kill decisions agree
// with an FP64 reference without a guard band).  The t-product S = U^T * P * V (Eq. 19) is taken
// along the band axis through its DFT (Eq. 4-5): the real band DFT of each of the 64 tubes of a
// patch, per frequency f the 8 x 8 complex slice products U_hat_f^H P_hat_f V_hat_f, and the
// inverse band DFT, with the patch spectra in LDS.
//
// The Haar transform runs along the group and the t-product along the patch, so they commute, and
// the transform along the group comes first, on the whole-number pixels (band_haar_kernel).  Each
// Haar row of a group is then a patch of its own: t-product, threshold (Eq. 20) and inverse
// t-product (Eq. 21) in one kernel (band_rows_kernel), the coefficients never leaving the
// registers, and most difference rows are shown to keep nothing in fp16 before (band_test_kernel).
// Last the inverse Haar transform and the uniform aggregation sums (Algorithm 1) in 64-bit fixed
// point, exact, so that the result does not depend on the order of the additions (band_add_kernel).
//
// 256 x 256 x 31, K = 16, noise 30 (63,504 rows): 71 + 113 + 118 + 129 us in this order, against
// 2,062 us with the coefficients of the members in memory between the t-product (630 us), the Haar
// transform with the threshold (349) and the inverse t-product with an atomic per value (1,082).
// With every row kept the whole call takes 1.42 ms (2.13).
#include "common.h"

namespace htsvd {

namespace {

constexpr int BFS = 16;   // aggregation fixed point: values in units of 2^-16

__global__ void guide_kernel(const uint8_t *__restrict__ cube, int64_t stride, int h, int w, int B,
                             uint8_t *__restrict__ guide) {
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= (int64_t)h * w) return;
    const int y = (int)(q / w), x = (int)(q % w);
    const uint8_t *p = cube + (int64_t)y * stride + (int64_t)x * B;
    int s = 0;
    for (int b = 0; b < B; ++b) s += p[b];
    guide[q] = (uint8_t)((s + B / 2) / B);
}

typedef double dbl4 __attribute__((ext_vector_type(4)));

// The real band DFT separates into cosines of the even part of a tube, x_b + x_{B-b}, and sines of
// the odd part, x_b - x_{B-b} (b < NF = B / 2 + 1; x_0, and x_{B/2} of an even B, stand alone), each
// half as many rows and columns as the whole DFT: a quarter of the products each.  FB is the number
// of 16-row blocks of the cosines: 1 for B <= 31, 2 up to 63, 3 for 64; and 0 for 32 bands, one block and a
// 17th cosine, which lanes sum from the operands of the block (with a second block, of that row alone,
// the call for 256 x 256 x 32 at K 16 and noise 10 took 2.40 ms instead of 1.42).
//
// The workgroup's patches and the LDS layout of their spectra: value (i, j) of component c of patch p
// at Z[p*ZP + c*64 + zpos(c, i, j)], component f the real part of frequency f and IM + f its
// imaginary part.  The XOR of j with a function of i, the rotation of the odd components by 16 and
// the patch stride of 16 modulo 32 doubles keep the accesses of the phases free of bank conflicts (64
// banks of 4 bytes: a wave's 32-lane halves reach 32 distinct double slots).
template <int FB> struct BandTile {
    static constexpr int PP = 2;                            // patches per workgroup (256 threads), two waves each
    static constexpr int CB = FB == 0 ? 1 : FB;
    static constexpr int KS = FB == 3 ? 9 : FB == 0 ? 5 : 4 * FB;   // k-steps of a cosine product
    static constexpr int KS1 = FB == 0 ? 4 : KS;                    // of a sine product
    // component of the imaginary part of frequency f, which frequency 0 has not, less f; odd where that costs
    // nothing, so that both parts of a frequency keep free of bank conflicts
    static constexpr int IM = FB == 3 ? 32 : FB == 0 ? 17 : 16 * FB - 1;
    static constexpr int ZP = (FB == 0 ? 33 : FB == 1 ? 31 : (FB == 2 ? 63 : 64)) * 64 + 16;   // doubles per patch
    static constexpr bool OPS = FB < 2;                             // operands in LDS
    static constexpr int N_OPS = OPS ? 4 * KS * 64 + (FB == 0 ? 2 * 4 * KS : 0) : 1;
};

__device__ inline int zpos(int c, int i, int j) {
    return (8 * i + (j ^ (((i >> 2) << 1) ^ (((i >> 1) & 1) << 2))) + 16 * (c & 1)) & 63;
}

// Every product below is on v_mfma_f64_16x16x4f64 (lanes: A(m, k) in m + 16 (k mod 4), B(k, n) in
// n + 16 (k mod 4), result (m, n) in register m / 4 of lane n + 16 (m mod 4)): with positions e as
// the columns, register r of block cb of a result, its row 16 cb + 4 r + q, is the B operand of
// k-step 4 cb + r of the next product.

// Row of the real part of frequency f in D, and column in Dinv; its imaginary part follows.
__device__ inline int re_row(int f, int B) { return f == 0 ? 0 : (2 * f == B ? B - 1 : 2 * f - 1); }

// A operands of block cb of the cosine (part 0) or sine (part 1) products: of the DFT (frequencies
// as rows, bands as columns), or of its inverse.  Rows and columns beyond NF repeat the last: those
// rows are not used, those columns meet zeros.  Read from memory a lane's rows lie apart, and the first
// cache's lookups bound the whole kernel (926 us for all of 63,504 rows of 31 bands; from LDS, with
// the next row's sums loaded ahead, 797), so for one block a workgroup keeps them in LDS.
template <int FB, bool INV>
__device__ __forceinline__ void band_operand(const double *__restrict__ M, int B, int nb, int part, int cb, int lane,
                                             double (&a)[BandTile<FB>::KS]) {
    const int q = lane >> 4, col = lane & 15;
#pragma unroll
    for (int s = 0; s < BandTile<FB>::KS; ++s) {
        const int m = 16 * cb + col, k = 4 * s + q;
        const int f = min(INV ? k : m, part ? (B - 1) / 2 : B / 2), b = min(INV ? m : k, B / 2);
        const int row = part ? 2 * f : re_row(f, B);   // the sine of frequency 0 meets zeros as well
        a[s] = M[INV ? b * nb + row : row * nb + b];
    }
}

// The same from LDS.
template <int FB, bool INV>
__device__ __forceinline__ void band_operand_lds(const double *ops, int part, int lane, double (&a)[BandTile<FB>::KS]) {
#pragma unroll
    for (int s = 0; s < BandTile<FB>::KS; ++s) a[s] = ops[((2 * INV + part) * BandTile<FB>::KS + s) * 64 + lane];
}

// Row 16 of the cosine product of 32 bands, or of its inverse, in every lane of a position: columns 4 s + q by
// the lanes q, whose sums are added.
template <bool INV>
__device__ __forceinline__ double band_last(const double *ops, const double (&x)[BandTile<0>::KS], int q) {
    constexpr int KS = BandTile<0>::KS;
    const double *a = ops + 4 * KS * 64 + 4 * KS * INV + q;
    double t = 0.0;
#pragma unroll
    for (int s = 0; s < KS; ++s) t = fma(a[4 * s], x[s], t);
    t += __shfl_xor(t, 16);
    return t + __shfl_xor(t, 32);
}

// Band DFT of a wave's 32 positions: component c of e from the even and odd parts x of its tube.
template <int FB>
__device__ __forceinline__ void band_dft(const double *__restrict__ D, const double *ops, int nb,
                                         const double (&x)[2][2][BandTile<FB>::KS],
                                         double *z, int B, int half, int lane) {
    const int q = lane >> 4, col = lane & 15, NF = B / 2 + 1, NS = (B + 1) / 2;
#pragma unroll
    for (int part = 0; part < 2; ++part) {
        const int rows = part ? NS : NF;
#pragma unroll
        for (int cb = 0; cb < BandTile<FB>::CB; ++cb) {
            if (FB > 1 && 16 * cb >= rows) continue;
            double a[BandTile<FB>::KS];
            if constexpr (BandTile<FB>::OPS)
                band_operand_lds<FB, false>(ops, part, lane, a);
            else
                band_operand<FB, false>(D, B, nb, part, cb, lane, a);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int e = 32 * half + 16 * u + col;
                dbl4 t = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int s = 0; s < (part ? BandTile<FB>::KS1 : BandTile<FB>::KS); ++s)
                    if (FB < 2 || 4 * s < rows) t = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], x[part][u][s], t, 0, 0, 0);
                // the parity of a component is that of q (of its imaginary part, the other): constant steps
                const int c0 = (part ? BandTile<FB>::IM : 0) + 16 * cb + q;
                double *zc = z + c0 * 64 + zpos(c0, e >> 3, e & 7);
#pragma unroll
                for (int r = 0; r < 4; ++r)   // FB = 1: rows past the last frequency land in slots nobody reads
                    if ((FB < 2 || 16 * cb + q + 4 * r < rows) && (!part || cb || r || q)) zc[r * 256] = t[r];
                if constexpr (FB == 0) {
                    if (part == 0) {
                        const double last = band_last<false>(ops, x[0][u], q);
                        if (q == 0) z[16 * 64 + zpos(16, e >> 3, e & 7)] = last;
                    }
                }
            }
        }
    }
}

// Inverse band DFT of a wave's 32 positions: the even and odd parts E and O of the tube, as
// y[0] = E + O at band b = 4 s + q and y[1] = E - O at band B - b.
template <int FB>
__device__ __forceinline__ void band_idft(const double *__restrict__ Dinv, const double *ops, int nb,
                                          const double *z, double (&y)[2][2][BandTile<FB>::KS], int B, int half, int lane) {
    constexpr int KS = BandTile<FB>::KS;
    const int q = lane >> 4, col = lane & 15, NF = B / 2 + 1, NS = (B + 1) / 2;
    double v[2][2][KS];
#pragma unroll
    for (int part = 0; part < 2; ++part)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const int f = 4 * s + q, e = 32 * half + 16 * u + col, c0 = (part ? BandTile<FB>::IM : 0) + q;
                const bool in = f >= part && f < (part ? NS : NF);
                // 32 and 64 bands: 4 s + q may pass the last slot
                const int c = FB == 1 || FB == 2 || in ? c0 + 4 * s : c0;
                const double t = z[c * 64 + zpos(c0, e >> 3, e & 7)];
                v[part][u][s] = in ? t : 0.0;
            }
#pragma unroll
    for (int cb = 0; cb < BandTile<FB>::CB; ++cb) {
        dbl4 t[2][2];
#pragma unroll
        for (int part = 0; part < 2; ++part) {
            double a[KS];
            if constexpr (BandTile<FB>::OPS)
                band_operand_lds<FB, true>(ops, part, lane, a);
            else
                band_operand<FB, true>(Dinv, B, nb, part, cb, lane, a);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                t[part][u] = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int s = 0; s < (part ? BandTile<FB>::KS1 : KS); ++s)
                    if (FB < 2 || 4 * s < (part ? NS : NF))
                        t[part][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], v[part][u][s], t[part][u], 0, 0, 0);
            }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (4 * cb + r < KS) {
                    y[0][u][4 * cb + r] = t[0][u][r] + t[1][u][r];
                    y[1][u][4 * cb + r] = t[0][u][r] - t[1][u][r];
                }
    }
    if constexpr (FB == 0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {   // band 16 has no odd part; lanes q > 0 hold no band here
            y[0][u][4] = band_last<true>(ops, v[0][u], q);
            y[1][u][4] = 0.0;
        }
    }
}

// Per frequency f (f = wave modulo 4) the slice products T = L * P_f and Y_f = T * R of the two
// patches at once, with complex 8 x 8 matrices in their real 16 x 16 embeddings:
//   L on the left,  [[Lr, -Li], [Li, Lr]] times P stacked as [Pr; Pi] (columns: 2 patches x 8);
//   R on the right, T laid out as [Tr | Ti] (rows: 2 patches x 8) times [[Rr, Ri], [-Ri, Rr]];
// T goes back to the LDS slots of P_f and Y_f to the same slots (the slots of f belong to one wave,
// and its LDS accesses execute in order).  The operands of the next f are loaded ahead of use.
template <int FB>
__device__ __forceinline__ void band_slices(const double *__restrict__ frag, double (&nx)[8], double *Z, int B, int wave,
                                            int lane) {
    constexpr int ZP = BandTile<FB>::ZP, IM = BandTile<FB>::IM;
    const int q = lane >> 4, col = lane & 15, NF = B / 2 + 1;
    // f keeps its parity, so every place moves by the same step; [part][i or j = q, 4 + q]
    double *left[2][2], *mid[2][2], *out[4];
#pragma unroll
    for (int ri = 0; ri < 2; ++ri) {
        const int c = (ri ? IM : 0) + wave;
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            left[ri][v] = Z + (col >> 3) * ZP + c * 64 + zpos(c, 4 * v + q, col & 7);   // columns (p, j)
            mid[ri][v] = Z + (col >> 3) * ZP + c * 64 + zpos(c, col & 7, 4 * v + q);    // rows (p, i')
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int c = (col >> 3 ? IM : 0) + wave;
        out[r] = Z + (r >> 1) * ZP + c * 64 + zpos(c, q + 4 * (r & 1), col & 7);   // rows (p, i'), columns (ri', j')
    }
    const double *fp = frag + (size_t)wave * 512 + lane;
    for (int f = wave, step = 0; f < NF; f += 4, step += 256) {
        double fr[8];
#pragma unroll
        for (int v = 0; v < 8; ++v) fr[v] = nx[v];
        fp += 4 * 512;
        if (f + 4 < NF) {
#pragma unroll
            for (int v = 0; v < 8; ++v) nx[v] = fp[v * 64];
        }
        const bool real = f == 0 || 2 * f == B;   // no imaginary part: its slot belongs to no component or another one
        // T = L * [Pr; Pi]: B operand rows k = 4s + q = (ri, i), columns col = (p, j)
        dbl4 t = {0.0, 0.0, 0.0, 0.0};
        double v[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) v[s] = left[real ? 0 : s >> 1][s & 1][step];
        if (real) v[2] = v[3] = 0.0;
#pragma unroll
        for (int s = 0; s < 4; ++s) t = __builtin_amdgcn_mfma_f64_16x16x4f64(fr[s], v[s], t, 0, 0, 0);
        // result rows q + 4r = (ri', i'), columns (p, j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (!(r >> 1 && real)) left[r >> 1][r & 1][step] = t[r];
        // Y = [Tr | Ti] * R: A operand rows col = (p, i'), columns k = 4s + q = (ri, j)
#pragma unroll
        for (int s = 0; s < 4; ++s) v[s] = mid[real ? 0 : s >> 1][s & 1][step];
        if (real) v[2] = v[3] = 0.0;
        t = dbl4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 4; ++s) t = __builtin_amdgcn_mfma_f64_16x16x4f64(v[s], fr[4 + s], t, 0, 0, 0);
        if (!real || col < 8) {
#pragma unroll
            for (int r = 0; r < 4; ++r) out[r][step] = t[r];
        }
    }
}

// The first operands of a wave's slices.
__device__ __forceinline__ void band_slices_load(const double *__restrict__ frag, double (&nx)[8], int B, int wave, int lane) {
    if (wave < B / 2 + 1) {
#pragma unroll
        for (int v = 0; v < 8; ++v) nx[v] = frag[(size_t)wave * 512 + v * 64 + lane];
    }
}

// Slot of row n of the chunk's groups (row r of group g is n = g K + r): 64 B doubles.  First the
// even and odd parts of the row's whole-number sums, 16-bit, (part, k-step s, position, band 4 s + i)
// per block of 16 positions, which fit the slot at any B; then its estimate (block of 8 bands,
// position e, band), or in the first double a NaN where no coefficient is kept.
//
// Haar sums of the pixels of a group before any scaling: whole numbers of at most 14 bits and a sign,
// the folding included.  The transform runs along the group and the t-product along the patch, so
// they commute, and 2 bytes per value are written here where the coefficients would take 8.  One
// wave per group and block of 16 positions; a lane takes bands 4 s .. 4 s + 3 and their partners
// B - 4 s - 3 .. B - 4 s as 4 bytes each (one byte per lane and load was bound by the number of
// memory instructions: 183 us for 63,504 patches of 31 bands).
typedef short sh2 __attribute__((ext_vector_type(2)));

template <int K, bool TWO>   // TWO: two bands, which have no partners (B = 3 is no band count)
__global__ __launch_bounds__(256) void band_haar_kernel(const uint8_t *__restrict__ cube, int64_t stride, int w, int B,
                                                        const int32_t *__restrict__ idx, double *__restrict__ S) {
    const int64_t g = blockIdx.x;
    const int lane = threadIdx.x & 63, blk = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int e = 16 * blk + (lane & 15), NF = B / 2 + 1, KS = (NF + 3) >> 2;
    const int32_t lin = idx[g * K + (lane & (K - 1))];
    const int64_t off = (int64_t)(lin / w) * stride + (int64_t)(lin % w) * B;
    const int64_t pos = (e >> 3) * stride + (e & 7) * B;
    for (int s0 = 0; s0 < KS; s0 += 4) {   // all lanes stay active: the members' offsets lie in the lanes
        const int s = min(s0 + (lane >> 4), KS - 1);
        const bool own = s0 + (lane >> 4) < KS;
        // bytes of the bands below NF, of those with an odd part (not B / 2), and of the partners of
        // bands b >= 1 with 2 b < B (the partner of band 4 s + i in byte 3 - i; from byte B - 4 on
        // where s = 0, shifted down by one)
        const int nf = min(4, NF - 4 * s), np = min(4, (B + 1) / 2 - 4 * s);
        const uint32_t fm = (uint32_t)((1ull << (8 * nf)) - 1);
        const uint32_t om = np > 0 ? (uint32_t)((1ull << (8 * np)) - 1) : 0u;
        const uint32_t rm = np > 0 ? (uint32_t)~((1ull << (32 - 8 * np)) - 1) : 0u;
        const int rs = s == 0 ? 8 : 0, rat = s == 0 ? B - 4 : B - 4 * s - 3;
        uint32_t f[K], r[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint8_t *m = cube + (((int64_t)__builtin_amdgcn_readlane((int)(off >> 32), k) << 32) |
                                       (uint32_t)__builtin_amdgcn_readlane((int)off, k));
            r[k] = 0;
            if constexpr (TWO) {
                f[k] = m[pos] | (uint32_t)m[pos + 1] << 8;
            } else {
                __builtin_memcpy(&f[k], m + pos + 4 * s, 4);
                __builtin_memcpy(&r[k], m + pos + rat, 4);
            }
        }
#pragma unroll
        for (int part = 0; part < 2; ++part) {
            sh2 v[2][K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const uint32_t fk = f[k] & (part ? om : fm), rk = (r[k] >> rs) & rm;
                const sh2 f0 = __builtin_bit_cast(sh2, __builtin_amdgcn_perm(0u, fk, 0x0c010c00u));
                const sh2 f1 = __builtin_bit_cast(sh2, __builtin_amdgcn_perm(0u, fk, 0x0c030c02u));
                const sh2 r0 = __builtin_bit_cast(sh2, __builtin_amdgcn_perm(0u, rk, 0x0c020c03u));
                const sh2 r1 = __builtin_bit_cast(sh2, __builtin_amdgcn_perm(0u, rk, 0x0c000c01u));
                v[0][k] = part ? f0 - r0 : f0 + r0;
                v[1][k] = part ? f1 - r1 : f1 + r1;
            }
            // at each level the pair sums move to the front, the differences stay in place
#pragma unroll
            for (int h = 1; h < K; h <<= 1)
#pragma unroll
                for (int i = 0; i < K; i += 2 * h)
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const sh2 a = v[t][i], c = v[t][i + h];
                        v[t][i] = a + c;
                        v[t][i + h] = a - c;
                    }
            if (own) {
                uint2 *out = reinterpret_cast<uint2 *>(S + g * K * 64 * B) + ((2 * blk + part) * KS + s) * 16 + (lane & 15);
#pragma unroll
                for (int k = 0; k < K; ++k)
                    out[k * 64 * B] = make_uint2(__builtin_bit_cast(uint32_t, v[0][k]), __builtin_bit_cast(uint32_t, v[1][k]));
            }
        }
    }
}

constexpr double R2 = 0.70710678118654752440;

// A wave's LDS accesses execute in order; the compiler may not move them over this point.
__device__ inline void wave_lds_sync() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

// Scale of row r of a group of K: row 0 has been summed log2 K times, row r as often as its lowest set
// bit says and once more.
__device__ inline double row_scale(int r, int K) {
    const int lev = r ? __builtin_ctz(r) + 1 : __builtin_ctz(K);
    return ((lev & 1) ? R2 : 1.0) / (double)(1 << (lev >> 1));
}

typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ inline h4 to_h4(f4 v) { return __builtin_convertvector(v, h4); }

// Which rows need the FP64 transform (B <= 31).  Nearly all differences of a group hold noise alone and
// keep no coefficient, and FP64 products are 16 times as dear as fp16 ones, so every row is transformed
// in fp16 first (63,504 rows of 31 bands: 113 us, and 118 us for the rows listed, against 797 us for
// all of them in FP64), with a bound on its error, and only rows whose largest coefficient may reach tau are
// listed (row 0 always); the others get their mark here.
//
// Bound.  All three stages are written with orthonormal factors (the DFT scaled by c_f = sqrt(2 / B),
// sqrt(1 / B) at frequencies 0 and B / 2; unitary slices), so an error vector reaches one coefficient
// with at most its 2-norm.  With u = 2^-11 and |x| the norm of the row: the DFT's factors are split
// into two halves and whole numbers up to 2048 are exact in fp16 (else their rounding adds u |x| at most, as
// the DFT of the folded row has a spectral norm of 1 at most; 1.1 sqrt(B) u |x| is taken, which is more for
// every B); each of the two slice products errs by
// u per entry of its factor, 16 entries of unit norm to a row: 4 u |x|; each of the three
// results stored as fp16 adds u |x|; the last factor u |x|.  Sum 12 u |x|, 13 with the second-order and
// FP32 terms, and 0.02 for values below fp16's normal range.  Infinities and NaN count as large.
//
// One wave per two rows and pass, every product on v_mfma_f32_16x16x16_f16 (A(m, k) in lane
// m + 16 (k / 4), element k mod 4; B(k, n) likewise; result row 4 (lane / 16) + r, column lane mod 16):
//   1. Z'(e, f) = sum_b x(e, b) D'(b, f): the row's sums lie in memory as the A operand; stored as
//      [f][re, im][row][e];
//   2. per frequency T = [Pr | Pi] R (rows: 2 rows x 8), then Y = L [Tr; Ti] (columns: 2 rows x 8):
//      the lanes swap bits 3 and 5 in between;
//   3. E(e, b) and O(e, b), the even and odd part of the coefficients, from Y stored as
//      [row][re, im][e][f]: the larger of |E + O| and |E - O| is |E| + |O|.
// The test takes 20 us however few rows there are, and up to 2,048 rows go through the FP64 transform in
// one round of the workgroups, with a time that goes with the bands: 968 rows of 31 bands 76 us for the
// call with the test and 60 without (16 bands: 72 and 54), 1,936 rows 88 and 82, 3,600 rows 95 and 111
// (16 bands: 90 and 95; 7 bands: 79 and 82).  Passes of more rows than this are tested.
inline int test_min_rows(int B) { return 2048 + 64 * (31 - B); }
constexpr int TEST_ROWS = 8;         // rows per wave and pass: one list reservation
constexpr int TEST_F = 544;          // bytes per frequency of Z' (512 and 8 banks)
__global__ __launch_bounds__(256, 3) void band_test_kernel(int B, int nb, int K, int64_t n_row,
                                                        const double *__restrict__ D, const double *__restrict__ frag,
                                                        double tau, double *__restrict__ S, int *__restrict__ list,
                                                        int *__restrict__ n_list) {
    __shared__ __align__(16) h4 fac[16 * 2 * 64];              // R and L of every frequency
    __shared__ __align__(16) unsigned char buf[4][16 * TEST_F];   // per wave: Z', then Y
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, col = lane & 15, NF = B / 2 + 1, KS = (NF + 3) >> 2;
    for (int t = tid; t < 16 * 128; t += 256) {   // zero beyond the last frequency
        const double *fr = frag + (size_t)min(t >> 7, NF - 1) * 512 + ((t >> 6 & 1 ? 0 : 4) + q) * 64 + col;
        const float on = t >> 7 < NF ? 1.0f : 0.0f;
        fac[t] = to_h4((f4){(float)fr[0], (float)fr[16], (float)fr[32], (float)fr[48]} * on);
    }
    // D' by (band 4 q + i, frequency col) in two halves, and by (frequency 4 q + i, band col)
    h4 dh[2], dl[2], di[2];
    const double c1 = sqrt(1.0 / B), c2 = sqrt(2.0 / B);
#pragma unroll
    for (int part = 0; part < 2; ++part)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            auto entry = [&](int f, int b) {   // loads without branches, so that they overlap
                const int fc = min(f, part ? (B - 1) / 2 : NF - 1), bc = min(b, NF - 1);
                const double c = D[(part ? 2 * fc : re_row(fc, B)) * nb + bc] * (f == 0 || 2 * f == B ? c1 : c2);
                return f < part || f != fc || b != bc ? 0.0f : (float)c;
            };
            const float v = entry(col, 4 * q + i);
            dh[part][i] = (_Float16)v;
            dl[part][i] = (_Float16)(v - (float)dh[part][i]);
            di[part][i] = (_Float16)entry(4 * q + i, col);
        }
    __syncthreads();
    unsigned char *zb = buf[wave];
    const float width = 1.1f * sqrtf((float)B);

    for (int64_t n8 = ((int64_t)blockIdx.x * 4 + wave) * TEST_ROWS; n8 < n_row; n8 += (int64_t)gridDim.x * 4 * TEST_ROWS) {
        uint32_t need = 0;   // bit i: row n8 + i goes on the list
        uint2 raw[2][4][2];  // (row, block of 16 positions, part), loaded a pair ahead
        auto load = [&](int64_t n2) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const uint2 *in = reinterpret_cast<const uint2 *>(S + min(n2 + p, n_row - 1) * 64 * B) + min(q, KS - 1) * 16 + col;
#pragma unroll
                for (int blk = 0; blk < 4; ++blk)
#pragma unroll
                    for (int part = 0; part < 2; ++part) raw[p][blk][part] = in[(2 * blk + part) * KS * 16];
            }
        };
        load(n8);
        for (int n2 = 0; n2 < TEST_ROWS && n8 + n2 < n_row; n2 += 2) {
            float sq[2];
            bool big[2];
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                int two = 0;    // twice the squared norm, saturating
                int twin = 0;   // squares at band B / 2, which has no odd part
#pragma unroll
                for (int blk = 0; blk < 4; ++blk) {
                    f4 z[2];
#pragma unroll
                    for (int part = 0; part < 2; ++part) {
                        const uint2 w = raw[p][blk][part];   // lanes q >= KS: any number, times zero
                        const sh2 w0 = __builtin_bit_cast(sh2, w.x), w1 = __builtin_bit_cast(sh2, w.y);
                        two = __builtin_amdgcn_sdot2(w0, w0, __builtin_amdgcn_sdot2(w1, w1, two, true), true);
                        if (part == 0 && !(B & 1)) {
                            const int m = (B >> 1) & 3, xm = m < 2 ? w0[m & 1] : w1[m & 1];
                            twin += q == B >> 3 ? (xm * xm >> 2) + 1 : 0;   // a quarter, rounded up: four blocks fit
                        }
                        const h4 x = (h4){(_Float16)w0[0], (_Float16)w0[1], (_Float16)w1[0], (_Float16)w1[1]};
                        z[part] = __builtin_amdgcn_mfma_f32_16x16x16f16(x, dl[part], (f4){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                        z[part] = __builtin_amdgcn_mfma_f32_16x16x16f16(x, dh[part], z[part], 0, 0, 0);
                    }
                    // positions 16 blk + 4 q .. + 3 of frequency col
#pragma unroll
                    for (int part = 0; part < 2; ++part)
                        *reinterpret_cast<h4 *>(zb + col * TEST_F + part * 256 + p * 128 + 32 * blk + 8 * q) = to_h4(z[part]);
                }
                two = q < KS ? two : 0;
                // a number beyond 2048 shows in its lane's sum
                big[p] = __builtin_amdgcn_ballot_w64(two > 4194304) != 0;
                float sum = two == 0x7fffffff ? __builtin_inff() : (float)two + 4.0f * (float)twin;
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
                sq[p] = 0.5f * sum;
            }
            if (n2 + 2 < TEST_ROWS && n8 + n2 + 2 < n_row) load(n8 + n2 + 2);
            wave_lds_sync();
            h4 y[4][4];   // (quad of frequencies, register r), element: the frequency
#pragma unroll
            for (int fq = 0; fq < 4; ++fq)
#pragma unroll
                for (int fi = 0; fi < 4; ++fi) {
                    const int f = 4 * fq + fi;
                    const h4 pa = *reinterpret_cast<const h4 *>(zb + f * TEST_F + (q >> 1) * 256 + col * 16 + (q & 1) * 8);
                    const f4 t = __builtin_amdgcn_mfma_f32_16x16x16f16(pa, fac[f * 128 + lane], (f4){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                    const uint2 th = __builtin_bit_cast(uint2, to_h4(t));
                    const int from = (lane & 23) | (lane & 8) << 2 | (lane & 32) >> 2;
                    const uint2 sw = make_uint2((uint32_t)__builtin_amdgcn_ds_bpermute(4 * from, (int)th.x),
                                                (uint32_t)__builtin_amdgcn_ds_bpermute(4 * from, (int)th.y));
                    const f4 v = __builtin_amdgcn_mfma_f32_16x16x16f16(fac[f * 128 + 64 + lane], __builtin_bit_cast(h4, sw),
                                                                       (f4){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < 4; ++r) y[fq][r][fi] = (_Float16)v[r];
                }
            // lane: re or im q / 2, row col / 8, position (4 (q mod 2) + r, col mod 8)
            wave_lds_sync();
            {
                const int pr = 2 * (col >> 3) + (q >> 1);
#pragma unroll
                for (int fq = 0; fq < 4; ++fq)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        *reinterpret_cast<h4 *>(zb + pr * 2048 + ((4 * (q & 1) + r) * 8 + (col & 7)) * 32 + 8 * (fq ^ pr)) = y[fq][r];
            }
            wave_lds_sync();
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                uint32_t top = 0;   // bits of the largest sum; infinities and NaN are larger still
#pragma unroll
                for (int blk = 0; blk < 4; ++blk) {
                    f4 eo[2];
#pragma unroll
                    for (int part = 0; part < 2; ++part) {
                        const h4 a = *reinterpret_cast<const h4 *>(zb + (2 * p + part) * 2048 + (16 * blk + col) * 32 + 8 * (q ^ (2 * p + part)));
                        eo[part] = __builtin_amdgcn_mfma_f32_16x16x16f16(a, di[part], (f4){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float v = fabsf(eo[0][r]) + fabsf(eo[1][r]);
                        top = max(top, __builtin_bit_cast(uint32_t, v));
                    }
                }
                const int64_t n = n8 + n2 + p;
                const int r = (int)(n & (K - 1));
                const double bound = (13.0 + (big[p] ? width : 0.0f)) / 2048.0 * sqrt((double)sq[p]) + 0.02;
                const bool may = !((double)__builtin_bit_cast(float, top) + bound < tau / row_scale(r, K)) || r == 0;
                if (n < n_row && __builtin_amdgcn_ballot_w64(may)) need |= 1u << (n2 + p);
            }
            wave_lds_sync();
        }
        int at = 0;
        if (lane == 0 && need) at = atomicAdd(n_list, __popc(need));
        at = __builtin_amdgcn_readfirstlane(at);
        if (lane < TEST_ROWS && n8 + lane < n_row) {
            if (need >> lane & 1u)
                list[at + __popc(need & ((1u << lane) - 1u))] = (int)(n8 + lane);
            else
                S[(n8 + lane) * 64 * B] = __builtin_nan("");
        }
    }
}

// The t-product of two of the listed Haar rows, or of all of them where there is no list (Eq. 19), the
// hard threshold |s| >= tau (Eq. 20) and, where a coefficient is kept, the inverse t-product (Eq. 21):
// U_hat_f^H P_hat_f V_hat_f per frequency and back with the factors swapped.  The coefficients never leave
// the registers; a row without kept coefficients stores only its mark.
template <int FB>
__global__ __launch_bounds__(256, FB == 1 ? 4 : FB == 0 ? 3 : 2) void band_rows_kernel(
    int B, int nb, int K, int64_t n_rows, const int *__restrict__ list, const int *__restrict__ n_list,
    const double *__restrict__ D, const double *__restrict__ Dinv, const double *__restrict__ frag_fwd,
    const double *__restrict__ frag_inv, double tau, double *__restrict__ S) {
    using T = BandTile<FB>;
    __shared__ double Z[T::PP * T::ZP];
    __shared__ double ops[T::N_OPS];
    __shared__ int kept[2][T::PP];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), p = wave & 1, half = wave >> 1;
    const int NF = B / 2 + 1, KS = (NF + 3) >> 2;
    int lane = tid & 63;
    double *z = Z + p * T::ZP;
    if (tid < 2 * T::PP) kept[tid / T::PP][tid % T::PP] = 0;
    if constexpr (T::OPS) {   // wave = (inverse, part)
        double a[T::KS];
        if (wave < 2)
            band_operand<FB, false>(D, B, nb, wave, 0, lane, a);
        else
            band_operand<FB, true>(Dinv, B, nb, wave - 2, 0, lane, a);
#pragma unroll
        for (int s = 0; s < T::KS; ++s) ops[(wave * T::KS + s) * 64 + lane] = a[s];
        if constexpr (FB == 0) {   // row 16 of both, zero beyond its 17 columns
            if (tid < 2 * 4 * T::KS) {
                const bool inv = tid >= 4 * T::KS;
                const int k = tid - (inv ? 4 * T::KS : 0), c = min(k, 16);
                const double d = inv ? Dinv[16 * nb + re_row(c, 32)] : D[re_row(16, 32) * nb + c];
                ops[4 * T::KS * 64 + tid] = k > 16 ? 0.0 : d;
            }
        }
    }
    __syncthreads();

    int par = 0;
    int raw[2][2][T::KS];   // the next row's sums
    int64_t next = 0;       // and its number
    const int64_t n_row = list ? (int64_t)*n_list : n_rows;
    auto load = [&](int64_t n0) {
        next = n0 + p < n_row ? n0 + p : n0;
        if (list) next = list[next];
        const int16_t *in = reinterpret_cast<const int16_t *>(S + next * 64 * B) +
                            2 * half * 2 * KS * 64 + 4 * (lane & 15) + (lane >> 4);
#pragma unroll
        for (int part = 0; part < 2; ++part)
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int s = 0; s < T::KS; ++s) raw[part][u][s] = in[((2 * u + part) * KS + min(s, KS - 1)) * 64];
    };
    if ((int64_t)blockIdx.x * T::PP < n_row) load((int64_t)blockIdx.x * T::PP);
    for (int64_t n0 = (int64_t)blockIdx.x * T::PP, n1; n0 < n_row; n0 = n1, par ^= 1) {
        asm volatile("" : "+v"(lane));   // addresses are made anew: kept over the loop they cost 70 registers
        n1 = n0 + (int64_t)gridDim.x * T::PP;
        const int q = lane >> 4, col = lane & 15;
        const int64_t n = next;
        const bool valid = n0 + p < n_row;
        double *slot = S + n * 64 * B;
        double x[2][2][T::KS];   // (even and odd part, block of 16 positions, k-step)
        {
            const double scale = row_scale((int)(n & (K - 1)), K);
#pragma unroll
            for (int part = 0; part < 2; ++part)
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int s = 0; s < T::KS; ++s) x[part][u][s] = s < KS ? (double)raw[part][u][s] * scale : 0.0;
        }
        double nx[8];
        band_slices_load(frag_fwd, nx, B, wave, lane);
        // the DFTs read and write only the wave's own positions of Z, the slices all of them
        band_dft<FB>(D, ops, nb, x, z, B, half, lane);
        __syncthreads();
        if (tid < T::PP) kept[par ^ 1][tid] = 0;   // read by all before this barrier, set after the next
        band_slices<FB>(frag_fwd, nx, Z, B, wave, lane);
        if (n1 < n_row) load(n1);
        __syncthreads();
        band_idft<FB>(Dinv, ops, nb, z, x, B, half, lane);
        bool any = false;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int s = 0; s < T::KS; ++s) {
                const int b = 4 * s + q;
                const bool k0 = b < NF && fabs(x[0][u][s]) >= tau;
                const bool k1 = b > 0 && 2 * b < B && fabs(x[1][u][s]) >= tau;
                const double y0 = k0 ? x[0][u][s] : 0.0, y1 = k1 ? x[1][u][s] : 0.0;
                x[0][u][s] = y0 + y1;
                x[1][u][s] = b > 0 && 2 * b < B ? y0 - y1 : 0.0;
                any |= k0 || k1;
            }
        if (__builtin_amdgcn_ballot_w64(any && valid) && lane == 0) kept[par][p] = 1;
        __syncthreads();
        const int mine = kept[par][p], either = kept[par][0] | kept[par][1];
        if (valid && !mine && half == 0 && lane == 0) slot[0] = __builtin_nan("");
        if (!either) continue;

        asm volatile("" : "+v"(lane));
        band_slices_load(frag_inv, nx, B, wave, lane);
        band_dft<FB>(D, ops, nb, x, z, B, half, lane);
        __syncthreads();
        band_slices<FB>(frag_inv, nx, Z, B, wave, lane);
        __syncthreads();
        if (!mine) continue;
        band_idft<FB>(Dinv, ops, nb, z, x, B, half, lane);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int s = 0; s < T::KS; ++s) {
                const int e = 32 * half + 16 * u + col;
                int b = 4 * s + q;
                if (b < NF) slot[64 * (b & ~7) + e * min(8, B - (b & ~7)) + (b & 7)] = x[0][u][s];
                if (b > 0 && 2 * b < B) {
                    b = B - b;
                    slot[64 * (b & ~7) + e * min(8, B - (b & ~7)) + (b & 7)] = x[1][u][s];
                }
            }
    }
}

// Inverse Haar transform of the groups and uniform aggregation sums (Algorithm 1).  One workgroup
// adds the 8 bands b8 .. b8 + 7 of the groups of a TR x TR tile of references in LDS, over the
// pixels their windows reach, and each sum goes to memory once: 126 million values in 129 us, bound by
// the LDS atomics, where an atomic in memory for each took most of 1,082 us.  Each wave takes
// lines of 8 positions of a group's patches: lane (position j, band).
struct BandAgg {
    int h, w, s, ny, nx, R;
    int TR, RH, RW;   // tile side and capacity (rows, columns) of its pixels
};

// A tile's groups go through one workgroup one after the other (16 groups of 32 members: 40 us), so tiles
// shrink where a pass has few of them: 27 x 36 x 5, K 32, 75 us for the call with tiles of 4 x 4 and 42
// with single references; 48 x 48 x 31, K 16, 82 and 68; 64 x 64 x 31, K 32, 136 and (2 x 2) 114.  At
// 256 workgroups instead of 64 smaller tiles add more to memory than they gain (64 x 64 x 31: 126).
constexpr int ADD_BLOCKS = 64;

template <int K>
__global__ __launch_bounds__(1024) void band_add_kernel(const BandAgg a, int B, const int32_t *__restrict__ idx,
                                                        const double *__restrict__ S, int64_t g0, int64_t ng, int ty0,
                                                        unsigned long long *__restrict__ acc, int *__restrict__ cnt) {
    extern __shared__ unsigned long long sums[];   // [RH][RW][8], then counts [RH][RW]
    int *counts = reinterpret_cast<int *>(sums + a.RH * a.RW * 8);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles_x = (a.nx + a.TR - 1) / a.TR, ty = ty0 + (int)blockIdx.x / tiles_x, tx = (int)blockIdx.x % tiles_x;
    const int b8 = 8 * blockIdx.y, wd = min(8, B - b8), j = lane >> 3, b = lane & 7;
    const int iy0 = ty * a.TR, ix0 = tx * a.TR, th = min(a.TR, a.ny - iy0), tw = min(a.TR, a.nx - ix0);
    const int y0 = max(0, ref_pos(iy0, a.ny, a.h, a.s) - a.R), x0 = max(0, ref_pos(ix0, a.nx, a.w, a.s) - a.R);
    const int rh = min(a.h, ref_pos(iy0 + th - 1, a.ny, a.h, a.s) + a.R + PS) - y0;
    const int rw = min(a.w, ref_pos(ix0 + tw - 1, a.nx, a.w, a.s) + a.R + PS) - x0;
    for (int i = tid; i < rh * rw * 8; i += 1024) sums[i] = 0;
    for (int i = tid; i < rh * rw; i += 1024) counts[i] = 0;
    __syncthreads();

    const int n_line = th * tw * 8, per = (n_line + 15) >> 4;
    int have = -1, off = 0;
    uint32_t rows = 0;
    const double *base = nullptr;
    for (int l = wave * per; l < min(n_line, (wave + 1) * per); ++l) {
        const int gi = l >> 3, i = l & 7;
        const int64_t g = (int64_t)(iy0 + gi / tw) * a.nx + ix0 + gi % tw - g0;
        if (g < 0 || g >= ng) continue;
        if (gi != have) {
            have = gi;
            base = S + g * K * 64 * B;
            const int m = lane & (K - 1);
            const int32_t lin = idx[g * K + m];
            off = (lin / a.w - y0) * rw + lin % a.w - x0;
            const double mark = base[(int64_t)m * 64 * B];
            rows = (uint32_t)__builtin_amdgcn_ballot_w64(lane < K && mark == mark);
        }
        const double *src = base + 64 * b8 + (8 * i + j) * wd + min(b, wd - 1);
        const int at = (i * rw + j) * 8 + b;
        const bool in = b < wd;
        constexpr double MAGIC = 6755399441055744.0 / (1 << BFS);   // 1.5 2^52 units: rounds to nearest, ties to even
        const long long MBITS = __builtin_bit_cast(long long, MAGIC);
        auto units = [&](double v) {
            return (unsigned long long)(__builtin_bit_cast(long long, fmin(fmax(v, -1024.0), 1024.0) + MAGIC) - MBITS);
        };
        if (rows <= 1u) {   // every member gets the same estimate
            double m = rows ? *src : 0.0;
            m = in ? m : 0.0;   // lanes past the last band add nothing to sums that nobody reads
#pragma unroll
            for (int h = 1; h < K; h <<= 1) m *= R2;
            const unsigned long long u = units(m);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int o = __builtin_amdgcn_readlane(off, k) * 8;   // with every lane active
                atomicAdd(sums + o + at, u);
            }
        } else {
            double v[K];
#pragma unroll
            for (int k = 0; k < K; ++k) v[k] = rows >> k & 1u ? src[(int64_t)k * 64 * B] : 0.0;
#pragma unroll
            for (int k = 0; k < K; ++k) v[k] = in ? v[k] : 0.0;
#pragma unroll
            for (int h = K / 2; h >= 1; h >>= 1)
#pragma unroll
                for (int k = 0; k < K; k += 2 * h) {
                    const double c = v[k], d = v[k + h];
                    v[k] = (c + d) * R2;
                    v[k + h] = (c - d) * R2;
                }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int o = __builtin_amdgcn_readlane(off, k) * 8;
                atomicAdd(sums + o + at, units(v[k]));
            }
        }
        if (b8 == 0) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int o = __builtin_amdgcn_readlane(off, k);
                if (b == 0) atomicAdd(counts + o + i * rw + j, 1);
            }
        }
    }
    __syncthreads();
    for (int t = tid; t < rh * rw * 8; t += 1024) {
        const unsigned long long v = sums[t];
        const int px = t >> 3;
        if (v) atomicAdd(acc + ((int64_t)(y0 + px / rw) * a.w + x0 + px % rw) * B + b8 + (t & 7), v);
    }
    if (b8 == 0)
        for (int t = tid; t < rh * rw; t += 1024)
            if (counts[t]) atomicAdd(cnt + (int64_t)(y0 + t / rw) * a.w + x0 + t % rw, counts[t]);
}

__global__ void normalize_kernel(const unsigned long long *__restrict__ acc, const int *__restrict__ cnt,
                                 const uint8_t *__restrict__ cube, int64_t stride, int h, int w, int B,
                                 float *__restrict__ out, int64_t out_stride) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= (int64_t)h * w * B) return;
    const int b = (int)(t % B);
    const int64_t pix = t / B;
    const int y = (int)(pix / w), x = (int)(pix % w);
    const int n = cnt[pix];
    out[(int64_t)y * out_stride + (int64_t)x * B + b] =
        n > 0 ? (float)((double)(long long)acc[t] / ((double)n * (double)(1 << BFS)))
              : (float)cube[(int64_t)y * stride + (int64_t)x * B + b];
}

// out(y, x, b) = alt(y, x, b) for the bands with sel[b] != 0.
__global__ void select_bands_kernel(const float *__restrict__ alt, int64_t alt_stride, const uint8_t *__restrict__ sel,
                                    int h, int w, int B, float *__restrict__ out, int64_t out_stride) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= (int64_t)h * w * B) return;
    const int b = (int)(t % B);
    if (!sel[b]) return;
    const int64_t pix = t / B;
    const int y = (int)(pix / w), x = (int)(pix % w);
    out[(int64_t)y * out_stride + (int64_t)x * B + b] = alt[(int64_t)y * alt_stride + (int64_t)x * B + b];
}

unsigned nb(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

template <int K>
hipError_t launch_pass(const BandMaps &bm, const uint8_t *cube, int64_t stride, int B, const int32_t *idx, int64_t g0,
                       int64_t ng, double tau, const BandAgg &a, double *S, int *n_list, unsigned long long *acc, int *cnt,
                       hipStream_t st) {
    const auto haar = B == 2 ? band_haar_kernel<K, true> : band_haar_kernel<K, false>;
    hipLaunchKernelGGL(haar, dim3((unsigned)ng), dim3(256), 0, st, cube, stride, a.w, B, idx, S);
    const auto rows = B <= 31   ? band_rows_kernel<1>
                      : B == 32 ? band_rows_kernel<0>
                      : B <= 63 ? band_rows_kernel<2>
                                : band_rows_kernel<3>;
    // workgroups that go through the rows: three per CU, then four (FB = 1), three (0) or two are resident
    int *list = n_list + 1;
    const bool test = B <= 31 && ng * K > test_min_rows(B);
    if (test) {
        if (g0 > 0) {   // zero before the first pass
            const hipError_t e = launch_zero(n_list, sizeof(int), st);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(band_test_kernel, dim3(std::min<unsigned>(nb(ng * K, 4 * TEST_ROWS), 768)), dim3(256), 0, st, B,
                           bm.nb, K, ng * K, bm.D, bm.frag_fwd, tau, S, list, n_list);
    }
    const unsigned grid = std::min<unsigned>(nb(ng * K, BandTile<1>::PP), B <= 31 ? 1024 : B == 32 ? 768 : 512);
    hipLaunchKernelGGL(rows, dim3(grid), dim3(256), 0, st, B, bm.nb, K, ng * K, test ? list : nullptr, n_list, bm.D,
                       bm.Dinv, bm.frag_fwd, bm.frag_inv, tau, S);
    const int tiles_x = (a.nx + a.TR - 1) / a.TR;
    const int ty0 = (int)(g0 / a.nx) / a.TR, ty1 = (int)((g0 + ng - 1) / a.nx) / a.TR;
    const int lds = a.RH * a.RW * (8 * 8 + 4);
    const hipError_t e = prepare_dynamic_lds(reinterpret_cast<const void *>(&band_add_kernel<K>), lds, 0);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(band_add_kernel<K>, dim3((unsigned)((ty1 - ty0 + 1) * tiles_x), nb(B, 8)), dim3(1024), lds, st, a,
                       B, idx, S, g0, ng, ty0, acc, cnt);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_select_bands(const float *alt, int64_t alt_stride, const uint8_t *sel, int h, int w, int B,
                               float *out, int64_t out_stride, hipStream_t st) {
    hipLaunchKernelGGL(select_bands_kernel, dim3(nb((int64_t)h * w * B, 256)), dim3(256), 0, st, alt, alt_stride, sel,
                       h, w, B, out, out_stride);
    return hipGetLastError();
}

hipError_t launch_band_guide(const uint8_t *cube, int64_t stride, int h, int w, int B, uint8_t *guide,
                             hipStream_t st) {
    hipLaunchKernelGGL(guide_kernel, dim3(nb((int64_t)h * w, 256)), dim3(256), 0, st, cube, stride, h, w, B, guide);
    return hipGetLastError();
}

// Groups per pass of the filter: the FP64 patch matrix S stays below cap bytes, at least one group.
int64_t band_chunk_groups(int B, int K, int64_t n_group, int64_t cap) {
    const int64_t per = (int64_t)K * 64 * B * (int64_t)sizeof(double);
    return std::max<int64_t>(1, std::min<int64_t>(n_group, cap / per));
}

size_t band_ws_bytes(int h, int w, int B, int K, int64_t n_group, int64_t cap) {
    const int64_t n_patch = band_chunk_groups(B, K, n_group, cap) * K;
    const size_t mat = sizeof(double) * (size_t)n_patch * 64 * B;
    return ((mat + 255) & ~(size_t)255) + (((size_t)h * w * B * 8 + 255) & ~(size_t)255) +
           (((size_t)h * w * 4 + 255) & ~(size_t)255) + (((size_t)(n_patch + 1) * 4 + 255) & ~(size_t)255);
}

// Per pass: the Haar sums of the groups' pixels, the t-product, threshold and inverse t-product of
// their rows, and the inverse Haar transform with aggregation; then normalisation.
hipError_t launch_band_filter(const BandMaps &bm, const uint8_t *cube, int64_t stride, int h, int w, int B,
                              const int32_t *idx, int s, int W, int K, double tau, int64_t cap, void *ws, float *out,
                              int64_t out_stride, hipStream_t st) {
    if (bm.nb != band_nb(B)) return hipErrorInvalidValue;
    BandAgg a = {h, w, s, ref_count(h, s), ref_count(w, s), (W - 1) / 2, 4, 0, 0};
    const int64_t n_group = (int64_t)a.ny * a.nx, chunk = band_chunk_groups(B, K, n_group, cap);
    // the largest tile of references whose pixels fit 128 KB of LDS (one reference takes at most 98) and
    // of which a pass has ADD_BLOCKS
    for (;; a.TR >>= 1) {
        a.RH = (int)std::min<int64_t>(h, (int64_t)(a.TR - 1) * s + 2 * a.R + PS);
        a.RW = (int)std::min<int64_t>(w, (int64_t)(a.TR - 1) * s + 2 * a.R + PS);
        if (a.TR == 1 || ((int64_t)a.RH * a.RW * (8 * 8 + 4) <= 128 * 1024 &&
                          std::min(n_group, chunk) * nb(B, 8) >= (int64_t)ADD_BLOCKS * a.TR * a.TR))
            break;
    }
    const size_t mat = ((sizeof(double) * (size_t)(chunk * K) * 64 * B) + 255) & ~(size_t)255;
    double *S = (double *)ws;
    unsigned long long *acc = (unsigned long long *)((char *)ws + mat);
    int *cnt = (int *)((char *)acc + (((size_t)h * w * B * 8 + 255) & ~(size_t)255));
    int *n_list = (int *)((char *)cnt + (((size_t)h * w * 4 + 255) & ~(size_t)255));   // number of listed rows, then these
    hipError_t e;
    if ((e = launch_zero(acc, (size_t)((char *)(n_list + 1) - (char *)acc), st)) != hipSuccess) return e;
    for (int64_t g0 = 0; g0 < n_group; g0 += chunk) {
        const int64_t ng = std::min<int64_t>(chunk, n_group - g0);
        const int32_t *ix = idx + g0 * K;
        switch (K) {
            case 4: e = launch_pass<4>(bm, cube, stride, B, ix, g0, ng, tau, a, S, n_list, acc, cnt, st); break;
            case 8: e = launch_pass<8>(bm, cube, stride, B, ix, g0, ng, tau, a, S, n_list, acc, cnt, st); break;
            case 16: e = launch_pass<16>(bm, cube, stride, B, ix, g0, ng, tau, a, S, n_list, acc, cnt, st); break;
            case 32: e = launch_pass<32>(bm, cube, stride, B, ix, g0, ng, tau, a, S, n_list, acc, cnt, st); break;
            default: return hipErrorInvalidValue;
        }
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(normalize_kernel, dim3(nb((int64_t)h * w * B, 256)), dim3(256), 0, st, acc, cnt, cube, stride, h,
                       w, B, out, out_stride);
    return hipGetLastError();
}

}  // namespace htsvd
