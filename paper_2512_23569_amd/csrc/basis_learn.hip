// Channel Gram sums of all reference patches of one image: the device half of learning the
// t-SVD basis pair from the image itself (Sec. III-B, Eq. 10-11).
//
// Over the reference grid (rows ys, columns xs, Algorithm 1) the row sums
//   G_row[a][b][i][k] = sum_{y in ys, x in xs} sum_j X(y+i, x+j, a) X(y+k, x+j, b)
// regroup by image column: for a fixed y the pair (x, j) only enters through col = x + j, so
//   G_row = sum_{y in ys} sum_col m(col) v v^T,   v = X(y..y+7, col, :),
// with m(col) the number of reference columns whose patch covers col.  The column sums are the
// same with the roles of rows and columns swapped (horizontal 8-vectors at the reference
// columns, weighted by the number of reference rows covering the pixel row).  Every entry is an
// exact integer (below 2^50 for any image the library accepts), accumulated in 32-bit per staged
// chunk and in 64-bit across chunks.
#include "common.h"

namespace htsvd {

namespace {

constexpr int GR_THREADS = 256;
constexpr int GR_CHUNK = 256;    // vectors staged per step, one per thread
constexpr int GR_MAX_BLOCKS = 1024;

// Reference positions along a side of n pixels (n_ref of them) whose patch covers pixel pos:
// regular positions i*s for i <= n_ref - 2, plus the last one at n - 8.
__device__ inline int cover_count(int pos, int n, int n_ref, int s) {
    int cnt = 0;
    if (n_ref >= 2) {
        const int lo = pos >= PS - 1 ? (pos - (PS - 1) + s - 1) / s : 0;
        const int hi = min(n_ref - 2, pos / s);
        cnt = max(0, hi - lo + 1);
    }
    return cnt + (pos >= n - PS ? 1 : 0);
}

// Thread tasks: an entry row r = ch*8 + i (A = 8c of them) times a block of 4 entry columns
// starting at 4*bb, for bb >= r/4 (the other blocks follow by symmetry).  T = 4c(2c+1) tasks.
template <int C>
__global__ __launch_bounds__(GR_THREADS) void gram_kernel(const uint8_t *__restrict__ img, int64_t stride, int h,
                                                          int w, int s, int ny, int nx,
                                                          unsigned long long *__restrict__ out) {
    constexpr int A = 8 * C, NBB = 2 * C, T = 4 * C * (2 * C + 1), GRP = GR_THREADS / T;
    __shared__ __align__(16) uint32_t sv[GR_CHUNK * A];    // the staged vectors
    __shared__ __align__(16) uint32_t smv[GR_CHUNK * A];   // the same, times their weight
    __shared__ unsigned long long sred[GRP * T * 4];
    const int g = blockIdx.y;   // 0: row sums, 1: column sums
    const int64_t n_vec = g == 0 ? (int64_t)ny * w : (int64_t)nx * h;
    const int64_t n_chunks = (n_vec + GR_CHUNK - 1) / GR_CHUNK;
    const int tid = threadIdx.x;
    const int grp = tid / T, task = tid % T;
    const bool active = grp < GRP;
    int r = 0, bb = 0;
    {
        int rem = task;
        while (rem >= NBB - r / 4) {
            rem -= NBB - r / 4;
            ++r;
        }
        bb = r / 4 + rem;
    }
    unsigned long long tot0 = 0, tot1 = 0, tot2 = 0, tot3 = 0;
    for (int64_t ch = blockIdx.x; ch < n_chunks; ch += gridDim.x) {
        const int64_t q0 = ch * GR_CHUNK;
        const int nv = (int)min<int64_t>(GR_CHUNK, n_vec - q0);
        if (tid < nv) {
            const int64_t q = q0 + tid;
            const uint8_t *p;
            int64_t step;
            uint32_t m;
            if (g == 0) {
                const int iy = (int)(q / w), col = (int)(q % w);
                p = img + (int64_t)ref_pos(iy, ny, h, s) * stride + (int64_t)col * C;
                step = stride;
                m = cover_count(col, w, nx, s);
            } else {
                const int row = (int)(q / nx), ix = (int)(q % nx);
                p = img + (int64_t)row * stride + (int64_t)ref_pos(ix, nx, w, s) * C;
                step = C;
                m = cover_count(row, h, ny, s);
            }
#pragma unroll
            for (int i = 0; i < PS; ++i)
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const uint32_t v = p[i * step + c];
                    sv[tid * A + c * PS + i] = v;
                    smv[tid * A + c * PS + i] = __umul24(m, v);
                }
        }
        __syncthreads();
        if (active) {
            // At most 256/GRP vectors of weight <= 9 per chunk: every partial sum stays below 2^32.
            // Factors below 2^24 (weighted value <= 9 * 255, value <= 255): 24-bit multiply-adds.
            uint32_t a0 = 0, a1 = 0, a2 = 0, a3 = 0;
            int v = grp;
            for (; v + 3 * GRP < nv; v += 4 * GRP) {
                uint32_t x[4];
                uint4 y[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    x[u] = smv[(v + u * GRP) * A + r];
                    y[u] = *reinterpret_cast<const uint4 *>(&sv[(v + u * GRP) * A + 4 * bb]);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    a0 = __umul24(x[u], y[u].x) + a0;
                    a1 = __umul24(x[u], y[u].y) + a1;
                    a2 = __umul24(x[u], y[u].z) + a2;
                    a3 = __umul24(x[u], y[u].w) + a3;
                }
            }
            for (; v < nv; v += GRP) {
                const uint32_t x = smv[v * A + r];
                const uint4 y = *reinterpret_cast<const uint4 *>(&sv[v * A + 4 * bb]);
                a0 = __umul24(x, y.x) + a0;
                a1 = __umul24(x, y.y) + a1;
                a2 = __umul24(x, y.z) + a2;
                a3 = __umul24(x, y.w) + a3;
            }
            tot0 += a0;
            tot1 += a1;
            tot2 += a2;
            tot3 += a3;
        }
        __syncthreads();
    }
    if (active) {
        unsigned long long *d = sred + (grp * T + task) * 4;
        d[0] = tot0;
        d[1] = tot1;
        d[2] = tot2;
        d[3] = tot3;
    }
    __syncthreads();
    // One atomic per entry and block; the mirrored entry (b, r) is added too where no task of
    // its own covers it (column block below its row's block).
    for (int e = tid; e < T * 4; e += GR_THREADS) {
        unsigned long long sum = 0;
        for (int k = 0; k < GRP; ++k) sum += sred[k * T * 4 + e];
        if (sum == 0) continue;
        int rr = 0, rem = e / 4;
        while (rem >= NBB - rr / 4) {
            rem -= NBB - rr / 4;
            ++rr;
        }
        const int b = 4 * (rr / 4 + rem) + (e & 3);
        // entry (rr, b) = (ch1*8 + i, ch2*8 + k) -> out[g][ch1][ch2][i][k]
        unsigned long long *og = out + (size_t)g * C * C * 64;
        atomicAdd(og + ((rr / PS) * C + b / PS) * 64 + (rr % PS) * PS + b % PS, sum);
        if (b / 4 != rr / 4) atomicAdd(og + ((b / PS) * C + rr / PS) * 64 + (b % PS) * PS + rr % PS, sum);
    }
}

// The same sums for a runtime channel count C (hyperspectral bands, up to 64), taken before the
// regrouping by column: the row sums over the vectors v = X(y..y+7, x+j, :) of every reference
// (y, x) and offset j, the column sums over X(y+i, x..x+7, :), without weights.  A block owns a
// 64 x 64 tile pair (ta <= tb) of the A x A matrix (A = 8C) and a slice of the vectors.  It stages
// 64 vectors at a time in LDS, entry by entry (8 bands of 4 vectors per thread, the bytes transposed
// in registers), as v - 128 so that v_mfma_i32_16x16x64_i8 takes them: a wave's product of 16
// entries with all 64 over the 64 vectors is four instructions, and five more with ones in place of
// one side give the sums that undo the shift,
//   sum v v' = sum (v-128)(v'-128) + 128 (sum (v-128) + sum (v'-128)) + 128^2 n.
// The products are a small part of it: it is bound by the latency of the staging loads (the next
// chunk's are issued ahead) and by the 64-bit atomics at its end, 0.13 us per block.  63 x 63
// references, 31 bands: 75 us with 256 blocks, 89 with 512, 147 with 1,024 (212 us with byte loads and
// v_dot4); 126 x 126 references: 259, 186 and 242 us (434).  Four teams of waves per block that add
// their sums in LDS before the atomics were slower (107 us with 256).  32-bit partials hold GB_MAX chunks
// (64 128^2 each); the blocks add 64-bit totals with integer atomics (exact, so in any order).
constexpr int GB_VEC = 64;            // vectors per staged chunk
constexpr int GB_MAX = 1024;          // chunks per block
constexpr int GB_PITCH = 80;          // bytes per staged entry (64 and 4 banks)

typedef int gv4i __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void gram_bands_kernel(const uint8_t *__restrict__ img, int64_t stride, int h,
                                                         int w, int C, int s, int ny, int nx,
                                                         unsigned long long *__restrict__ out, int z0, int zs) {
    __shared__ __align__(16) unsigned char P[2][2][64 * GB_PITCH];   // (buffer, tile side)
    const int A = 8 * C;
    const int g = blockIdx.y;
    // tile pair (ta, tb), ta <= tb, row-major over the upper triangle of the tile grid
    const int nt = (A + 63) / 64;
    int ta = 0, rem = blockIdx.x;
    while (rem >= nt - ta) {
        rem -= nt - ta;
        ++ta;
    }
    const int tb = ta + rem;
    const int64_t n_ref = (int64_t)ny * nx;
    const int64_t n_chunks = (n_ref * 8 + GB_VEC - 1) / GB_VEC;
    const int z = z0 + (int)blockIdx.z;   // slice of zs
    const int64_t c_begin = n_chunks * z / zs, c_end = n_chunks * (z + 1) / zs;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // staging task: 4 vectors 4k .. 4k + 3 (of one reference) at entry offset e, the 8 bands of its side
    const int k = tid & 15, e = tid >> 4 & 7, side = tid >> 7;
    const int b0 = 8 * (side ? tb : ta), n_band = min(8, C - b0);
    uint32_t lo[4], hi[4];
    auto load = [&](int64_t ck) {
        const int64_t r = ck * 8 + (k >> 1);
        if (r < n_ref) {   // past the slice: loaded, not used
            const int iy = (int)((uint32_t)r / (uint32_t)nx), ix = (int)r - iy * nx, off = 4 * (k & 1);
            const int y = ref_pos(iy, ny, h, s), x = ref_pos(ix, nx, w, s);
            // g = 0: entry e is the row offset, the 4 vectors are columns x+off..x+off+3;
            // g = 1: entry e is the column offset, the 4 vectors are rows y+off..y+off+3
            const uint8_t *px = g == 0 ? img + (int64_t)(y + e) * stride + (int64_t)(x + off) * C
                                       : img + (int64_t)(y + off) * stride + (int64_t)(x + e) * C;
            const int64_t step = g == 0 ? C : stride;
            if (C >= 8) {   // the last bands of a tube: its last 8 bytes, shifted
                const int at = b0 + n_band - 8, sh = 8 * (8 - n_band);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    uint64_t t;
                    __builtin_memcpy(&t, px + v * step + at, 8);
                    t = (t >> sh) ^ 0x8080808080808080ull;
                    lo[v] = (uint32_t)t;
                    hi[v] = (uint32_t)(t >> 32);
                }
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    uint64_t t = 0;
                    for (int b = 0; b < C; ++b) t |= (uint64_t)px[v * step + b] << (8 * b);
                    t ^= 0x8080808080808080ull;
                    lo[v] = (uint32_t)t;
                    hi[v] = (uint32_t)(t >> 32);
                }
            }
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) lo[v] = hi[v] = 0;   // adds nothing
        }
    };
    // bytes of 4 vectors at one band, for 4 bands: word b of the entry's rows b*8 + e
    auto store4 = [&](const uint32_t (&v)[4], unsigned char *d) {
        const uint32_t t0 = __builtin_amdgcn_perm(v[1], v[0], 0x05010400u), t1 = __builtin_amdgcn_perm(v[3], v[2], 0x05010400u);
        const uint32_t t2 = __builtin_amdgcn_perm(v[1], v[0], 0x07030602u), t3 = __builtin_amdgcn_perm(v[3], v[2], 0x07030602u);
        *reinterpret_cast<uint32_t *>(d) = __builtin_amdgcn_perm(t1, t0, 0x05040100u);
        *reinterpret_cast<uint32_t *>(d + 8 * GB_PITCH) = __builtin_amdgcn_perm(t1, t0, 0x07060302u);
        *reinterpret_cast<uint32_t *>(d + 16 * GB_PITCH) = __builtin_amdgcn_perm(t3, t2, 0x05040100u);
        *reinterpret_cast<uint32_t *>(d + 24 * GB_PITCH) = __builtin_amdgcn_perm(t3, t2, 0x07060302u);
    };
    const int col = lane & 15, q = lane >> 4;
    const gv4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
    gv4i acc[4] = {}, sum_b[4] = {}, sum_a = {};
    load(c_begin);
    for (int64_t ck = c_begin; ck < c_end; ++ck) {
        unsigned char(*buf)[64 * GB_PITCH] = P[(ck - c_begin) & 1];
        store4(lo, buf[side] + e * GB_PITCH + 4 * k);
        store4(hi, buf[side] + (32 + e) * GB_PITCH + 4 * k);
        load(ck + 1);
        __syncthreads();   // the other buffer was read before the barrier of the chunk between
        const gv4i a = *reinterpret_cast<const gv4i *>(buf[0] + (16 * wave + col) * GB_PITCH + 16 * q);
        sum_a = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, ones, sum_a, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const gv4i b = *reinterpret_cast<const gv4i *>(buf[1] + (16 * j + col) * GB_PITCH + 16 * q);
            acc[j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, acc[j], 0, 0, 0);
            sum_b[j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ones, b, sum_b[j], 0, 0, 0);
        }
    }
    const int64_t n = min(n_ref * 8, c_end * GB_VEC) - c_begin * GB_VEC;
    if (n <= 0) return;
    unsigned long long *og = out + (size_t)g * C * C * 64;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int x = ta * 64 + 16 * wave + 4 * q + r, y = tb * 64 + 16 * j + col;
            if (x >= A || y >= A) continue;
            const unsigned long long t =
                (unsigned long long)((int64_t)acc[j][r] + 128 * ((int64_t)sum_a[r] + sum_b[j][r]) + 16384 * n);
            if (t == 0) continue;
            // staged entry x holds row or column offset x mod 8 of band x / 8
            atomicAdd(og + ((x / 8) * C + y / 8) * 64 + (x % 8) * 8 + y % 8, t);
            if (ta != tb) atomicAdd(og + ((y / 8) * C + x / 8) * 64 + (y % 8) * 8 + x % 8, t);
        }
}

// ---- from the Gram sums of a cube to its basis, on the device (hyperspectral path) ----
// The channel sums enter the slice covariances only through d = a - b mod c, so they are first added
// over the diagonals, exactly; then every slice and side is one 8 x 8 Hermitian eigenproblem for
// one wavefront, and the inverse channel DFT and the operands of the band filter follow from the
// vectors.  On the host the same work took 3.0 ms for 31 bands (a covariance sum over all 961
// channel pairs, cosines inside the loops, 32 eigenproblems one after another), here 80 us (the eigenproblems 57).

// fold[(g*c + d)*64 + e] = sum_{a - b = d mod c} gram[((g*c + a)*c + b)*64 + e].
__global__ __launch_bounds__(64) void gram_fold_kernel(const int64_t *__restrict__ gram, int c,
                                                       int64_t *__restrict__ fold) {
    const int g = blockIdx.x / c, d = blockIdx.x % c, e = threadIdx.x;
    int64_t v = 0;
    for (int a = 0; a < c; ++a) {
        const int b = a >= d ? a - d : a - d + c;
        v += gram[((int64_t)(g * c + a) * c + b) * 64 + e];
    }
    fold[(int64_t)blockIdx.x * 64 + e] = v;
}

struct cd {
    double re, im;
};
__device__ inline cd mul(cd a, cd b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }

// Eigenvectors of slice f (block f*2 + g; g = 0: C_row -> U, 1: C_col -> V) into vec[(f*2 + g)*64 + i*8 + j]
// (column j: the j-th largest eigenvalue, the entry of largest modulus real and positive).  Jacobi's
// method with the four disjoint rotations of a round at once (lane = entry (i, k); a tournament of
// 7 rounds meets every pair), each with a complex rotation: a unit phase makes the pivot real, a
// plane rotation removes it.
__global__ __launch_bounds__(64) void band_evd_kernel(const int64_t *__restrict__ fold, int c, cd *__restrict__ vec) {
    __shared__ cd A[64], V[64], W[64];
    __shared__ double ev[8];
    const int f = blockIdx.x >> 1, g = blockIdx.x & 1, lane = threadIdx.x, i = lane >> 3, k = lane & 7;
    {
        // C_row = sum_d w^(f d) fold_d, C_col the conjugate factors, w = exp(-2 pi i / c)
        double re = 0.0, im = 0.0;
        for (int d = 0; d < c; ++d) {
            double sn, cs;
            sincospi(2.0 * (double)((f * d) % c) / c, &sn, &cs);
            const double v = (double)fold[((int64_t)g * c + d) * 64 + lane];
            re += v * cs;
            im += (g == 0 ? -v : v) * sn;
        }
        W[lane] = {re, im};
        __syncthreads();
        const cd t = W[k * 8 + i];
        A[lane] = {0.5 * (re + t.re), i == k ? 0.0 : 0.5 * (im - t.im)};
        V[lane] = {i == k ? 1.0 : 0.0, 0.0};
        __syncthreads();
    }
    for (int sweep = 0; sweep < 100; ++sweep) {
        const cd own = A[lane];
        if (!__ballot(i < k && (own.re != 0.0 || own.im != 0.0))) break;
        for (int r = 0; r < 7; ++r) {
            auto partner = [&](int x) { return x == 7 ? r : (x == r ? 7 : (2 * r - x + 7) % 7); };
            // rotation of the pair that holds x: J[p][p] = co, J[p][q] = sn, J[q][p] = -sn conj(e),
            // J[q][q] = co conj(e)
            struct Rot {
                double co, sn;
                cd e;
                int p, q;
            };
            auto rotation = [&](int x) {
                const int y = partner(x);
                Rot t;
                t.p = min(x, y);
                t.q = max(x, y);
                const cd z = A[t.p * 8 + t.q];
                const double app = A[t.p * 9].re, aqq = A[t.q * 9].re;
                const double m = sqrt(z.re * z.re + z.im * z.im);
                // past the first sweeps a pivot below the last bit of both diagonal entries is
                // dropped instead of rotated (the usual termination of the method)
                const bool drop = m == 0.0 || (sweep > 3 && fabs(app) + 100.0 * m == fabs(app) &&
                                               fabs(aqq) + 100.0 * m == fabs(aqq));
                if (drop) {
                    t.co = 1.0;
                    t.sn = 0.0;
                    t.e = {1.0, 0.0};
                } else {
                    t.e = {z.re / m, z.im / m};
                    const double theta = (aqq - app) / (2.0 * m);
                    double tn = 1.0 / (fabs(theta) + sqrt(1.0 + theta * theta));
                    if (theta < 0.0) tn = -tn;
                    t.co = 1.0 / sqrt(1.0 + tn * tn);
                    t.sn = tn * t.co;
                }
                return t;
            };
            const Rot rk = rotation(k), ri = rotation(i);
            // column k of J, and the conjugate column i: factors of the entries p and q of the pair
            const cd kp = k == rk.p ? cd{rk.co, 0.0} : cd{rk.sn, 0.0};
            const cd kq = k == rk.p ? cd{-rk.sn * rk.e.re, rk.sn * rk.e.im} : cd{rk.co * rk.e.re, -rk.co * rk.e.im};
            const cd ip = i == ri.p ? cd{ri.co, 0.0} : cd{ri.sn, 0.0};
            const cd iq = i == ri.p ? cd{-ri.sn * ri.e.re, -ri.sn * ri.e.im} : cd{ri.co * ri.e.re, ri.co * ri.e.im};
            auto column = [&](const cd *M, int row) {
                const cd x = mul(M[row * 8 + rk.p], kp), y = mul(M[row * 8 + rk.q], kq);
                return cd{x.re + y.re, x.im + y.im};
            };
            const cd x = mul(ip, column(A, ri.p)), y = mul(iq, column(A, ri.q));
            cd a = {x.re + y.re, i == k ? 0.0 : x.im + y.im};
            if (k == partner(i)) a = {0.0, 0.0};
            const cd v = column(V, i);
            __syncthreads();
            A[lane] = a;
            V[lane] = v;
            __syncthreads();
        }
    }
    if (i == 0) ev[k] = A[k * 9].re;
    __syncthreads();
    int rank = 0;   // place of column k by descending eigenvalue, equal ones in order
    for (int j = 0; j < 8; ++j) rank += ev[j] > ev[k] || (ev[j] == ev[k] && j < k);
    int kmax = 0;
    double amax = -1.0;
    for (int j = 0; j < 8; ++j) {
        const cd v = V[j * 8 + k];
        const double m = sqrt(v.re * v.re + v.im * v.im);
        if (m > amax) {
            amax = m;
            kmax = j;
        }
    }
    const cd top = V[kmax * 8 + k], ph = amax > 0.0 ? cd{top.re / amax, -top.im / amax} : cd{1.0, 0.0};
    vec[(int64_t)blockIdx.x * 64 + i * 8 + rank] = i == kmax ? cd{amax, 0.0} : mul(V[lane], ph);
}

// T(k) = (1/c) sum_f T_hat^(f) exp(2 pi i f k / c) with T_hat^(c-f) = conj T_hat^(f): band k = blockIdx.x of
// U (threads 0 .. 63) and V into uv[(side*c + k)*64 + e].
__global__ __launch_bounds__(128) void band_basis_kernel(const cd *__restrict__ vec, int c, double *__restrict__ uv) {
    const int k = blockIdx.x, g = threadIdx.x >> 6, e = threadIdx.x & 63;
    double acc = 0.0;
    for (int f = 0; f <= c / 2; ++f) {
        double sn, cs;
        sincospi(2.0 * (double)((f * k) % c) / c, &sn, &cs);
        const cd v = vec[(f * 2 + g) * 64 + e];
        const double re = v.re * cs - v.im * sn;
        acc += f == 0 || 2 * f == c ? re : 2.0 * re;
    }
    uv[(int64_t)(g * c + k) * 64 + e] = acc / c;
}

// The band filter's maps (BandMaps): blocks f < NF: the slice products' operands of frequency f, both
// directions; block NF: the channel DFT D and its inverse.  Slice products: forward T = L P with
// L(a, b) = conj(U(b, a)), then Y = T R with R = V; inverse L = U, R(a, b) = conj(V(b, a)).  Real
// embeddings: L as [[Lr, -Li], [Li, Lr]] acting on [Pr; Pi], R as [[Rr, Ri], [-Ri, Rr]] acting on
// [Tr | Ti] from the right; operand lanes of v_mfma_f64_16x16x4f64: A(m, k) in lane m + 16 (k mod 4),
// B(k, n) in lane n + 16 (k mod 4).
__global__ __launch_bounds__(256) void band_maps_kernel(const cd *__restrict__ vec, int c, int nb,
                                                        double *__restrict__ maps) {
    const int NF = c / 2 + 1, f = blockIdx.x;
    double *D = maps, *Dinv = maps + nb * nb;
    if (f == NF) {
        for (int e = threadIdx.x; e < nb * nb; e += 256) {
            const int row = e / nb, b = e % nb;   // D[row][b] and Dinv[b][row]
            double d = 0.0, di = 0.0;
            if (row < c && b < c) {
                const int fr = (row + 1) / 2;
                double sn, cs;
                sincospi(2.0 * (double)((fr * b) % c) / c, &sn, &cs);
                const bool real = row == 0 || 2 * fr == c;
                d = real || (row & 1) ? cs : -sn;
                di = (real ? 1.0 : 2.0) * d / c;
            }
            D[row * nb + b] = d;
            Dinv[b * nb + row] = di;
        }
        return;
    }
    const cd *U = vec + (f * 2) * 64, *V = U + 64;
    const int st = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int m = lane & 15, k = 4 * st + (lane >> 4), rm = m >> 3, rk = k >> 3;
    for (int dir = 0; dir < 2; ++dir) {
        double *fr = maps + (int64_t)2 * nb * nb + ((int64_t)dir * NF + f) * 512;
        // left factor: row m = (rm, a), column k = (rk, b); right factor: row k = (rk, a), column m = (rm, b)
        const cd lu = dir == 0 ? U[(k & 7) * 8 + (m & 7)] : U[(m & 7) * 8 + (k & 7)];
        const cd l = {lu.re, dir == 0 ? -lu.im : lu.im};
        const cd rv = dir == 0 ? V[(k & 7) * 8 + (m & 7)] : V[(m & 7) * 8 + (k & 7)];
        const cd r = {rv.re, dir == 0 ? rv.im : -rv.im};
        fr[st * 64 + lane] = rm == rk ? l.re : (rm == 0 ? -l.im : l.im);
        fr[(4 + st) * 64 + lane] = rk == rm ? r.re : (rk == 0 ? r.im : -r.im);
    }
}

}  // namespace

hipError_t launch_gram(const uint8_t *img, int64_t stride, int h, int w, int c, int s, int64_t *out, hipStream_t st) {
    const int ny = ref_count(h, s), nx = ref_count(w, s);
    hipError_t e = launch_zero(out, sizeof(int64_t) * 2 * c * c * 64, st);
    if (e != hipSuccess) return e;
    if (c != 1 && c != 3) {
        const int nt = (8 * c + 63) / 64, n_tp = nt * (nt + 1) / 2;
        // vector slices for 256 to 512 workgroups of about 40 chunks, each with at least 8 and at most GB_MAX
        const int64_t n_chunks = ((int64_t)ny * nx * 8 + GB_VEC - 1) / GB_VEC;
        const int64_t blocks = std::min<int64_t>(512, std::max<int64_t>(256, n_chunks * 2 * n_tp / 40));
        const int64_t zs = std::max<int64_t>(
            {1, std::min<int64_t>((blocks + 2 * n_tp - 1) / (2 * n_tp), n_chunks / 8), (n_chunks + GB_MAX - 1) / GB_MAX});
        for (int64_t z0 = 0; z0 < zs; z0 += 65535) {   // blocks along z of a launch
            hipLaunchKernelGGL(gram_bands_kernel, dim3((unsigned)n_tp, 2, (unsigned)std::min<int64_t>(65535, zs - z0)),
                               dim3(256), 0, st, img, stride, h, w, c, s, ny, nx,
                               reinterpret_cast<unsigned long long *>(out), (int)z0, (int)zs);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        return hipSuccess;
    }
    const int64_t n_vec = std::max<int64_t>((int64_t)ny * w, (int64_t)nx * h);
    const int nb = (int)std::min<int64_t>(GR_MAX_BLOCKS, (n_vec + GR_CHUNK - 1) / GR_CHUNK);
    unsigned long long *o = reinterpret_cast<unsigned long long *>(out);
    if (c == 3)
        hipLaunchKernelGGL(gram_kernel<3>, dim3(nb, 2), dim3(GR_THREADS), 0, st, img, stride, h, w, s, ny, nx, o);
    else
        hipLaunchKernelGGL(gram_kernel<1>, dim3(nb, 2), dim3(GR_THREADS), 0, st, img, stride, h, w, s, ny, nx, o);
    return hipGetLastError();
}

size_t band_learn_words(int c) { return (size_t)2 * c * 64 + (size_t)(c / 2 + 1) * 2 * 64 * 2 + (size_t)2 * c * 64; }

// Basis of a c-band cube from its Gram sums: maps (BandMaps layout) and uv = U then V, slice-major,
// (in work, band_learn_words 8-byte words; *uv is set to their place there).
hipError_t launch_band_learn(const int64_t *gram, int c, int nb, void *work, double *maps, double **uv,
                             hipStream_t st) {
    int64_t *fold = (int64_t *)work;
    cd *vec = (cd *)(fold + (size_t)2 * c * 64);
    *uv = (double *)(vec + (size_t)(c / 2 + 1) * 2 * 64);
    hipLaunchKernelGGL(gram_fold_kernel, dim3(2 * c), dim3(64), 0, st, gram, c, fold);
    hipLaunchKernelGGL(band_evd_kernel, dim3((c / 2 + 1) * 2), dim3(64), 0, st, fold, c, vec);
    hipLaunchKernelGGL(band_basis_kernel, dim3(c), dim3(128), 0, st, vec, c, *uv);
    hipLaunchKernelGGL(band_maps_kernel, dim3(c / 2 + 2), dim3(256), 0, st, vec, c, nb, maps);
    return hipGetLastError();
}

}  // namespace htsvd
