// Collaborative filtering (Eq. 19-21) and aggregation (Algorithm 1) on the matrix cores of gfx950.
//
// The per-patch transform S = U^T * G * V is linear in the patch, and with the 3-point DFT along
// the channel mode (Eq. 4-5) it splits into a real 64 x 64 map on the channel sum and a complex
// 64 x 64 map on the first Fourier slice; the third slice is the conjugate of the second.  The
// Haar transform along the group (Eq. 7-8) is a 32 x 32 map on the patches (block diagonal for
// groups of 4, 8 or 16).  A wavefront takes 32 patches (32 / K groups) per step through a chain of
// matrix products in which every result is already the operand layout of the next product
// (lane = Haar row or pixel, registers = the index summed over next), so that nothing is
// transposed through LDS:
//
//   1  first Haar level    D = X^T H^T: A = 16 pixels x 32 patches (bytes as fp16 1024 + b),
//      B = the scaled sums (tile 0) and differences (tile 1) of the 16 pairs of patches.
//      Chaining B, G, R in one accumulator gives a0 = R+G+B; p = a0 - 1.5 (G+B) = R - (G+B)/2
//      and q = B - G follow.  All of it is exact, and has at most 11 significant bits.
//   2  forward t-product      S = F [a0; p; q]: A = F (fp16 hi + lo, ~22-bit matrix), B = the pair
//      rows of the pixels, exact in fp16.  With re' = A p + B q and im' = 1.5 A q - 2 B p only
//      three 64 x 64 matrices are needed for both slices.
//      S0 = s0' + 2 re', S1 = s0' - re' - im', S2 = s0' - re' + im'  (1/3 and sqrt3 folded into F).
//      The further Haar levels are butterflies between the lanes of tile 0 (one multiply-add with
//      a moved operand per value and level; see HaarRow).
//   3  threshold              keep |s| >= tau (Eq. 20), with tau scaled per lane (a lane is one
//      Haar row); values within 0.05 of tau are re-decided in FP64 from the uint8 group and the
//      FP64 transform.
//   4  inverse t-product      A = the kept coefficients s0 = S0+S1+S2, sr = 2S0-S1-S2, dn = S1-S2,
//      split into fp16 hi + lo, B = F^T (hi + lo): all four products, in two instructions of
//      depth 32 = 16 coefficients x (hi, lo).  A (16 coefficients x 16 Haar rows) block that
//      thresholding killed is skipped.
//   5  inverse Haar           A = H (entries 0, +- powers of two), B = the Haar rows of the reconstructed pixels,
//      split into fp16 hi + lo; the result has 16 pixels along the lanes and the patches in
//      registers.
//   Algorithm 1: every reconstructed patch is added (sums and a count) into an LDS copy of the
//             image region the tile's groups reach; the region goes to the tile's slot of a
//             global buffer and the gather kernel divides.  Groups whose members lie anywhere
//             (the spatio-temporal groups of a video) add into global 64-bit fixed-point sums
//             instead, with a histogram of patch positions for the counts.
//
// c = 1 uses the single 64 x 64 map and no channel DFT.
#include <algorithm>

#include "common.h"

namespace htsvd {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef short v4s __attribute__((ext_vector_type(4)));

namespace {

constexpr int MW = 8;          // wavefronts per workgroup (two per SIMD)
constexpr int MNEAR = 64;      // near-threshold list capacity per wavefront
constexpr float MGUARD = 0.05f;

struct MfmaShared {
    int r0, c0;
    int near_n[MW];
    int near_a[MW][MNEAR];     // lane | bit of the lane's coefficient << 6
    int near_b[MW][MNEAR];     // coefficient q
    int near_kill[MW][MNEAR];
};

// Per-wave scratch: the address of every patch of the step and its offset in the region.
struct WaveScratch {
    uint64_t addr[32];
    int off[32];
};

// Operand tables (BasisDev::frag): the maps M0, A, B (c = 1: M0), each [coefficient tile 4][k-step
// 2][hi, lo][half of the k-step 2][lane][4 halves].  Entry j of lane 16 g + m is coefficient m of
// the tile against pixel 4 g + j of pixel set q = 2 (k-step) + half; pixel p of set q is row p / 2,
// column 4 (p % 2) + q of the patch.  The forward products read a lane's two halves of a k-step
// (lane = coefficient); the inverse products read 16 coefficients x 16 pixels of one set with the
// transposing LDS load (lane = pixel), so one copy in LDS serves both directions, without bank
// conflicts either way.
template <int C>
struct Frag {
    static constexpr int NM = C == 3 ? 3 : 1;           // 64 x 64 maps
    static constexpr int MAP = 4 * 2 * 2 * 64;          // 16-byte words per map
};
// LDS besides the region: the maps, the two Haar operands, the waves' scratch.
constexpr int HAAR_V8 = 4 * 64;   // [forward tile 2, inverse tile 2][lane]
template <int C>
__host__ __device__ constexpr int fixed_lds_bytes() {
    return (Frag<C>::NM * Frag<C>::MAP + HAAR_V8) * 16 + 16 * 32 + MW * (int)sizeof(WaveScratch);
}

// Haar rows of a step's 32 patches.  Tile 1, lane n: the difference of pair n (patches 2n, 2n + 1),
// times 1/2.  Tile 0 starts as the pair sums, times 2^-5, and each further level l = 2 .. log2 K
// makes a sum and a difference of two lanes: v += s v(partner), s = 1 in the lane that keeps the
// sum, -1 in the one that keeps the difference (its own side minus the partner's), 0 in lanes
// whose row is finished.  The partners n ^ 1, n ^ 2, n ^ 7, n ^ 15 are the lane permutations that
// an operand can take within a row of 16 lanes, so the sums stay in lanes that they pair: after
// level 2 in positions 0 and 2 of an even quad of lanes and 1 and 3 of an odd one, then in lanes
// 0, 7, 8, 15, then 0 and 15, then 0.
// The row of a lane covers patches first .. first + 2^l - 1: their sum, or the half that holds pair
// n minus the other.
struct HaarRow {
    int l, first;
    bool sum;
};
// s of lane n at level l (2 .. 5), before the levels past log2 K are dropped.
__device__ inline int haar_step(int l, int n) {
    const int odd = (n >> 2) & 1;                       // quad of lanes
    const bool sum2 = (n & 1) == odd;
    if (l == 2) return sum2 ? 1 : -1;
    const bool sum3 = sum2 && (n & 3) == 3 * odd;
    if (l == 3) return sum2 ? (sum3 ? 1 : -1) : 0;
    const bool sum4 = sum3 && (n == 0 || n == 15);
    if (l == 4) return sum3 ? (sum4 ? 1 : -1) : 0;
    return sum4 ? (n == 0 ? 1 : -1) : 0;
}
__device__ inline HaarRow haar_row_of(int K, int ht, int n) {
    if (ht == 1) return {1, 2 * n, false};
    int l = 2;
    while ((1 << l) < K && haar_step(l, n) == 1) ++l;   // the level the lane ends at
    return {l, (2 * n >> l) << l, haar_step(l, n) == 1};
}
__device__ inline float haar_sign(const HaarRow &r, int n, int mu, bool pair) {
    if ((mu >> r.l) != (r.first >> r.l)) return 0.f;
    if (pair) return (mu & 1) ? -1.f : 1.f;             // tile 1: first minus second
    return r.sum || ((mu ^ (2 * n)) >> (r.l - 1) & 1) == 0 ? 1.f : -1.f;
}
// 2^(e/2)
__device__ inline float root2(int e) {
    return __uint_as_float((uint32_t)(127 + (e >> 1)) << 23) * ((e & 1) ? 1.41421356237309505f : 1.f);
}
// The butterflies of levels 2 .. 5 on 4 C values per lane; s[l - 2] as above (0 past log2 K).  In one
// block of assembly because the moved operand is part of the multiply-add; a value is read by the
// move no sooner than 4 C - 1 instructions after it was written, and the block starts with the two
// wait states a move needs after the values' own instructions, which must be vector ones.
template <int C>
__device__ inline void haar_lanes(v4f (&v)[C], const float (&s)[4]) {
#define HB_ROW(x, y, z, w, cof, ctl)                                          \
    "v_fmac_f32_dpp %" #x ", %" #x ", %" #cof " " ctl " row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #y ", %" #y ", %" #cof " " ctl " row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #z ", %" #z ", %" #cof " " ctl " row_mask:0xf bank_mask:0xf\n" \
    "v_fmac_f32_dpp %" #w ", %" #w ", %" #cof " " ctl " row_mask:0xf bank_mask:0xf\n"
    if constexpr (C == 3) {
#define HB_LEVEL(cof, ctl) HB_ROW(0, 1, 2, 3, cof, ctl) HB_ROW(4, 5, 6, 7, cof, ctl) HB_ROW(8, 9, 10, 11, cof, ctl)
        asm("s_nop 1\n" HB_LEVEL(12, "quad_perm:[1,0,3,2]") HB_LEVEL(13, "quad_perm:[2,3,0,1]")
                HB_LEVEL(14, "row_half_mirror") HB_LEVEL(15, "row_mirror")
            : "+v"(v[0][0]), "+v"(v[0][1]), "+v"(v[0][2]), "+v"(v[0][3]), "+v"(v[1][0]), "+v"(v[1][1]), "+v"(v[1][2]),
              "+v"(v[1][3]), "+v"(v[2][0]), "+v"(v[2][1]), "+v"(v[2][2]), "+v"(v[2][3])
            : "v"(s[0]), "v"(s[1]), "v"(s[2]), "v"(s[3]));
#undef HB_LEVEL
    } else {
#define HB_LEVEL(cof, ctl) HB_ROW(0, 1, 2, 3, cof, ctl)
        asm("s_nop 1\n" HB_LEVEL(4, "quad_perm:[1,0,3,2]") HB_LEVEL(5, "quad_perm:[2,3,0,1]")
                HB_LEVEL(6, "row_half_mirror") HB_LEVEL(7, "row_mirror")
            : "+v"(v[0][0]), "+v"(v[0][1]), "+v"(v[0][2]), "+v"(v[0][3])
            : "v"(s[0]), "v"(s[1]), "v"(s[2]), "v"(s[3]));
#undef HB_LEVEL
    }
#undef HB_ROW
}

// 4 pixels (4 C bytes) of global memory, any alignment.
template <int C>
__device__ inline void load_seg(uint64_t addr, uint32_t (&out)[C]) {
    typedef uint32_t u32x __attribute__((ext_vector_type(C == 3 ? 3 : 2)));
    if constexpr (C == 3) {
        typedef u32x __attribute__((aligned(1))) u32xu;
        const u32x s = *(const __attribute__((address_space(1))) u32xu *)addr;
        out[0] = s[0];
        out[1] = s[1];
        out[2] = s[2];
    } else {
        typedef uint32_t __attribute__((aligned(1))) u32u;
        out[0] = *(const __attribute__((address_space(1))) u32u *)addr;
    }
}

// Two floats as a packed pair of fp16: round toward zero, and round to nearest even.
__device__ inline uint32_t pack_rtz(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(lo, hi));
}
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));
__device__ inline uint32_t pack_rne(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f){lo, hi}, v2h));
}
// The parts of (a, b) that the packed pair h leaves, rounded to nearest, packed.
__device__ inline uint32_t pack_rest(float a, float b, uint32_t h) {
    const v2h hv = __builtin_bit_cast(v2h, h);
    float m1 = -1.f;
    asm("" : "+s"(m1));   // not a plain subtraction, so that it becomes one mixed-precision instruction
    v2h r;
    r[0] = (_Float16)__builtin_fmaf((float)hv[0], m1, a);
    r[1] = (_Float16)__builtin_fmaf((float)hv[1], m1, b);
    return __builtin_bit_cast(uint32_t, r);
}

__device__ inline v8h as_v8h(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
    return __builtin_bit_cast(v8h, make_uint4(a, b, c, d));
}

__device__ inline v4f mfma(v8h a, v8h b, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }

// Transposing LDS load: each block of 16 lanes reads four rows of 16 halves (a lane points at
// halves 4 (i % 4) .. of row i / 4), and lane i receives column i of the four rows.
__device__ inline v4h lds_read_tr(const v4h *p) {
    return __builtin_bit_cast(v4h, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)p));
}

__device__ inline void wave_lds_fence() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

__device__ inline double wave_sum64(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Keeps the values of v with |v| > lo and zeroes the others; the lanes that kept one are added to
// `kept`, those with a kept one below hi to `band`.  In assembly so that the masks live for one
// call only (left to the compiler, the masks of a whole pass stay live and spill); every mask is
// read two or more vector instructions after it was written.
__device__ inline void threshold4(v4f &v, float lo, float hi, uint64_t &kept, uint64_t &band) {
    uint64_t m0, m1, m2, m3, n0, n1, n2, n3;
    asm("v_cmp_gt_f32_e64 %4, |%0|, %12\n"
        "v_cmp_gt_f32_e64 %5, |%1|, %12\n"
        "v_cmp_gt_f32_e64 %6, |%2|, %12\n"
        "v_cmp_gt_f32_e64 %7, |%3|, %12\n"
        "v_cmp_lt_f32_e64 %8, |%0|, %13\n"
        "v_cmp_lt_f32_e64 %9, |%1|, %13\n"
        "v_cmp_lt_f32_e64 %10, |%2|, %13\n"
        "v_cmp_lt_f32_e64 %11, |%3|, %13\n"
        "v_cndmask_b32_e64 %0, 0, %0, %4\n"
        "v_cndmask_b32_e64 %1, 0, %1, %5\n"
        "v_cndmask_b32_e64 %2, 0, %2, %6\n"
        "v_cndmask_b32_e64 %3, 0, %3, %7\n"
        "s_and_b64 %8, %8, %4\n"
        "s_and_b64 %9, %9, %5\n"
        "s_and_b64 %10, %10, %6\n"
        "s_and_b64 %11, %11, %7\n"
        "s_or_b64 %8, %8, %9\n"
        "s_or_b64 %10, %10, %11\n"
        "s_or_b64 %4, %4, %5\n"
        "s_or_b64 %6, %6, %7\n"
        "s_or_b64 %8, %8, %10\n"
        "s_or_b64 %4, %4, %6\n"
        : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "=&s"(m0), "=&s"(m1), "=&s"(m2), "=&s"(m3), "=&s"(n0),
          "=&s"(n1), "=&s"(n2), "=&s"(n3)
        : "v"(lo), "v"(hi)
        : "scc");
    kept |= m0;
    band |= n0;
}

// Contribution in fixed point (round to nearest even) plus the bits of MAGIC; |v| is clamped to
// 1024 (four times the 8-bit range) so that no region sum can overflow (see the accumulation
// shift of the tiling).  The scale 2^FS (FS <= 12) is applied here, after the fp16 products,
// whose range it would exceed.  |v| scale <= 2^22, so v scale + 1.5 * 2^23 lies in [2^23, 2^24],
// where floats are the integers: one fused multiply-add rounds to nearest even and the bits
// give the integer.  Sums of n such words hold n times the bits of MAGIC modulo 2^32; the flush
// of a tile, which knows n, takes them out.
constexpr float MAGIC = 12582912.0f;   // 1.5 * 2^23
constexpr uint32_t MAGIC_BITS = 0x4b400000u;
__device__ inline uint32_t to_fixed_biased(float v, float scale) {
    return __float_as_uint(fmaf(__builtin_amdgcn_fmed3f(v, -1024.f, 1024.f), scale, MAGIC));
}
__device__ inline int to_fixed(float v, float scale) { return (int)(to_fixed_biased(v, scale) - MAGIC_BITS); }

// Fixed-point shift of the global aggregation.  Its 64-bit sums cannot overflow; the int32 slot
// regions of a tile receive at most TY TX K contributions per pixel (one per member of each of
// the tile's groups), each of |v| <= 1024, so a tiling uses the largest shift <= GA_FS that
// keeps TY TX K 1024 2^FS below 2^31, and only tilings with a shift of at least GA_MIN_FS.
constexpr int GA_FS = 12;
constexpr int GA_MIN_FS = 10;
constexpr int GA_PADDED_MIN_FS = 9;   // of the tiles that set the least shift
constexpr int GA_MAX_TILE = 8;   // largest tile side of the slot regions, and that of the sums in memory

// Geometry of a video for the global aggregation: frames of h_frame rows stacked vertically,
// ny_frame reference rows each; with slot regions (GA == 2) a tile's references lie in one
// frame t and its LDS region holds the frames f_lo .. f_lo + nslot - 1 (f_lo =
// max(0, t - radius)) as nslot blocks of RH x RP pixels (columns RW used).
struct VideoTiling {
    int T = 1, h_frame = 0, ny_frame = 0, radius = 0, nslot = 1;
    int RH = 0, RW = 0, RP = 0;
};

// What a lane (by its place n in a row of 16) knows of its row of tile 0: the butterfly factors (0
// past log2 K), the factor of tau, the group, and whether it is a row of sums.  Rows are scaled by
// 2^-5 (in tile 1 by 2^-1), times the orthonormal 2^(l/2).  Kept in LDS and read once a step, so
// that nothing of it occupies registers between steps.
struct alignas(16) LaneRow {
    float hs[4];
    float rs;
    int gi, sum, pad;
};

// The LDS of a workgroup: tables (filled once), wave scratch, then the region.
template <int C>
struct FilterLds {
    const v4h *F;       // maps
    v8h *H;             // Haar operands
    LaneRow *rows;
    WaveScratch *ws;
    int *region;
};

// Fills the tables for group size K (the caller's barrier follows).
template <int C>
__device__ __forceinline__ FilterLds<C> filter_lds_init(float *smem, const v8h *__restrict__ FG, const int K) {
    FilterLds<C> L;
    v8h *F8 = reinterpret_cast<v8h *>(smem);
    L.F = reinterpret_cast<const v4h *>(smem);
    L.H = F8 + Frag<C>::NM * Frag<C>::MAP;
    L.rows = reinterpret_cast<LaneRow *>(L.H + HAAR_V8);
    L.ws = reinterpret_cast<WaveScratch *>(L.rows + 16);
    if (threadIdx.x < 16) {
        const int n = threadIdx.x, lk = 31 - __builtin_clz(K);
        const HaarRow r = haar_row_of(K, 0, n);
        LaneRow w;
        for (int l = 2; l <= 5; ++l) w.hs[l - 2] = l <= lk ? (float)haar_step(l, n) : 0.f;
        w.rs = root2(r.l - 10);
        w.gi = r.first >> lk;
        w.sum = r.sum;
        w.pad = 0;
        L.rows[n] = w;
    }
    L.region = reinterpret_cast<int *>(L.ws + MW);
    for (int e = threadIdx.x; e < Frag<C>::NM * Frag<C>::MAP; e += MW * 64) F8[e] = FG[e];
    for (int e = threadIdx.x; e < HAAR_V8; e += MW * 64) {
        const int l = e & 63, n = l & 15, g = l >> 4, t = (e >> 6) & 1;
        v8h v;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (e < 128) {   // first level: pair n of tile t, patch 8g + j
                const int mu = 8 * g + j;
                v[j] = (_Float16)((mu >> 1) != n ? 0.f : (t == 0 ? 0.03125f : ((mu & 1) ? -0.5f : 0.5f)));
            } else {         // inverse: patch 16t + n, lane row 4g + j%4 of tile j/4
                const int m = 4 * g + (j & 3);
                const HaarRow r = haar_row_of(K, j >> 2, m);
                v[j] = (_Float16)(haar_sign(r, m, 16 * t + n, j >= 4) * (j >= 4 ? 1.f : (float)(1 << (5 - r.l))));
            }
        }
        L.H[e] = v;
    }
    return L;
}

// One reference tile: every group of the tile, 32 patches (32/K groups) per wavefront step.
//   GA: global aggregation into gacc[pix*C + ch] (units of 2^-tg.FS) and ghist[pix] (patches by
//   top-left pixel).  GA == 1: every contribution goes to gacc, the tile only schedules
//   references and the region's place holds 256 C words per wave; GA == 2: the tile (references of one frame) adds into
//   its LDS slot region, which then goes to the tile's slot of a global region buffer (at gacc,
//   C * plane int32 per tile) for ga_gather_kernel.
//
// What bounds it, per 32-patch step at C = 3, two waves sharing a SIMD: 24 + 160 + at most 320 (106
// on the 12 MP image, where most blocks die) + 48 matrix instructions of 16 cycles, about 1,800
// vector instructions of 4, and the waits between a wave's phases that its one neighbour does not
// fill; the vector instructions lead.  Measured on the 12 MP image (stride 3, window 31, K 32,
// estimated noise level): 16.1 -> 9.0 ms against a form that transposed the coefficients through
// LDS, ran all Haar levels in registers on both sides and read its tables through the caches (3,840
// vector and 143 matrix instructions of twice the size per step); 0.57 -> 0.24 ms for 509 x 763 at
// sigma 10, K 16.  Of these, 1.5 and 0.18 ms are the FP64 re-decisions, which read the patches of a
// row side by side instead of one after the other.
template <int C, bool RA = false, int GA = 0>
__device__ __forceinline__ void filter_tile_mfma(const ImageGeom &g, const TileGeom &tg, const FilterLds<C> &L,
                                                 const double *__restrict__ T64, const int K,
                                                 const int32_t *__restrict__ idx, const int idx_stride,
                                                 const double *__restrict__ tau_ref, const double tau_mul,
                                                 float *__restrict__ regions,
                                                 unsigned long long *__restrict__ guard_count, const int tile,
                                                 MfmaShared &sh, const float *__restrict__ ra_d = nullptr,
                                                 const uint8_t *__restrict__ ra_flag = nullptr,
                                                 unsigned long long *__restrict__ gacc = nullptr,
                                                 int *__restrict__ ghist = nullptr,
                                                 const VideoTiling &vt = VideoTiling{}) {
    constexpr int P = 64 * C;
    const int lk = 31 - __builtin_clz(K);   // log2 K
    const int G = 32 >> lk;                 // groups per step
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ty = tile / tg.tiles_x, tx = tile % tg.tiles_x;
    WaveScratch &ws = L.ws[wave];
    const int plane = region_plane(tg), relems = region_elems(tg, C);
    // LDS accumulation in int32 (float atomics in LDS are far slower than integer ones):
    // channel sums in units of 2^-FS, then patches by top-left pixel, which become the count.
    int *iregion = L.region;
    int *hist = iregion + C * plane;
    const float fscale = (float)(1 << tg.FS);
    // references of the tile: rows iy0 .. iy0 + ny_t - 1 of the grid; with slot regions the
    // tiles are cut per frame (frame t_v, its reference rows from iyl0)
    int iy0 = ty * tg.TY, ny_t = min(tg.TY, g.ny - iy0);
    int t_v = 0, f_lo = 0;
    if constexpr (GA == 2) {
        const int tyf = (vt.ny_frame + tg.TY - 1) / tg.TY;
        t_v = ty / tyf;
        const int iyl0 = (ty - t_v * tyf) * tg.TY;
        iy0 = t_v * vt.ny_frame + iyl0;
        ny_t = min(tg.TY, vt.ny_frame - iyl0);
        f_lo = max(0, t_v - vt.radius);
        if (tid == 0) {
            sh.r0 = max(0, ref_pos(iyl0, vt.ny_frame, vt.h_frame, g.s) - tg.R);
            sh.c0 = max(0, ref_pos(tx * tg.TX, g.nx, g.w, g.s) - tg.R);
        }
        for (int e = tid; e < C * plane; e += MW * 64) iregion[e] = 0;
    }
    if constexpr (!GA) {
        if (tid == 0) {
            int r0, r1, c0, c1;
            region_rows(g, tg, ty, &r0, &r1);
            region_cols(g, tg, tx, &c0, &c1);
            sh.r0 = r0;
            sh.c0 = c0;
        }
        for (int e = tid; e < relems; e += MW * 64) iregion[e] = 0;
    }
    __syncthreads();
    const int r0 = sh.r0, c0 = sh.c0;
    const int ix0 = tx * tg.TX;
    const int nx_t = min(tg.TX, g.nx - ix0);
    const int nref = ny_t * nx_t;
    const int rp = GA == 1 ? g.w : tg.RP;   // row pitch of the aggregation target

    // Patch positions: lane mu (and mu + 32) looks up patch mu of a step; the position of the next
    // step's patch is loaded one step ahead, and its pixels while the last phase runs.
    const uint32_t w_inv = (uint32_t)(0xffffffffu / (uint32_t)g.w) + 1u;   // lin / w = mulhi(lin, w_inv), or one more
    const uint32_t nx_inv = 65535u / (uint32_t)nx_t + 1u;                  // t / nx_t = t nx_inv >> 16 for t < 256
    auto ref_at = [&](int b, int gi) -> int64_t {
        const int t = min(b + gi, nref - 1), q = (int)((uint32_t)t * nx_inv >> 16);
        return (int64_t)(iy0 + q) * g.nx + (ix0 + t - q * nx_t);
    };
    auto position = [&](int b) { return idx[ref_at(b, (tid & 31) >> lk) * idx_stride + (tid & (K - 1))]; };
    int off_own = 0;
    uint32_t raw[8][C];   // 4 pixels of patches 8 gq .. 8 gq + 7
    auto fetch = [&](int32_t lin, int lane) {
        const int n16 = lane & 15, gq = lane >> 4;
        // bytes of this lane's 4 pixels of a patch: row n16/2, columns 4 (n16 % 2) ..
        const int64_t seg = (int64_t)(n16 >> 1) * g.stride + (n16 & 1) * 4 * C;
        int yin = (int)__umulhi((uint32_t)lin, w_inv);
        if (yin * g.w > lin) --yin;
        const int xin = lin - yin * g.w;
        if constexpr (GA == 1) {
            off_own = lin;
        } else if constexpr (GA == 2) {
            const int f = yin / vt.h_frame;   // stacked row -> frame, slot and row in the frame
            off_own = ((f - f_lo) * vt.RH + (yin - f * vt.h_frame - r0)) * rp + (xin - c0);
        } else {
            off_own = (yin - r0) * rp + (xin - c0);
        }
        wave_lds_fence();   // earlier reads of the scratch are done
        if (lane < 32) {
            ws.addr[lane] = (uint64_t)(uintptr_t)(g.img + (int64_t)yin * g.stride + (int64_t)xin * C);
            ws.off[lane] = off_own;
        }
        wave_lds_fence();
#pragma unroll
        for (int j = 0; j < 8; ++j) load_seg<C>(ws.addr[8 * gq + j] + seg, raw[j]);
    };
    int32_t lin_next = 0;
    if (wave * G < nref) {
        lin_next = position(wave * G);
        fetch(lin_next, tid & 63);
    }
    for (int base = wave * G; base < nref; base += MW * G) {
        const bool full = base + G <= nref;
        auto ref_of = [&](int gi) { return ref_at(base, gi); };
        // everything that depends on the lane alone is made anew in each step (an opaque copy), so
        // that it does not hold registers across the product loop
        int lane = tid & 63;
        asm volatile("" : "+v"(lane));
        const int n16 = lane & 15, gq = lane >> 4;
        if (lane < 32 && (full || base + (lane >> lk) < nref)) {
            if constexpr (GA != 0)
                atomicAdd(ghist + lin_next, 1);
            else
                atomicAdd(hist + off_own, 1);
        }
        lin_next = position(base + MW * G);
        // ---- 1: pair sums and differences of the pixels ----
        // bh[sl][s][ht]: B operands of the forward products (pair n16 of tile ht, 32 pixels per k-step s)
        v8h bh[C][2][2];
        {
            // A operands: pixel byte t of patches 8 gq .. 8 gq + 7 as fp16 1024 + b
            uint32_t a[4 * C][4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int d = 0; d < C; ++d) {
                    const uint32_t x = raw[2 * i][d], y = raw[2 * i + 1][d];
                    const uint32_t lo = __builtin_amdgcn_perm(y, x, 0x05010400u);   // x0 y0 x1 y1
                    const uint32_t hi = __builtin_amdgcn_perm(y, x, 0x07030602u);   // x2 y2 x3 y3
                    const uint32_t k64 = 0x64646464u;
                    a[4 * d][i] = __builtin_amdgcn_perm(k64, lo, 0x04010400u);
                    a[4 * d + 1][i] = __builtin_amdgcn_perm(k64, lo, 0x04030402u);
                    a[4 * d + 2][i] = __builtin_amdgcn_perm(k64, hi, 0x04010400u);
                    a[4 * d + 3][i] = __builtin_amdgcn_perm(k64, hi, 0x04030402u);
                }
            const v4f zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ht = 0; ht < 2; ++ht) {
                const v8h hb = L.H[ht * 64 + lane];
                uint32_t ph[C][2][4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {   // pixel q of the lane's four: D rows 4 gq + r
                    v4f v[C];
                    if constexpr (C == 3) {
                        const v4f bb = mfma(as_v8h(a[3 * q + 2][0], a[3 * q + 2][1], a[3 * q + 2][2], a[3 * q + 2][3]), hb, zero);
                        const v4f t = mfma(as_v8h(a[3 * q + 1][0], a[3 * q + 1][1], a[3 * q + 1][2], a[3 * q + 1][3]), hb, bb);
                        const v4f s = mfma(as_v8h(a[3 * q][0], a[3 * q][1], a[3 * q][2], a[3 * q][3]), hb, t);
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            v[0][r] = ht == 0 ? s[r] - 192.f : s[r];   // 6 x 1024 / 32
                            v[1][r] = fmaf(-1.5f, t[r], s[r]);
                            v[2][r] = fmaf(2.f, bb[r], -t[r]);
                        }
                    } else {
                        v[0] = mfma(as_v8h(a[q][0], a[q][1], a[q][2], a[q][3]), hb, zero);
                        if (ht == 0) v[0] -= 64.f;   // 2 x 1024 / 32
                    }
#pragma unroll
                    for (int sl = 0; sl < C; ++sl)
#pragma unroll
                        for (int r2 = 0; r2 < 2; ++r2) {
                            ph[sl][q >> 1][2 * (q & 1) + r2] = pack_rtz(v[sl][2 * r2], v[sl][2 * r2 + 1]);
                        }
                }
#pragma unroll
                for (int sl = 0; sl < C; ++sl)
#pragma unroll
                    for (int s = 0; s < 2; ++s) {
                        bh[sl][s][ht] = as_v8h(ph[sl][s][0], ph[sl][s][1], ph[sl][s][2], ph[sl][s][3]);
                    }
            }
        }
        // ---- thresholds of this lane's Haar rows: keep-or-undecided above lo, undecided below hi
        // (the guard band (tau - g, tau + g) scaled alike); without a guard band lo is the
        // float just below the threshold and hi = lo (empty band)
        const LaneRow row0 = L.rows[n16];
        const int gi_row[2] = {row0.gi, (2 * n16) >> lk};
        const float rs[2] = {row0.rs, 0.70710678118654752f};
        const float (&hs)[4] = row0.hs;
        float tau_l[2], lo_t[2], hi_t[2];
        uint32_t rafl = 0;   // bit ht: this lane's row of tile ht is the first row of a refined group
        int64_t ra_row = 0;
#pragma unroll
        for (int ht = 0; ht < 2; ++ht) {
            const int gi = gi_row[ht];
            const bool valid = base + gi < nref;
            const int64_t rr = ref_of(gi);
            const double tau = tau_ref[rr] * tau_mul;
            const float tf = valid ? (float)tau : __builtin_inff();
            const bool guard = valid && tau > (double)MGUARD;
            const float tl = tf * rs[ht];
            // a >= tl  <=>  a > (the float just below tl); tl = 0 keeps everything
            const float below = tl > 0.f ? __int_as_float(__float_as_int(tl) - 1) : -1.f;
            tau_l[ht] = tl;
            lo_t[ht] = guard ? tl - MGUARD * rs[ht] : below;
            hi_t[ht] = guard ? tl + MGUARD * rs[ht] : lo_t[ht];
            if constexpr (RA) {
                // RA-Haar-tSVD: the row of sums of a refined group, K times the transform of the mean,
                // becomes K T p_est by taking off K ra_d(q), and is kept without threshold
                if (ht == 0 && row0.sum != 0 && valid && ra_flag[rr]) {
                    rafl = 1;
                    ra_row = rr * P;
                    lo_t[0] = hi_t[0] = -1.f;
                }
            }
        }

        const v4h *FL = L.F + lane;                                      // forward operands
        const v4h *FT = L.F + (4 * gq + (n16 >> 2)) + 16 * (n16 & 3);    // transposing reads
        v4f out[C][4][2];   // [p0, 2 pr, pi][pixel set][Haar tile]
#pragma unroll
        for (int sl = 0; sl < C; ++sl)
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int ht = 0; ht < 2; ++ht) out[sl][t][ht] = (v4f){0.f, 0.f, 0.f, 0.f};

        // four passes over the coefficients 16 ct + 4 gq + r of every slice
#pragma unroll 1
        for (int ct = 0; ct < 4; ++ct) {
            // ---- 2: forward products ----
            // acc[.][ht]: s0'; A p + B q; B p; A q
            constexpr int NA = C == 3 ? 4 : 1;
            v4f acc[NA][2];
#pragma unroll
            for (int i = 0; i < NA; ++i)
#pragma unroll
                for (int ht = 0; ht < 2; ++ht) acc[i][ht] = (v4f){0.f, 0.f, 0.f, 0.f};
            // The maps' operands of k-step 1 take the registers of k-step 0 as soon as those are used,
            // so their LDS latency passes under the products in between; the barriers keep the
            // compiler from moving the loads back to their uses.
            auto table = [&](int m, int s, int term) {
                const v4h *f = FL + m * 2 * Frag<C>::MAP + ((ct * 2 + s) * 2 + term) * 128;
                const v4h lo = f[0], hi = f[64];
                return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            };
            constexpr int NM = Frag<C>::NM;
            v8h f[NM][2];
#pragma unroll
            for (int m = 0; m < NM; ++m)
#pragma unroll
                for (int term = 0; term < 2; ++term) f[m][term] = table(m, 0, term);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
#pragma unroll
                for (int m = 0; m < NM; ++m) {
#pragma unroll
                    for (int term = 0; term < 2; ++term)
#pragma unroll
                        for (int ht = 0; ht < 2; ++ht) {
                            if (m == 0) acc[0][ht] = mfma(f[0][term], bh[0][s][ht], acc[0][ht]);
                            if constexpr (C == 3) {
                                if (m == 1) {
                                    acc[1][ht] = mfma(f[1][term], bh[1][s][ht], acc[1][ht]);
                                    acc[3][ht] = mfma(f[1][term], bh[2][s][ht], acc[3][ht]);
                                }
                                if (m == 2) {
                                    acc[1][ht] = mfma(f[2][term], bh[2][s][ht], acc[1][ht]);
                                    acc[2][ht] = mfma(f[2][term], bh[1][s][ht], acc[2][ht]);
                                }
                            }
                        }
                    if (s == 0) {
                        f[m][0] = table(m, 1, 0);
                        f[m][1] = table(m, 1, 1);
                    }
                }
            }
            // ---- inverse channel DFT, threshold ----
            v4f S[2][C];
            bool any[2], near[2];
#pragma unroll
            for (int ht = 0; ht < 2; ++ht) {
                if constexpr (C == 3) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float s0 = acc[0][ht][r], re = acc[1][ht][r];
                        const float u = fmaf(-0.75f, acc[3][ht][r], acc[2][ht][r]);   // -im'/2
                        const float t0 = s0 - re;
                        S[ht][0][r] = fmaf(2.f, re, s0);
                        S[ht][1][r] = fmaf(2.f, u, t0);
                        S[ht][2][r] = fmaf(-2.f, u, t0);
                    }
                } else {
                    // by a vector instruction: the assembly below must not read a matrix result directly
                    float one = 1.f;
                    asm("" : "+s"(one));
                    S[ht][0] = acc[0][ht] * one;
                }
                if (ht == 0) {
                    haar_lanes<C>(S[0], hs);
                    if constexpr (RA) {
                        if (rafl) {
                            const float kd = (float)K * 0.03125f;
#pragma unroll
                            for (int sl = 0; sl < C; ++sl) {
                                const float4 d = *reinterpret_cast<const float4 *>(ra_d + ra_row + 64 * sl + 16 * ct + 4 * gq);
                                S[0][sl][0] = fmaf(-kd, d.x, S[0][sl][0]);
                                S[0][sl][1] = fmaf(-kd, d.y, S[0][sl][1]);
                                S[0][sl][2] = fmaf(-kd, d.z, S[0][sl][2]);
                                S[0][sl][3] = fmaf(-kd, d.w, S[0][sl][3]);
                            }
                        }
                    }
                }
                uint64_t kept = 0, band = 0;
#pragma unroll
                for (int sl = 0; sl < C; ++sl) threshold4(S[ht][sl], lo_t[ht], hi_t[ht], kept, band);
                any[ht] = kept != 0;
                near[ht] = band != 0;
            }
            if (!(any[0] | any[1])) continue;

            // ---- FP64 re-decision of the coefficients inside the guard band (rare) ----
            if (near[0] | near[1]) {
                if (lane == 0) sh.near_n[wave] = 0;
                wave_lds_fence();
                // the comparisons are made again (opaque copies keep the masks of the threshold short-lived)
                float lo_o[2] = {lo_t[0], lo_t[1]}, hi_o[2] = {hi_t[0], hi_t[1]};
                asm volatile("" : "+v"(lo_o[0]), "+v"(lo_o[1]), "+v"(hi_o[0]), "+v"(hi_o[1]));
                uint32_t kill = 0, bits = 0;   // bit (ht * C + sl) * 4 + r
#pragma unroll
                for (int ht = 0; ht < 2; ++ht)
#pragma unroll
                    for (int sl = 0; sl < C; ++sl)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const float av = fabsf(S[ht][sl][r]);
                            bits |= (uint32_t)(av > lo_o[ht] && av < hi_o[ht]) << ((ht * C + sl) * 4 + r);
                        }
                while (bits) {
                    const int bit = __builtin_ctz(bits), r = bit & 3, ht = bit >= 4 * C, sl = (bit >> 2) - ht * C;
                    bits &= bits - 1;
                    const int e = atomicAdd(&sh.near_n[wave], 1);
                    if (e < MNEAR) {
                        sh.near_a[wave][e] = lane | (bit << 6);
                        sh.near_b[wave][e] = 64 * sl + 16 * ct + 4 * gq + r;
                    } else {   // list full: the FP32 value decides
                        float av = 0.f;
#pragma unroll
                        for (int i = 0; i < 8 * C; ++i)
                            if (i == bit) av = fabsf(S[i / (4 * C)][(i >> 2) % C][i & 3]);
                        if (!(av >= (ht ? tau_l[1] : tau_l[0]))) kill |= 1u << bit;
                    }
                }
                wave_lds_fence();
                const int n_all = sh.near_n[wave];
                const int nn = min(n_all, MNEAR);
                if (lane == 0) {
                    atomicAdd(guard_count, (unsigned long long)nn);
                    if (n_all > nn) atomicAdd(guard_count + 1, (unsigned long long)(n_all - nn));
                }
                for (int e = 0; e < nn; ++e) {
                    // sum over the patches of the row (signs +-1, exact in integers) at this lane's
                    // pixel, then against row q of the transform; eight patches' bytes in flight
                    const int ia = sh.near_a[wave][e], q = sh.near_b[wave][e];
                    const int n = ia & 15, ht = (ia >> 6) >= 4 * C;
                    const HaarRow hr = haar_row_of(K, ht, n);
                    const int cnt = 1 << hr.l;
                    const int64_t pix = (int64_t)(lane >> 3) * g.stride + (lane & 7) * C;
                    int sum[C] = {};
                    for (int m0 = 0; m0 < cnt; m0 += 8) {
                        int b[8][C];
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            const uint64_t a = ws.addr[hr.first + min(m0 + i, cnt - 1)] + pix;
#pragma unroll
                            for (int ch = 0; ch < C; ++ch)
                                b[i][ch] = ((const __attribute__((address_space(1))) uint8_t *)a)[ch];
                        }
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            const int w = m0 + i < cnt ? (int)haar_sign(hr, n, hr.first + m0 + i, ht) : 0;
#pragma unroll
                            for (int ch = 0; ch < C; ++ch) sum[ch] += w * b[i][ch];
                        }
                    }
                    double part = 0.0;
#pragma unroll
                    for (int ch = 0; ch < C; ++ch) part += T64[(int64_t)q * P + 64 * ch + lane] * (double)sum[ch];
                    part *= ((hr.l & 1) ? 0.70710678118654752440 : 1.0) / (double)(1 << (hr.l >> 1));
                    const int64_t rr = ref_of(hr.first >> lk);
                    const double sv = wave_sum64(part);
                    const double tau = tau_ref[rr] * tau_mul;
                    if (lane == 0) sh.near_kill[wave][e] = !(fabs(sv) >= tau);
                }
                wave_lds_fence();
                for (int e = 0; e < nn; ++e) {
                    const int ia = sh.near_a[wave][e];
                    if ((ia & 63) == lane && sh.near_kill[wave][e]) kill |= 1u << (ia >> 6);
                }
#pragma unroll
                for (int ht = 0; ht < 2; ++ht)
#pragma unroll
                    for (int sl = 0; sl < C; ++sl)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if ((kill >> ((ht * C + sl) * 4 + r)) & 1u) S[ht][sl][r] = 0.f;
            }

            // ---- 4: inverse products ----
#pragma unroll
            for (int ht = 0; ht < 2; ++ht) {
                if (!any[ht]) continue;   // wave-uniform: nothing kept, the products are zero
                // A operands [hi, hi] and [lo, lo] (coefficients 4 gq + j%4)
                auto split = [&](const v4f x, v8h &hh, v8h &ll) {
                    const uint32_t h0 = pack_rne(x[0], x[1]), h1 = pack_rne(x[2], x[3]);
                    const uint32_t l0 = pack_rest(x[0], x[1], h0), l1 = pack_rest(x[2], x[3], h1);
                    hh = as_v8h(h0, h1, h0, h1);
                    ll = as_v8h(l0, l1, l0, l1);
                };
                v8h xh[4], xl[4];   // s0, sr, 2 dn, -1.5 dn
                if constexpr (C == 3) {
                    v4f s0, sr, d2, d3;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float a0 = S[ht][0][r], b0 = S[ht][1][r], c0v = S[ht][2][r];
                        const float u = b0 + c0v;
                        s0[r] = a0 + u;
                        sr[r] = fmaf(2.f, a0, -u);
                        const float dn = b0 - c0v;
                        d2[r] = dn + dn;
                        d3[r] = -1.5f * dn;
                    }
                    split(s0, xh[0], xl[0]);
                    split(sr, xh[1], xl[1]);
                    split(d2, xh[2], xl[2]);
                    split(d3, xh[3], xl[3]);
                } else {
                    split(S[ht][0], xh[0], xl[0]);
                }
                // [hi | lo] of coefficients 4 gq + j against pixel n16 of set t; the operands of the next
                // set are loaded before the products of this one
                auto table_t = [&](int m, int t) {
                    const v4h *f = FT + m * 2 * Frag<C>::MAP + (ct * 2 + (t >> 1)) * 256 + (t & 1) * 64;
                    const v4h hi = lds_read_tr(f), lo = lds_read_tr(f + 128);
                    return __builtin_shufflevector(hi, lo, 0, 1, 2, 3, 4, 5, 6, 7);
                };
                v8h f[2][NM];
#pragma unroll
                for (int m = 0; m < NM; ++m) f[0][m] = table_t(m, 0);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    if (t < 3) {
#pragma unroll
                        for (int m = 0; m < NM; ++m) f[(t + 1) & 1][m] = table_t(m, t + 1);
                    }
                    const v8h (&ft)[NM] = f[t & 1];
                    out[0][t][ht] = mfma(xh[0], ft[0], out[0][t][ht]);
                    if constexpr (C == 3) {
                        out[1][t][ht] = mfma(xh[1], ft[1], out[1][t][ht]);
                        out[2][t][ht] = mfma(xh[3], ft[1], out[2][t][ht]);
                    }
                    out[0][t][ht] = mfma(xl[0], ft[0], out[0][t][ht]);
                    if constexpr (C == 3) {
                        out[1][t][ht] = mfma(xl[1], ft[1], out[1][t][ht]);
                        out[2][t][ht] = mfma(xl[3], ft[1], out[2][t][ht]);
                        out[1][t][ht] = mfma(xh[2], ft[2], out[1][t][ht]);
                        out[2][t][ht] = mfma(xh[1], ft[2], out[2][t][ht]);
                        out[1][t][ht] = mfma(xl[2], ft[2], out[1][t][ht]);
                        out[2][t][ht] = mfma(xl[1], ft[2], out[2][t][ht]);
                    }
                }
            }
        }

        // ---- 5: inverse Haar and aggregation, one pixel set (16 pixels) at a time ----
        const v8h hi0 = L.H[128 + lane], hi1 = L.H[192 + lane];
        int offs[2][4];   // patches 16 mt + 4 gq + r: word of this lane's pixel of set 0
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            const int4 o4 = *reinterpret_cast<const int4 *>(&ws.off[16 * mt + 4 * gq]);
            const int lp = GA == 1 ? 0 : (n16 >> 1) * rp + 4 * (n16 & 1);
            offs[mt][0] = o4.x + lp;
            offs[mt][1] = o4.y + lp;
            offs[mt][2] = o4.z + lp;
            offs[mt][3] = o4.w + lp;
            if constexpr (GA != 1)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    offs[mt][r] *= C;
                    asm volatile("" : "+v"(offs[mt][r]));   // computed once, not per pixel set
                }
        }
        if (base + MW * G < nref) fetch(lin_next, lane);
        uint32_t skip = 0;   // patches (bit 4 mt + r) of groups past the tile's last
        if (!full) {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                skip |= (uint32_t)(base + ((16 * (i >> 2) + 4 * gq + (i & 3)) >> lk) >= nref) << i;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            v4f px[C][2];   // R, G, B: [patch tile], patches 4 gq + r
#pragma unroll
            for (int ht = 0; ht < 2; ++ht)
                if constexpr (C == 3) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float p0 = out[0][t][ht][r], pr = out[1][t][ht][r], pi = out[2][t][ht][r];
                        const float t0 = fmaf(-0.5f, pr, p0);   // pr is twice the real part
                        out[0][t][ht][r] = p0 + pr;
                        out[1][t][ht][r] = t0 - pi;
                        out[2][t][ht][r] = t0 + pi;
                    }
                }
#pragma unroll
            for (int ch = 0; ch < C; ++ch) {
                const v4f a = out[ch][t][0], b = out[ch][t][1];
                const uint32_t h0 = pack_rne(a[0], a[1]), h1 = pack_rne(a[2], a[3]);
                const uint32_t h2 = pack_rne(b[0], b[1]), h3 = pack_rne(b[2], b[3]);
                const v8h xh = as_v8h(h0, h1, h2, h3);
                const v8h xl = as_v8h(pack_rest(a[0], a[1], h0), pack_rest(a[2], a[3], h1), pack_rest(b[0], b[1], h2),
                                      pack_rest(b[2], b[3], h3));
                const v4f zero = {0.f, 0.f, 0.f, 0.f};
                px[ch][0] = mfma(hi0, xl, mfma(hi0, xh, zero));
                px[ch][1] = mfma(hi1, xl, mfma(hi1, xh, zero));
            }
            if constexpr (GA == 1) {   // kept for the loop below, in the place of the rows
#pragma unroll
                for (int ch = 0; ch < C; ++ch) {
                    out[ch][t][0] = px[ch][0];
                    out[ch][t][1] = px[ch][1];
                }
                continue;
            }
            auto add = [&](int i) {
                const int mt = i >> 2, r = i & 3;
#pragma unroll
                for (int ch = 0; ch < C; ++ch) {
                    if constexpr (GA == 2)
                        atomicAdd(iregion + offs[mt][r] + (t * C + ch), to_fixed(px[ch][mt][r], fscale));
                    else
                        atomicAdd(iregion + offs[mt][r] + (t * C + ch), (int)to_fixed_biased(px[ch][mt][r], fscale));
                }
            };
            if (full) {
#pragma unroll
                for (int i = 0; i < 8; ++i) add(i);
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (!((skip >> i) & 1u)) add(i);
            }
        }
        if constexpr (GA == 1) {
            // Four patches at a time through LDS, so that an atomic instruction adds to whole rows of one
            // patch (64 C words = C instructions; every 8 pixels are 64 C consecutive bytes).  From the
            // registers its lanes would reach 64 rows apart: 20 gray 128 x 128 frames, radius 10, K 32,
            // 1,511 us instead of 505, ten 200 x 300 RGB frames, radius 3, 9.99 ms instead of 1.83.
            int *stage = iregion + wave * 256 * C;
            int po[C];   // this lane's pixel of word lane + 64 j of a patch
#pragma unroll
            for (int j = 0; j < C; ++j) {
                const int wp = (lane + 64 * j) / C;
                po[j] = (wp >> 3) * rp + (wp & 7);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int mt = i >> 2, r = i & 3;
                wave_lds_fence();   // the words before were read
#pragma unroll
                for (int k = 0; k < C; ++k) {
                    int4 v;
                    v.x = to_fixed(out[(4 * k) % C][(4 * k) / C][mt][r], fscale);
                    v.y = to_fixed(out[(4 * k + 1) % C][(4 * k + 1) / C][mt][r], fscale);
                    v.z = to_fixed(out[(4 * k + 2) % C][(4 * k + 2) / C][mt][r], fscale);
                    v.w = to_fixed(out[(4 * k + 3) % C][(4 * k + 3) / C][mt][r], fscale);
                    *reinterpret_cast<int4 *>(stage + (64 * gq + 4 * n16) * C + 4 * k) = v;
                }
                wave_lds_fence();
#pragma unroll
                for (int gp = 0; gp < 4; ++gp) {
                    if (!full && base + ((16 * mt + 4 * gp + r) >> lk) >= nref) continue;   // past the tile's last
                    const int o = __builtin_amdgcn_readlane(offs[mt][r], 16 * gp);
#pragma unroll
                    for (int j = 0; j < C; ++j)
                        atomicAdd(gacc + (int64_t)(o + po[j]) * C + (lane + 64 * j) % C,
                                  (unsigned long long)(long long)stage[64 * C * gp + lane + 64 * j]);
                }
            }
        }
    }
    if constexpr (GA == 1) return;   // the caller's barrier follows
    if constexpr (GA == 2) {
        // the slot region to the tile's own slot of the global region buffer (plain stores; the
        // gather kernel sums the regions covering each pixel)
        __syncthreads();
        int4 *dst = reinterpret_cast<int4 *>(reinterpret_cast<int *>(gacc) + (int64_t)tile * C * plane);
        const int4 *src = reinterpret_cast<const int4 *>(iregion);
        for (int e = tid; e < C * plane / 4; e += MW * 64) dst[e] = src[e];
        return;   // the caller's barrier follows
    }
    __syncthreads();
    // coverage count of every pixel: 8 x 8 box sum of the patch histogram (separable, in place,
    // one row then one column per thread; prev[] holds the histogram values leaving the window)
    for (int y = tid; y < tg.RH; y += MW * 64) {
        int *row = hist + y * tg.RP;
        int prev[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        int run = 0;
        for (int x0 = 0; x0 < tg.RW; x0 += 8) {
            int cur[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) cur[i] = x0 + i < tg.RW ? row[x0 + i] : 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                run += cur[i] - prev[i];
                if (x0 + i < tg.RW) row[x0 + i] = run;
                prev[i] = cur[i];
            }
        }
    }
    __syncthreads();
    for (int x = tid; x < tg.RW; x += MW * 64) {
        int prev[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        int run = 0;
        for (int y0 = 0; y0 < tg.RH; y0 += 8) {
            int cur[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) cur[i] = y0 + i < tg.RH ? hist[(y0 + i) * tg.RP + x] : 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                run += cur[i] - prev[i];
                if (y0 + i < tg.RH) hist[(y0 + i) * tg.RP + x] = run;
                prev[i] = cur[i];
            }
        }
    }
    __syncthreads();
    // sums (the bits of MAGIC taken out once per contribution), then counts
    float *dst = regions + (int64_t)tile * relems;
    const float unscale = 1.f / fscale;
    for (int e = tid; e < plane; e += MW * 64) {
        const int cnt = hist[e];
#pragma unroll
        for (int ch = 0; ch < C; ++ch)
            dst[e * C + ch] = (float)(int)((uint32_t)iregion[e * C + ch] - (uint32_t)cnt * MAGIC_BITS) * unscale;
        dst[C * plane + e] = (float)cnt;
    }
}

// Persistent over the tiles of one image: workgroup b takes tiles b, b + grid, ... in an
// XCD-aware order (consecutive ids go round-robin over the 8 XCDs; with grid a multiple of 8
// each workgroup stays in one class, whose tiles form a contiguous run).
template <int C, bool RA>
__global__ __launch_bounds__(MW * 64) void filter_mfma_kernel(ImageGeom g, TileGeom tg, int K,
                                                             const v8h *__restrict__ F,
                                                             const double *__restrict__ T64,
                                                             const int32_t *__restrict__ idx,
                                                             const double *__restrict__ tau_ref,
                                                             float *__restrict__ regions,
                                                             unsigned long long *__restrict__ guard_count,
                                                             const float *__restrict__ ra_d,
                                                             const uint8_t *__restrict__ ra_flag) {
    extern __shared__ __align__(16) float smem[];
    __shared__ MfmaShared sh;
    const FilterLds<C> L = filter_lds_init<C>(smem, F, K);
    __syncthreads();
    const int n_tiles = tg.tiles_y * tg.tiles_x;
    const int per = (n_tiles + 7) / 8;
    for (int v = blockIdx.x; v < 8 * per; v += gridDim.x) {
        const int tile = (v & 7) * per + (v >> 3);
        if (tile >= n_tiles) continue;
        filter_tile_mfma<C, RA>(g, tg, L, T64, K, idx, K, tau_ref, 1.0, regions, guard_count, tile, sh, ra_d,
                                ra_flag);
        __syncthreads();
    }
}

// Groups anywhere in the image (video), global aggregation: GA == 1 the tiles only schedule the
// work; GA == 2 each tile also has its slot region.
template <int C, bool RA, int GA>
__global__ __launch_bounds__(MW * 64) void filter_mfma_ga_kernel(ImageGeom g, TileGeom tg, VideoTiling vt, int K,
                                                                const v8h *__restrict__ F,
                                                                const double *__restrict__ T64,
                                                                const int32_t *__restrict__ idx,
                                                                const double *__restrict__ tau_ref,
                                                                unsigned long long *__restrict__ gacc,
                                                                int *__restrict__ ghist,
                                                                unsigned long long *__restrict__ guard_count,
                                                                const float *__restrict__ ra_d,
                                                                const uint8_t *__restrict__ ra_flag) {
    extern __shared__ __align__(16) float smem[];
    __shared__ MfmaShared sh;
    const FilterLds<C> L = filter_lds_init<C>(smem, F, K);
    __syncthreads();
    const int n_tiles = tg.tiles_y * tg.tiles_x;
    const int per = (n_tiles + 7) / 8;   // XCD-aware order, as in filter_mfma_kernel
    for (int v = blockIdx.x; v < 8 * per; v += gridDim.x) {
        const int tile = (v & 7) * per + (v >> 3);
        if (tile >= n_tiles) continue;
        filter_tile_mfma<C, RA, GA>(g, tg, L, T64, K, idx, K, tau_ref, 1.0, nullptr, guard_count, tile, sh, ra_d,
                                    ra_flag, gacc, ghist, vt);
        __syncthreads();
    }
}

// out = sum / (count 2^fs), count = 8 x 8 box sum of the patch histogram; the noisy value
// where no patch landed.
template <int C>
__global__ void ga_normalize_kernel(const unsigned long long *__restrict__ gacc, const int *__restrict__ ghist,
                                    const uint8_t *__restrict__ img, int64_t stride, int h, int w, int fs,
                                    float *__restrict__ out, int64_t out_stride) {
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e >= (int64_t)h * w) return;
    const int y = (int)(e / w), x = (int)(e % w);
    int n = 0;
    for (int dy = 0; dy < PS && dy <= y; ++dy)
        for (int dx = 0; dx < PS && dx <= x; ++dx) n += ghist[(int64_t)(y - dy) * w + (x - dx)];
    float *o = out + (int64_t)y * out_stride + (int64_t)x * C;
    const uint8_t *px = img + (int64_t)y * stride + (int64_t)x * C;
    const double inv = n > 0 ? 1.0 / ((double)n * (double)(1 << fs)) : 0.0;
#pragma unroll
    for (int ch = 0; ch < C; ++ch)
        o[ch] = n > 0 ? (float)((double)(long long)gacc[e * C + ch] * inv) : (float)px[ch];
}

// Patches covering each pixel of a 64 x 4 tile at (Y0, x0) of a hh x w image, from the patches by
// top-left pixel: 8 x 8 box sums, separable, in LDS (256 threads; 64 loads per pixel took most of the
// 229 us of the gather of four 720 x 1280 frames, 112 us so).  Thread t gets the count of pixel
// (Y0 + t / 64, x0 + t % 64).  Tiles of 16 rows, 4 pixels to a thread, load less around them, but a
// pixel's sum over its regions waits for memory at every one, and small frames then have too few threads:
// four 150 x 200 frames 41 us so and 16 with 4 rows (24 with the 64 loads), three of 70 x 70 at step 1
// 250 and 71 (68); four of 720 x 1280 the same.
constexpr int BOX_W = 64, BOX_H = 4;
struct BoxShared {
    int hist[BOX_H + PS - 1][BOX_W + PS - 1];
    int row[BOX_H + PS - 1][BOX_W];
};
__device__ __forceinline__ int box_count(BoxShared &sh, const int *__restrict__ ghist, int hh, int w, int Y0, int x0) {
    constexpr int RW = BOX_W + PS - 1, RH = BOX_H + PS - 1;
    for (int t = threadIdx.x; t < RH * RW; t += 256) {
        const int r = t / RW, c = t - r * RW, Y = Y0 - (PS - 1) + r, x = x0 - (PS - 1) + c;
        sh.hist[r][c] = Y >= 0 && Y < hh && x >= 0 && x < w ? ghist[(int64_t)Y * w + x] : 0;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < RH * BOX_W; t += 256) {
        const int r = t / BOX_W, c = t % BOX_W;
        int a = 0;
#pragma unroll
        for (int d = 0; d < PS; ++d) a += sh.hist[r][c + d];
        sh.row[r][c] = a;
    }
    __syncthreads();
    int a = 0;
#pragma unroll
    for (int d = 0; d < PS; ++d) a += sh.row[(threadIdx.x >> 6) + d][threadIdx.x & 63];
    return a;
}

// Slot regions (GA == 2): pixel (f, y, x) of the stacked frames sums, over the frames t within
// the radius of f, the regions of frame t's tiles that cover (y, x) at f's slot; the count is
// the 8 x 8 box sum of the patch histogram.  out = sum / (count 2^fs), or the noisy value.
template <int C>
__global__ void ga_gather_kernel(const int *__restrict__ regions, TileGeom tg, VideoTiling vt, int s, int nx,
                                 const int *__restrict__ ghist, const uint8_t *__restrict__ img, int64_t stride,
                                 int w, int box0, float *__restrict__ out, int64_t out_stride) {
    __shared__ BoxShared sh;
    const int hh = vt.T * vt.h_frame, tiles = (w + BOX_W - 1) / BOX_W;
    const int box = box0 + (int)blockIdx.x, Y0 = box / tiles * BOX_H, x0 = box % tiles * BOX_W;
    const int n = box_count(sh, ghist, hh, w, Y0, x0);
    const int Y = Y0 + (threadIdx.x >> 6), x = x0 + (threadIdx.x & 63);
    if (Y >= hh || x >= w) return;
    const int f = Y / vt.h_frame, y = Y - f * vt.h_frame;
    float *o = out + (int64_t)Y * out_stride + (int64_t)x * C;
    const uint8_t *px = img + (int64_t)Y * stride + (int64_t)x * C;
    if (n == 0) {
#pragma unroll
        for (int ch = 0; ch < C; ++ch) o[ch] = (float)px[ch];
        return;
    }
    const int plane = region_plane(tg);
    const int tyf = (vt.ny_frame + tg.TY - 1) / tg.TY;
    const int span_y = tg.TY * s, span_x = tg.TX * s;
    // tiles whose region rows r0 .. r0 + RH - 1 can hold y: r0 = max(0, first reference row - R), and
    // the windows end R + 7 past the last reference (RH, which ends at the frame, says less: a tile
    // whose r0 is 0 may reach every row of a small frame)
    const int ty_hi = min(tyf - 1, (y + tg.R) / span_y + 1), ty_lo = max(0, (y - tg.R - PS - span_y) / span_y - 1);
    const int tx_hi = min(tg.tiles_x - 1, (x + tg.R) / span_x + 1), tx_lo = max(0, (x - tg.R - PS - span_x) / span_x - 1);
    long long acc[C];
#pragma unroll
    for (int ch = 0; ch < C; ++ch) acc[ch] = 0;
    for (int t = max(0, f - vt.radius); t <= min(vt.T - 1, f + vt.radius); ++t) {
        const int slot = f - max(0, t - vt.radius);
        for (int tyl = ty_lo; tyl <= ty_hi; ++tyl) {
            const int r0 = max(0, ref_pos(tyl * tg.TY, vt.ny_frame, vt.h_frame, s) - tg.R);
            if (y < r0 || y >= r0 + vt.RH) continue;
            for (int tx = tx_lo; tx <= tx_hi; ++tx) {
                const int c0 = max(0, ref_pos(tx * tg.TX, nx, w, s) - tg.R);
                if (x < c0 || x >= c0 + vt.RW) continue;
                const int *src = regions + ((int64_t)(t * tyf + tyl) * tg.tiles_x + tx) * C * plane +
                                 ((slot * vt.RH + (y - r0)) * tg.RP + (x - c0)) * C;
#pragma unroll
                for (int ch = 0; ch < C; ++ch) acc[ch] += src[ch];
            }
        }
    }
    const double inv = 1.0 / ((double)n * (double)(1 << tg.FS));
#pragma unroll
    for (int ch = 0; ch < C; ++ch) o[ch] = (float)((double)acc[ch] * inv);
}

template <int C>
__global__ __launch_bounds__(MW * 64) void filter_mfma_kernel_batched(const BatchItem *__restrict__ items, int K,
                                                                     int n_items, const int *__restrict__ unit_start,
                                                                     const v8h *__restrict__ F,
                                                                     const double *__restrict__ T64,
                                                                     unsigned long long *__restrict__ guard_count,
                                                                     int *__restrict__ queue) {
    extern __shared__ __align__(16) float smem[];
    __shared__ MfmaShared sh;
    __shared__ int s_u;
    const FilterLds<C> L = filter_lds_init<C>(smem, F, K);
    __syncthreads();
    const int total = unit_start[n_items];
    for (;;) {
        // thread 0 claims the next unit of an image filtered with this group size; units of an
        // image that took the other size are skipped by moving the queue past the image's end
        // (every value below the end that the queue then skips is one of its units).  The skip
        // loop holds no barrier, so the block's barriers below stay on uniform paths.
        if (threadIdx.x == 0) {
            int c;
            for (;;) {
                c = atomicAdd(queue, 1);
                if (c >= total) break;
                const int ic = find_unit(unit_start, n_items, c);
                const int *ks = items[ic].ksel;
                if (!ks || *ks == K) break;
                atomicMax(queue, unit_start[ic + 1]);
            }
            s_u = c;
        }
        __syncthreads();
        const int u = s_u;
        __syncthreads();
        if (u >= total) break;
        const int i = find_unit(unit_start, n_items, u);
        const BatchItem it = items[i];
        filter_tile_mfma<C>(it.g, it.tg, L, T64, K, it.idx, it.idx_stride, it.tau, it.tau_mul, it.regions,
                            guard_count, u - unit_start[i], sh);
        __syncthreads();
    }
}

}  // namespace

int filter_mfma_group_bytes(int C) { return C == 3 ? fixed_lds_bytes<3>() : fixed_lds_bytes<1>(); }

int filter_mfma_lds_bytes(const TileGeom &tg, int C) { return filter_mfma_group_bytes(C) + region_elems(tg, C) * 4; }

size_t filter_mfma_table_halves(int C) { return (size_t)(C == 3 ? 3 : 1) * Frag<1>::MAP * 8; }

// Fills the operand tables from the FP64 maps fwd and inv (64 C x 64 C, row-major; the forward map
// of (a0, ar, ai) to (s0', re', im') and its inverse on (s0, sr, d)), h16 rounding to fp16 bits and
// h16v giving their value.  Returns false if the maps have not the structure the kernel relies on:
// slice 0 apart, re' = A ar + B ai, im' = -B ar + 3 A ai, and the inverse its transpose.
bool filter_mfma_tables(int C, const double *fwd, const double *inv, uint16_t (*h16)(double), double (*h16v)(uint16_t),
                        uint16_t *out) {
    const int P = 64 * C, NM = C == 3 ? 3 : 1;
    auto F = [&](int n, int k) { return fwd[(size_t)n * P + k]; };
    auto I = [&](int n, int k) { return inv[(size_t)n * P + k]; };
    auto far = [](double a, double b) { return !(fabs(a - b) <= 1e-12); };
    if (C == 3)
        for (int n = 0; n < 64; ++n)
            for (int k = 0; k < 64; ++k) {
                for (int a = 1; a < 3; ++a)
                    if (far(F(n, 64 * a + k), 0) || far(F(64 * a + n, k), 0)) return false;
                if (far(F(128 + n, 64 + k), -F(64 + n, 128 + k)) || far(F(128 + n, 128 + k), 3 * F(64 + n, 64 + k)))
                    return false;
            }
    // the inverse is the transposed forward map, so the kernel reads one table both ways
    for (int n = 0; n < P; ++n)
        for (int k = 0; k < P; ++k)
            if (far(F(n, k), I(k, n))) return false;
    auto map = [&](int m, int n, int k) {   // p = ar / 2 doubles A
        return m == 0 ? F(n, k) : (m == 1 ? 2 * F(64 + n, 64 + k) : F(64 + n, 128 + k));
    };
    uint16_t *o = out;
    for (int m = 0; m < NM; ++m)
        for (int ct = 0; ct < 4; ++ct)
            for (int s = 0; s < 2; ++s)
                for (int term = 0; term < 2; ++term)
                    for (int q = 2 * s; q < 2 * s + 2; ++q)
                        for (int l = 0; l < 64; ++l)
                            for (int j = 0; j < 4; ++j) {
                                const int px = 4 * (l >> 4) + j;   // of set q
                                const double v = map(m, 16 * ct + (l & 15), 8 * (px >> 1) + 4 * (px & 1) + q);
                                const uint16_t hi = h16(v);
                                *o++ = term == 0 ? hi : h16(v - h16v(hi));
                            }
    return true;
}

int filter_mfma_static_bytes() { return (int)sizeof(MfmaShared) + 16; }

template <int C, bool RA>
static hipError_t launch_mfma_t(const ImageGeom &g, const TileGeom &tg, int K, const BasisDev &b, const int32_t *idx,
                                const double *tau_ref, float *regions, unsigned long long *gc, const float *ra_d,
                                const uint8_t *ra_flag, hipStream_t st) {
    const int n_tiles = tg.tiles_y * tg.tiles_x;
    const int lds = filter_mfma_lds_bytes(tg, C);
    hipError_t e = prepare_dynamic_lds((const void *)filter_mfma_kernel<C, RA>, lds, (int)sizeof(MfmaShared));
    if (e != hipSuccess) return e;
    int dev = 0, n_cu = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
    if (n_cu < 8) n_cu = 8;
    const int per = (n_tiles + 7) / 8;
    const int grid = min(8 * per, (n_cu / 8) * 8);
    hipLaunchKernelGGL((filter_mfma_kernel<C, RA>), dim3(grid), dim3(MW * 64), lds, st, g, tg, K, (const v8h *)b.frag,
                       b.T64, idx, tau_ref, regions, gc, ra_d, ra_flag);
    return hipGetLastError();
}

hipError_t launch_filter_mfma(const ImageGeom &g, const TileGeom &tg, int K, const BasisDev &b, const int32_t *idx,
                              const double *tau_ref, float *regions, unsigned long long *gc, hipStream_t st,
                              const float *ra_d, const uint8_t *ra_flag) {
    if (!b.frag || !(K == 4 || K == 8 || K == 16 || K == 32)) return hipErrorInvalidValue;
    if (g.c == 3)
        return ra_d ? launch_mfma_t<3, true>(g, tg, K, b, idx, tau_ref, regions, gc, ra_d, ra_flag, st)
                    : launch_mfma_t<3, false>(g, tg, K, b, idx, tau_ref, regions, gc, nullptr, nullptr, st);
    if (g.c == 1)
        return ra_d ? launch_mfma_t<1, true>(g, tg, K, b, idx, tau_ref, regions, gc, ra_d, ra_flag, st)
                    : launch_mfma_t<1, false>(g, tg, K, b, idx, tau_ref, regions, gc, nullptr, nullptr, st);
    return hipErrorInvalidValue;
}

template <int C, bool RA, int GA>
static hipError_t launch_mfma_ga_t(const ImageGeom &g, const TileGeom &tg, const VideoTiling &vt, int K, int lds,
                                   const BasisDev &b, const int32_t *idx, const double *tau_ref,
                                   unsigned long long *gacc, int *ghist, unsigned long long *gc, const float *ra_d,
                                   const uint8_t *ra_flag, hipStream_t st) {
    const int n_tiles = tg.tiles_y * tg.tiles_x;
    hipError_t e = prepare_dynamic_lds((const void *)filter_mfma_ga_kernel<C, RA, GA>, lds, (int)sizeof(MfmaShared));
    if (e != hipSuccess) return e;
    int dev = 0, n_cu = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
    if (n_cu < 8) n_cu = 8;
    const int per = (n_tiles + 7) / 8;
    const int grid = min(8 * per, (n_cu / 8) * 8);
    hipLaunchKernelGGL((filter_mfma_ga_kernel<C, RA, GA>), dim3(grid), dim3(MW * 64), lds, st, g, tg, vt, K,
                       (const v8h *)b.frag, b.T64, idx, tau_ref, gacc, ghist, gc, ra_d, ra_flag);
    return hipGetLastError();
}

// Largest fixed-point shift (<= GA_FS) for slot regions of side x side references of K members.
static int ga_shift(int side, int K) {
    int fs = GA_FS;
    while (fs > 0 && (double)side * side * K * 1024.0 * (double)(1 << fs) >= 2147483647.0) --fs;
    return fs;
}

// Shift that slot regions keep at least: that of the largest tile whose slots, rows padded to 8 modulo 16
// words, fit in LDS beside 65 KB (or of the sums in memory where none does), whatever side the estimated
// time would take.
static int ga_least_shift(int C, int K, int h_frame, int w, int s, int R, int nslot) {
    for (int side = GA_MAX_TILE; side >= 1; --side) {
        const int reach = (side - 1) * s + 2 * R + PS;
        if (ga_shift(side, K) >= GA_PADDED_MIN_FS && padded_region_fits(C, nslot * min(reach, h_frame), min(reach, w)))
            return max(GA_MIN_FS, ga_shift(side, K));
    }
    return GA_FS;
}

// Tiling of the video filter: the tile side (<= GA_MAX_TILE) with the lowest estimated time among
// those whose fixed-point shift is at least ga_least_shift and whose slot region fits in LDS beside the
// tables; 0 where the sums straight to memory are estimated to take less.  Besides the filter and the
// regions' way to memory (as for one image): the gather reads 300 region pixels per nanosecond, but a
// thread waits some 0.7 us at each of its own; sums in memory take 118 values per nanosecond (RGB) or 78
// (gray), one pixel's about 0.3 us each, and two launches more.  Measured with either forced, filter and
// gather: six 200 x 300 RGB frames, radius 2, window 31, K 32: 2,096 us with single references to a region
// (2.1 GB), 1,168 without; twenty 128 x 128 gray frames, radius 10: 2,376 (2.5 GB) and 518; ten 200 x 300
// RGB frames, radius 3, window 21, K 32: 930 (2 x 2) and 1,856; four 720 x 1280 RGB frames, radius 1: 1,953
// (7 x 7) and 11,944.
static int video_tile_side(int C, int K, int T, int ny_frame, int nx, int h_frame, int w, int s, int W, int nslot,
                           VideoTiling *vt) {
    const int R = (W - 1) / 2;
    const int least = ga_least_shift(C, K, h_frame, w, s, R, nslot);
    const double pixels = (double)T * h_frame * w, added = (double)T * ny_frame * nx * K * 64;
    const int64_t units = (int64_t)((T * ny_frame + GA_MAX_TILE - 1) / GA_MAX_TILE) * ((nx + GA_MAX_TILE - 1) / GA_MAX_TILE);
    int best = 0;
    double best_cost = 10.0 + std::max({C == 3 ? added * 3 / 118e3 : added / 78e3, 0.3 * added / pixels,
                                        filter_tiles_cost(C, K, units, GA_MAX_TILE * GA_MAX_TILE, 1.0)});
    for (int side = 1; side <= GA_MAX_TILE; ++side) {
        const int RH = min((side - 1) * s + 2 * R + PS, h_frame), RW = min((side - 1) * s + 2 * R + PS, w);
        const int RP = region_pitch(RW);
        const int64_t bytes = filter_mfma_group_bytes(C) + (int64_t)C * (((int64_t)nslot * RH * RP + 3) & ~3) * 4;
        if (ga_shift(side, K) < least || bytes > filter_lds_budget()) break;
        const int64_t n_tiles = (int64_t)T * ((ny_frame + side - 1) / side) * ((nx + side - 1) / side);
        const double visits = (double)n_tiles * nslot * RH * RW;
        const double cost = filter_tiles_cost(C, K, n_tiles, side * side, 1.0) +
                            (double)n_tiles * nslot * RH * RP * C * 4 / 2.5e6 +
                            std::max(visits / 300e3, 0.7 * visits / pixels);
        if (cost <= best_cost) {
            best = side;
            best_cost = cost;
            vt->RH = RH;
            vt->RW = RW;
            vt->RP = RP;
        }
    }
    return best;
}

// Plan of the video filter: frame-aligned tiles with slot regions (side > 0), or the direct
// global sums (side 0).
static int plan_video(const ImageGeom &g, int T, int radius, int W, int K, bool force_direct, VideoTiling *vt,
                      TileGeom *tg) {
    vt->T = T;
    vt->h_frame = g.h / T;
    vt->ny_frame = g.ny / T;
    vt->radius = radius;
    vt->nslot = min(2 * radius + 1, T);
    const int side = force_direct ? 0 : video_tile_side(g.c, K, T, vt->ny_frame, g.nx, vt->h_frame, g.w, g.s, W, vt->nslot,
                                                        vt);
    *tg = TileGeom{};
    tg->R = (W - 1) / 2;
    tg->FS = side > 0 ? ga_shift(side, K) : GA_FS;
    if (side > 0) {   // frame-aligned tiles with slot regions
        tg->TY = tg->TX = side;
        tg->tiles_y = T * ((vt->ny_frame + side - 1) / side);
        tg->tiles_x = (g.nx + side - 1) / side;
        tg->RH = vt->nslot * vt->RH;   // one plane per channel: the slots stacked
        tg->RW = vt->RW;
        tg->RP = vt->RP;
    } else {          // direct: 8 x 8 references of the stacked grid per scheduling unit
        tg->TY = tg->TX = GA_MAX_TILE;
        tg->tiles_y = (g.ny + tg->TY - 1) / tg->TY;
        tg->tiles_x = (g.nx + tg->TX - 1) / tg->TX;
    }
    return side;
}

// Bytes of the accumulation buffer of launch_filter_mfma_global: the tiles' slot regions, or
// the 64-bit global sums.
size_t filter_mfma_global_bytes(const ImageGeom &g, int T, int radius, int W, int K, bool force_direct) {
    if (T < 1 || g.h % T || g.ny % T) return 0;
    VideoTiling vt;
    TileGeom tg;
    const int side = plan_video(g, T, radius, W, K, force_direct, &vt, &tg);
    if (side > 0) return (size_t)tg.tiles_y * tg.tiles_x * g.c * region_plane(tg) * sizeof(int);
    return (size_t)g.h * g.w * g.c * sizeof(unsigned long long);
}

// Filtering of groups whose members lie anywhere in the frames of a video (T frames of g.h / T
// rows stacked vertically, reference grid T*ny x nx frame-major, members within `radius` frames
// of their reference's), then the normalisation.  accum: filter_mfma_global_bytes of scratch;
// ghist (h*w int32) must be zero on entry.  force_direct skips the slot regions.
hipError_t launch_filter_mfma_global(const ImageGeom &g, int T, int radius, int W, int K, const BasisDev &b,
                                     const int32_t *idx, const double *tau_ref, void *accum, int *ghist,
                                     unsigned long long *gc, float *out, int64_t out_stride, hipStream_t st,
                                     const float *ra_d, const uint8_t *ra_flag, bool force_direct) {
    if (!b.frag || T < 1 || g.h % T || g.ny % T || !(K == 4 || K == 8 || K == 16 || K == 32))
        return hipErrorInvalidValue;
    VideoTiling vt;
    TileGeom tg;
    const int side = plan_video(g, T, radius, W, K, force_direct, &vt, &tg);
    int lds = filter_mfma_group_bytes(g.c);
    unsigned long long *gacc = (unsigned long long *)accum;
    hipError_t e;
    lds += side > 0 ? g.c * region_plane(tg) * 4 : MW * 256 * g.c * 4;
    if (side == 0 && (e = launch_zero(accum, (size_t)g.h * g.w * g.c * sizeof(unsigned long long), st)) != hipSuccess)
        return e;
    e = hipErrorInvalidValue;
#define HG_CASE(CC, RR, GG) \
    launch_mfma_ga_t<CC, RR, GG>(g, tg, vt, K, lds, b, idx, tau_ref, gacc, ghist, gc, ra_d, ra_flag, st)
    if (g.c == 3)
        e = side > 0 ? (ra_d ? HG_CASE(3, true, 2) : HG_CASE(3, false, 2))
                     : (ra_d ? HG_CASE(3, true, 1) : HG_CASE(3, false, 1));
    else if (g.c == 1)
        e = side > 0 ? (ra_d ? HG_CASE(1, true, 2) : HG_CASE(1, false, 2))
                     : (ra_d ? HG_CASE(1, true, 1) : HG_CASE(1, false, 1));
#undef HG_CASE
    if (e != hipSuccess) return e;
    const int64_t n = (int64_t)g.h * g.w;
    const unsigned grid = (unsigned)((n + 255) / 256);
    if (side > 0) {
        const int n_box = ((g.w + BOX_W - 1) / BOX_W) * ((g.h + BOX_H - 1) / BOX_H);   // 2^25 at most (2^30 pixels)
        for (int b0 = 0; b0 < n_box; b0 += 1 << 23) {   // a launch has less than 2^32 threads
            const auto gather = g.c == 3 ? ga_gather_kernel<3> : ga_gather_kernel<1>;
            hipLaunchKernelGGL(gather, dim3((unsigned)min(n_box - b0, 1 << 23)), dim3(256), 0, st, (const int *)accum, tg,
                               vt, g.s, g.nx, ghist, g.img, g.stride, g.w, b0, out, out_stride);
        }
    } else if (g.c == 3) {
        hipLaunchKernelGGL(ga_normalize_kernel<3>, dim3(grid), dim3(256), 0, st, gacc, ghist, g.img, g.stride, g.h,
                           g.w, tg.FS, out, out_stride);
    } else {
        hipLaunchKernelGGL(ga_normalize_kernel<1>, dim3(grid), dim3(256), 0, st, gacc, ghist, g.img, g.stride, g.h,
                           g.w, tg.FS, out, out_stride);
    }
    return hipGetLastError();
}

template <int C>
static hipError_t launch_mfma_batched_t(int K, const BatchItem *items, int n_items, const int *unit_start, int lds,
                                        const BasisDev &b, unsigned long long *gc, int *queue, int grid,
                                        hipStream_t st) {
    hipError_t e = prepare_dynamic_lds((const void *)filter_mfma_kernel_batched<C>, lds,
                                       (int)sizeof(MfmaShared) + 16);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(filter_mfma_kernel_batched<C>, dim3(grid), dim3(MW * 64), lds, st, items, K, n_items,
                       unit_start, (const v8h *)b.frag, b.T64, gc, queue);
    return hipGetLastError();
}

hipError_t launch_filter_mfma_batched(int C, int K, const BatchItem *items, int n_items, const int *unit_start,
                                      int lds, const BasisDev &b, unsigned long long *gc, int *queue, int grid,
                                      hipStream_t st) {
    if (!b.frag || !(K == 4 || K == 8 || K == 16 || K == 32)) return hipErrorInvalidValue;
    if (C == 3) return launch_mfma_batched_t<3>(K, items, n_items, unit_start, lds, b, gc, queue, grid, st);
    if (C == 1) return launch_mfma_batched_t<1>(K, items, n_items, unit_start, lds, b, gc, queue, grid, st);
    return hipErrorInvalidValue;
}

}  // namespace htsvd
