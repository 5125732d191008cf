// Block matching (grouping) for Haar-tSVD on gfx950.
//
// Sec. III-A, Eq. 9: the distance between the reference patch and a candidate is the
// green-channel distance when gamma^2 ||G_ref||^2 >= max(||R_ref||^2, ||B_ref||^2), and the
// distance of the channel averages otherwise (here the channel sum: same order and ties).
// Distances are squared Euclidean and exact.  Algorithm 1 "Grouping" keeps the K
// smallest, ordered by (distance, row, column).
//
// Mapping.  One workgroup (16 waves) owns a 4x4 tile of references, or with windows past 640
// positions and steps up to 4 a 3x4 tile (12 waves), so that two workgroups share a CU.  The union of
// their search windows (at most 64x64 candidate positions) is staged in LDS as
//   - the shifted green (or gray) plane x-128 in int8, in 4 byte-shifted copies so any
//     8-pixel row segment is a 4-byte-aligned pair of dwords, and
//   - the shifted channel-sum plane R+G+B-384 in fp16 (exact: |v| <= 384), in 2 copies.
// ||a-b||^2 = ||a||^2 + ||b||^2 - 2 a.b, where a.b for 16 references x 16 candidates is one
// v_mfma_i32_16x16x64_i8 (one 8x8 patch = the whole k = 64 contraction), or two
// v_mfma_f32_16x16x32_f16 for the sum plane (all partial sums are integers < 2^24, so the
// fp32 accumulation is exact).  Distances of each reference land in an LDS table indexed
// by the raster position inside its clipped window, so (distance, position) orders like
// (distance, row, column).  Each wave then selects the K smallest keys of one reference: the
// larger of the (K/2)-th smallest lane minima of its two halves bounds the answer from above, the
// keys under that bound are compacted and sorted with a wave bitonic network.
//
// It is bound by vector instructions, so the work per candidate is kept to few: in the distance
// phase a wave takes a fixed block of columns and steps through the rows, so that addresses advance
// by constants and a window's columns are tested once, and the keys sorted are 32 bits wide
// wherever their range allows: 12 MP, step 3, window 31, noise known, 4.70 -> 4.20 ms (when both sides of
// each window were tested per reference and position, the keys were counted before they were
// compacted, and channel sums took 64-bit keys).  The waits at the barriers between a tile's phases are
// filled by a second workgroup on the CU: 3.44 ms.  With it vector instructions are active in 88% of the
// cycles, 1,649 per reference (noise 50, 12 references to a tile).  The kernels are compiled for windows of up to 256, 448, 640 and 961 positions (the
// windows of all frames of a video also for up to 704: window 15 in three frames), so that
// small windows neither walk empty table rows nor hold LDS for them: 1536 x 2048 gray, window 21,
// 560 -> 423 us; four 720 x 1280 frames with window 15, 2,505 -> 981 us.
//
// Video (Sec. IV-C): the frames are stacked vertically, and a reference's candidates are the
// positions of its clipped window in every frame within a temporal radius.  The workgroup keeps
// the reference patches of its own frame in registers and stages one frame after another.  Where
// a row of the table holds the windows of all frames, position frame slot x window + place, a
// reference selects once at the end; else each frame's K best (distance, frame slot, position) keys
// are merged into a running list in LDS.
#include <algorithm>

#include "common.h"

namespace htsvd {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

namespace {

constexpr int NREF = REF_TILE * REF_TILE;  // 16
constexpr int BMW = 16;                    // wavefronts per workgroup (four per SIMD)
constexpr int BMT = BMW * 64;
constexpr int RUN_K = 32;                  // running list per reference of the video search
// Words per reference row of the distance table for windows of at most 64 NPL positions: 4 (mod
// 64), so the four references a quarter-wave writes for 16 consecutive candidates land on disjoint
// LDS banks.  Once in registers, a row gives its place to the compacted keys: at most RUN_K lanes
// hold keys under an exact bound, with at most NPL keys each (of 961 positions only lane 0 has 16),
// so the row holds them as 64-bit keys.
template <int NPL>
__host__ __device__ constexpr int tab_stride() { return NPL == 16 ? 964 : 64 * NPL + 4; }
static_assert(tab_stride<16>() >= MAX_CAND && tab_stride<16>() >= 2 * (15 * RUN_K + 1), "a whole window");
static_assert(tab_stride<4>() >= 2 * 4 * RUN_K && tab_stride<7>() >= 2 * 7 * RUN_K && tab_stride<10>() >= 2 * 10 * RUN_K,
              "the keys under the bound");

// Frames of a video search: g.img is frame 0 of T frames of g.h rows each, frame_bytes apart.
struct VideoArgs {
    int T, radius;
    int64_t frame_bytes;
};

struct TileInfo {
    int ry[NREF], rx[NREF];        // reference position, ry = -1 if the slot is empty
    int wy0[NREF], wx0[NREF];      // clipped window origin (candidate positions)
    int wh[NREF], ww[NREF];        // clipped window size
    int green[NREF];               // Eq. 9 branch: 1 green/gray distance, 0 channel-sum distance
    int any_sum;                   // some reference uses the channel-sum distance
};

// Byte layout of the dynamic LDS for one launch.
struct BmLds {
    int pitch8;     // bytes per row of one int8 plane copy
    int pitch16;    // halves per row of one fp16 plane copy
    int rows;       // plane rows (union rows + 7)
    int plane8;     // bytes between the int8 plane copies (a row multiple plus a bank offset)
    int off_p8, off_p16, off_n8, off_n16, off_tab, off_rs, total;   // video: running lists last
};

__device__ inline uint32_t lds_u32(const unsigned char *base, int byte_off) {
    return *reinterpret_cast<const uint32_t *>(base + byte_off);
}

__device__ inline void wave_lds_sync() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

__device__ inline uint64_t readlane_u64(uint64_t v, int l) {
    uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, l);
    uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}

// Ascending sort of one u64 per lane across the 64 lanes of a wave.
__device__ inline uint64_t wave_sort64(uint64_t v, int lane) { return wave_sort_asc<uint64_t>(v, lane); }

// Ascending bitonic sort of n keys in LDS by one wave, in the form whose comparators are all
// ascending (see wave_sort_asc), so that the places from n to the next power of two can be taken as
// larger than any key without existing.
template <typename T>
__device__ void lds_sort(T *a, int n, int lane) {
    for (int k = 2; k < 2 * n; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int t = lane; 2 * t < 2 * n; t += 64) {   // pairs beyond n have no upper element
                const int i = ((t & ~(j - 1)) << 1) | (t & (j - 1));
                const int m = j == k >> 1 ? i ^ (k - 1) : i + j;
                if (i < n && m < n) {
                    const T x = a[i], y = a[m];
                    if (y < x) {
                        a[i] = y;
                        a[m] = x;
                    }
                }
            }
            wave_lds_sync();
        }
}

// Sort across each half of the wave (two independent sorts of 32 keys).
__device__ inline uint32_t half_sort_asc(uint32_t v, int lane) {
#pragma unroll
    for (int k = 2; k <= 32; k <<= 1) {
        {
            const uint32_t p = mirror_lane(v, k, lane);
            v = (lane & (k >> 1)) ? max(v, p) : min(v, p);
        }
#pragma unroll
        for (int j = k >> 2; j > 0; j >>= 1) {
            const uint32_t p = xor_lane(v, j, lane);
            v = (lane & j) ? max(v, p) : min(v, p);
        }
    }
    return v;
}

// Number of set bits of m below this lane.
__device__ inline int bits_below(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// The K smallest (distance, position) keys d << 10 | p of a row of n distances dv (position lane +
// 64 i in register i, 0xFFFFFFFF past n), ascending, lane k the k-th.  `row` is the reference's LDS
// row (its distances are in registers).  small: distances below 2^22 (green or gray), whose keys
// fit 32 bits; otherwise (channel sum, below 2^26) the bound is found on the coarser key d << 6 |
// p >> 4, which orders alike, and the sort takes distances from the smallest one.
template <int NPL>
__device__ __forceinline__ uint64_t select_k(const uint32_t (&dv)[NPL], const int n, const int K, const bool small,
                                             uint32_t *row, const int lane) {
    const int shift = small ? 10 : 6;
    const uint32_t pl = small ? (uint32_t)lane : (uint32_t)lane >> 4;
    uint32_t key[NPL], m = ~0u;
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
        key[i] = (dv[i] << shift) | (pl + (small ? 64u * i : 4u * i));
        if (64 * (i + 1) > n) key[i] = lane + 64 * i < n ? key[i] : ~0u;   // the first test is uniform
        m = min(m, key[i]);
    }
    const uint32_t s = half_sort_asc(m, lane);
    const uint32_t t0 = __builtin_amdgcn_readlane(s, K / 2 - 1), t1 = __builtin_amdgcn_readlane(s, 32 + K / 2 - 1);
    const uint32_t theta = min(max(t0, t1), 0xFFFFFFFEu);   // ~0 marks an empty place
    // 32-bit keys in the row: distances from their smallest where they are wide (their range under
    // the bound nearly always fits 22 bits; the 64-bit form below takes the rest)
    const uint32_t dmin = small ? 0u : min((uint32_t)__builtin_amdgcn_readlane(s, 0), (uint32_t)__builtin_amdgcn_readlane(s, 32)) >> 6;
    if (small || (theta >> 6) - dmin < (1u << 22) - 1u) {
        int total = 0;
#pragma unroll
        for (int i = 0; i < NPL; ++i) {
            const bool in = key[i] <= theta;
            const uint64_t mask = __builtin_amdgcn_ballot_w64(in);
            if (in) row[total + bits_below(mask)] = small ? key[i] : (((key[i] >> 6) - dmin) << 10) | (uint32_t)(lane + 64 * i);
            total += __popcll(mask);
        }
        wave_lds_sync();
        uint32_t v;
        if (total <= 64) {
            v = wave_sort_asc<uint32_t>(lane < total ? row[lane] : ~0u, lane);
        } else if (total <= 128) {
            // two sorted halves: the smaller of each key and its mirror in the other half are the 64
            // smallest, in bitonic order
            v = wave_sort_asc<uint32_t>(row[lane], lane);
            const uint32_t u = wave_sort_asc<uint32_t>(lane + 64 < total ? row[lane + 64] : ~0u, lane);
            v = min(v, mirror_lane(u, 64, lane));
#pragma unroll
            for (int j = 32; j > 0; j >>= 1) {
                const uint32_t p = xor_lane(v, j, lane);
                v = (lane & j) ? max(v, p) : min(v, p);
            }
        } else {
            lds_sort(row, total, lane);
            v = row[lane];
        }
        return small ? (uint64_t)v : ((uint64_t)((v >> 10) + dmin) << 10) | (v & 1023u);
    }
    // (the distances are in the coarse keys)  The K-th smallest of the exact lane minima, under which at most RUN_K lanes hold keys
    uint64_t *sel = reinterpret_cast<uint64_t *>(row);
    uint64_t mm = ~0ull;
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
        const int p = lane + 64 * i;
        const uint64_t k64 = ((uint64_t)(key[i] >> 6) << 10) | (uint64_t)p;
        mm = p < n && k64 < mm ? k64 : mm;
    }
    const uint64_t bound = readlane_u64(wave_sort64(mm, lane), K - 1);
    int total = 0;
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
        const int p = lane + 64 * i;
        const uint64_t k64 = ((uint64_t)(key[i] >> 6) << 10) | (uint64_t)p;
        const bool in = p < n && k64 <= bound;
        const uint64_t mask = __builtin_amdgcn_ballot_w64(in);
        if (in) sel[total + bits_below(mask)] = k64;
        total += __popcll(mask);
    }
    wave_lds_sync();
    if (total <= 64) return wave_sort64(lane < total ? sel[lane] : ~0ull, lane);
    lds_sort(sel, total, lane);
    return sel[lane];
}

// Whether the columns that blocks of 16 leave over are few enough to be taken a row per lane.  Such a
// step makes its addresses anew, hence the factor 2.
__host__ __device__ inline bool turn_columns(int uh, int uw) {
    return (uw & 15) && 2 * (uw & 15) * ((uh + 15) >> 4) < uh;
}

// Groups of the 4 TR references of tile b, TR rows of 4, by as many wavefronts (VIDEO: tile b of the frames' tiles, frame-major; ONE: the
// table holds the windows of all its frames and a reference selects once).
template <bool VIDEO, int NPL, bool ONE = false, int TR = REF_TILE, bool TURN = false>
__device__ __forceinline__ void bm_tile(const ImageGeom &g0, const MethodParams &mp, const int tiles_x, const int b_in,
                                        const BmLds &L, int32_t *__restrict__ idx_out,
                                        int32_t *__restrict__ dist_out, unsigned char *smem, TileInfo &ti,
                                        const VideoArgs &va) {
    constexpr int NW = 4 * TR, NR = 4 * TR, THREADS = 64 * NW;   // wavefronts, references
    int tid_f = threadIdx.x;
    asm volatile("" : "+v"(tid_f));   // nothing per thread is kept from tile to tile
    const int tid = tid_f, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int b = b_in, t = 0, f_lo = 0, nf = 1;
    ImageGeom g = g0;   // the reference's frame
    if constexpr (VIDEO) {
        const int tiles_frame = ((g0.ny + TR - 1) / TR) * tiles_x;
        t = b_in / tiles_frame;
        b = b_in - t * tiles_frame;
        g.img = g0.img + (int64_t)t * va.frame_bytes;
        f_lo = max(0, t - va.radius);
        nf = min(va.T - 1, t + va.radius) - f_lo + 1;
    }
    const int tyi = b / tiles_x, txi = b % tiles_x;
    const int R = (mp.W - 1) / 2;

    // ---- tile geometry ----
    // The union of the 16 windows in closed form (positions increase along each side), so every
    // thread has it at once and the staging loads need not wait for the per-reference table.
    const int iya = tyi * TR, iyb = min(iya + TR, g.ny) - 1;
    const int ixa = txi * REF_TILE, ixb = min(ixa + REF_TILE, g.nx) - 1;
    const int uy0 = max(0, ref_pos(iya, g.ny, g.h, g.s) - R);
    const int ux0 = max(0, ref_pos(ixa, g.nx, g.w, g.s) - R);
    const int uh = min(g.h - PS, ref_pos(iyb, g.ny, g.h, g.s) + R) - uy0 + 1;
    const int uw = min(g.w - PS, ref_pos(ixb, g.nx, g.w, g.s) + R) - ux0 + 1;
    if (tid < NREF) {
        const int iy = iya + tid / REF_TILE, ix = txi * REF_TILE + tid % REF_TILE;
        if (tid < NR && iy < g.ny && ix < g.nx) {
            const int y = ref_pos(iy, g.ny, g.h, g.s), x = ref_pos(ix, g.nx, g.w, g.s);
            const int y0 = max(0, y - R), y1 = min(g.h - PS, y + R);
            const int x0 = max(0, x - R), x1 = min(g.w - PS, x + R);
            ti.ry[tid] = y; ti.rx[tid] = x;
            ti.wy0[tid] = y0; ti.wx0[tid] = x0;
            ti.wh[tid] = y1 - y0 + 1; ti.ww[tid] = x1 - x0 + 1;
        } else {
            ti.ry[tid] = -1; ti.rx[tid] = -1;
            ti.wy0[tid] = 0; ti.wx0[tid] = 0; ti.wh[tid] = 0; ti.ww[tid] = 0;
        }
    }
    // Eq. 9 branch per reference from the raw channel norms (16 threads per reference; the
    // reference position is recomputed here, so these loads overlap with the staging below).
    if (g.c == 3) {
        const int i = tid >> 4, sub = tid & 15;   // 16 threads per reference (the first 256 threads)
        int nr = 0, ng = 0, nb = 0;
        const int iy = iya + i / REF_TILE, ix = ixa + i % REF_TILE;
        if (i < NR && iy < g.ny && ix < g.nx) {
            const int ry = ref_pos(iy, g.ny, g.h, g.s), rx = ref_pos(ix, g.nx, g.w, g.s);
            for (int p = sub; p < PS * PS; p += 16) {
                const uint8_t *px = g.img + (int64_t)(ry + p / PS) * g.stride + (int64_t)(rx + p % PS) * 3;
                nr += px[0] * px[0]; ng += px[1] * px[1]; nb += px[2] * px[2];
            }
        }
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) {
            nr += __shfl_xor(nr, o); ng += __shfl_xor(ng, o); nb += __shfl_xor(nb, o);
        }
        if (sub == 0 && i < NREF) {
            const int64_t mx = nr > nb ? nr : nb;
            ti.green[i] = (int64_t)mp.gnum * mp.gnum * ng >= (int64_t)mp.gden * mp.gden * mx ? 1 : 0;
        }
    } else if (tid < NREF) {
        ti.green[tid] = 1;
    }
    const int prow = uh + PS - 1, pcol = uw + PS - 1;

    unsigned char *p8 = smem + L.off_p8;
    _Float16 *p16 = reinterpret_cast<_Float16 *>(smem + L.off_p16);
    int32_t *n8 = reinterpret_cast<int32_t *>(smem + L.off_n8);
    int32_t *n16 = reinterpret_cast<int32_t *>(smem + L.off_n16);
    uint32_t *tab = reinterpret_cast<uint32_t *>(smem + L.off_tab);
    const int plane8 = L.plane8;
    const int plane16 = L.rows * L.pitch16;

    // Per-lane state of the distance phase, kept across the frames of a video search: the A
    // fragments of reference i16 and the window and norm of the 4 references of this lane's
    // accumulators.
    v4i a8;
    v8h a16a = {}, a16b = {};
    bool any_sum = false;
    int rn[4];             // squared norms of the references 4 q + r
    int gmask[4];          // all ones where reference 4 q + r takes the green distance
    constexpr int TAB = tab_stride<NPL>();
    uint64_t *run = reinterpret_cast<uint64_t *>(smem + L.total - NREF * RUN_K * 8);
    const int K = mp.K;

    for (int fi = 0; fi < nf; ++fi) {
        // addresses are made anew for each frame: kept over the loop they cost 50 registers
        if constexpr (VIDEO) asm volatile("" : "+v"(tid_f));
        const int tid = tid_f, lane = tid & 63, i16 = lane & 15, q = lane >> 4;
        int slot = 0;
        const uint8_t *fimg = g.img;
        if constexpr (VIDEO) {
            // the reference's own frame first (its patches become the A fragments), then the others
            const int f = fi == 0 ? t : f_lo + fi - 1 + (f_lo + fi - 1 >= t ? 1 : 0);
            slot = f - f_lo;
            fimg = g0.img + (int64_t)f * va.frame_bytes;
            if (fi > 0) __syncthreads();   // the last frame's planes and table or selection scratch are reused
        }

        // ---- stage the shifted planes: one thread per (row, group of 4 columns) ----
        // Dword w of int8 copy k holds the row's pixels 4w + k .. 4w + k + 3, and halves 4w .. 4w + 3
        // of fp16 copy k hold the pixels 4w + k .. 4w + k + 3, so a thread needs pixels 4w .. 4w + 6.
        // Bytes at or beyond the staged width pcol are never read (candidates end at pcol - 1).
        {
            const int nw = (pcol + 3) >> 2;
            const uint8_t *img_end = fimg + (int64_t)(g.h - 1) * g.stride + (int64_t)g.w * g.c;
            uint32_t *p8w = reinterpret_cast<uint32_t *>(p8);
            uint32_t *p16w = reinterpret_cast<uint32_t *>(p16);
            for (int e = tid; e < prow * nw; e += THREADS) {
                const int r = e / nw, w4 = 4 * (e - r * nw);
                const int npx = min(7, pcol - w4);
                const uint8_t *a = fimg + (int64_t)(uy0 + r) * g.stride + (int64_t)(ux0 + w4) * g.c;
                uint32_t raw[6];   // bytes 0 .. 23 from a
                const uintptr_t ai = (uintptr_t)a;
                const uint32_t *ab = reinterpret_cast<const uint32_t *>(ai & ~(uintptr_t)3);
                if (npx == 7 && (const uint8_t *)(ab + 7) <= img_end) {
                    const uint32_t sh = (uint32_t)(ai & 3);
                    uint32_t d[7];
#pragma unroll
                    for (int i = 0; i < 7; ++i) d[i] = ab[i];
#pragma unroll
                    for (int i = 0; i < 6; ++i) raw[i] = __builtin_amdgcn_alignbyte(d[i + 1], d[i], sh);
                } else {   // row end: only the pixels that exist, byte by byte
#pragma unroll
                    for (int i = 0; i < 6; ++i) raw[i] = 0u;
                    const int nb = npx * g.c;
                    for (int b = 0; b < nb; ++b) raw[b >> 2] |= (uint32_t)a[b] << (8 * (b & 3));
                }
                auto byte_at = [&](int i) { return (int)((raw[i >> 2] >> (8 * (i & 3))) & 0xffu); };
                int v8[7], vs[7];
#pragma unroll
                for (int q = 0; q < 7; ++q) {
                    if (g.c == 3) {
                        const int R = byte_at(3 * q), G = byte_at(3 * q + 1), B = byte_at(3 * q + 2);
                        v8[q] = G - 128;
                        vs[q] = R + G + B - 384;
                    } else {
                        v8[q] = byte_at(q) - 128;
                        vs[q] = 0;
                    }
                }
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    p8w[(k * plane8 + r * L.pitch8 + w4) >> 2] =
                        (uint32_t)(uint8_t)v8[k] | ((uint32_t)(uint8_t)v8[k + 1] << 8) |
                        ((uint32_t)(uint8_t)v8[k + 2] << 16) | ((uint32_t)(uint8_t)v8[k + 3] << 24);
                if (g.c == 3) {
#pragma unroll
                    for (int k = 0; k < 2; ++k)
#pragma unroll
                        for (int hh = 0; hh < 2; ++hh) {
                            const uint32_t lo = __builtin_bit_cast(uint16_t, (_Float16)vs[2 * hh + k]);
                            const uint32_t hi = __builtin_bit_cast(uint16_t, (_Float16)vs[2 * hh + k + 1]);
                            p16w[(k * plane16 + r * L.pitch16 + w4 + 2 * hh) >> 1] = lo | (hi << 16);
                        }
                }
            }
        }
        __syncthreads();
        if (fi == 0 && tid == 0) {   // read after the norm phase's barriers
            int any = 0;
            for (int i = 0; i < NREF; ++i) any |= (ti.ry[i] >= 0 && !ti.green[i]);
            ti.any_sum = any;
        }

        // ---- squared norms at every candidate position (horizontal then vertical 8-sums) ----
        // Four consecutive outputs per thread from one window of 11 values, sliding (exact integers).
        // Reads past the last valid output stay inside the staged planes and the row sums' place (see
        // bm_lds_layout); the outputs they feed are not stored.
        {
            // prow x uw; but for the windows of earlier frames the table is free now
            int32_t *rs8 = reinterpret_cast<int32_t *>(ONE ? smem + L.off_rs : smem + L.off_tab);
            int32_t *rs16 = rs8 + prow * uw;
            const int ng = (uw + 3) >> 2;
            for (int e = tid; e < prow * ng; e += THREADS) {
                const int r = e / ng, c0 = 4 * (e - r * ng);
                int q8[11], q16[11];
                {
                    const uint32_t *w8 = reinterpret_cast<const uint32_t *>(p8 + r * L.pitch8 + c0);
                    const uint32_t b[3] = {w8[0], w8[1], w8[2]};
#pragma unroll
                    for (int j = 0; j < 11; ++j) {
                        const int v = (int)(int8_t)(b[j >> 2] >> (8 * (j & 3)));
                        q8[j] = v * v;
                    }
                }
                if (g.c == 3) {
                    const uint32_t *w16 = reinterpret_cast<const uint32_t *>(p16 + r * L.pitch16 + c0);
                    uint32_t b[6];
#pragma unroll
                    for (int i = 0; i < 6; ++i) b[i] = w16[i];
#pragma unroll
                    for (int j = 0; j < 11; ++j) {
                        const int t = (int)__builtin_bit_cast(_Float16, (uint16_t)(b[j >> 1] >> (16 * (j & 1))));
                        q16[j] = t * t;
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < 11; ++j) q16[j] = 0;
                }
                int a = 0, t = 0;
#pragma unroll
                for (int j = 0; j < PS; ++j) {
                    a += q8[j];
                    t += q16[j];
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (c0 + k < uw) {
                        rs8[r * uw + c0 + k] = a;
                        rs16[r * uw + c0 + k] = t;
                    }
                    if (k < 3) {
                        a += q8[k + PS] - q8[k];
                        t += q16[k + PS] - q16[k];
                    }
                }
            }
            __syncthreads();
            const int nr4 = (uh + 3) >> 2;
            for (int e = tid; e < nr4 * uw; e += THREADS) {
                const int r4 = 4 * (e / uw), col = e - (r4 >> 2) * uw;
                int c8[11], c16[11];
#pragma unroll
                for (int i = 0; i < 11; ++i) {
                    c8[i] = rs8[(r4 + i) * uw + col];
                    c16[i] = rs16[(r4 + i) * uw + col];
                }
                int a = 0, t = 0;
#pragma unroll
                for (int i = 0; i < PS; ++i) {
                    a += c8[i];
                    t += c16[i];
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (r4 + k < uh) {
                        n8[(r4 + k) * uw + col] = a;
                        n16[(r4 + k) * uw + col] = t;
                    }
                    if (k < 3) {
                        a += c8[k + PS] - c8[k];
                        t += c16[k + PS] - c16[k];
                    }
                }
            }
            __syncthreads();
        }

        // ---- distances on the matrix cores ----
        {
            if (fi == 0) {
                // A fragments: reference i16, rows 2q, 2q+1 (int8) and rows q, q+4 (fp16).
                int ar = ti.ry[i16] >= 0 ? ti.ry[i16] - uy0 : 0;
                int ac = ti.ry[i16] >= 0 ? ti.rx[i16] - ux0 : 0;
                {
                    const int k = ac & 3;
                    const unsigned char *base = p8 + k * plane8;
                    const int o0 = (ar + 2 * q) * L.pitch8 + ac - k, o1 = o0 + L.pitch8;
                    a8[0] = (int)lds_u32(base, o0); a8[1] = (int)lds_u32(base, o0 + 4);
                    a8[2] = (int)lds_u32(base, o1); a8[3] = (int)lds_u32(base, o1 + 4);
                }
                any_sum = ti.any_sum != 0;
                if (any_sum) {
                    const int k = ac & 1;
                    const _Float16 *base = p16 + k * plane16;
                    const _Float16 *ra = base + (ar + q) * L.pitch16 + ac - k;
                    const _Float16 *rb = base + (ar + q + 4) * L.pitch16 + ac - k;
#pragma unroll
                    for (int t = 0; t < 8; ++t) { a16a[t] = ra[t]; a16b[t] = rb[t]; }
                }
                // Per-lane info of the 4 references this lane's accumulators belong to.
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int ii = 4 * q + r;
                    rn[r] = gmask[r] = 0;
                    if (ti.ry[ii] >= 0) {
                        const int pe = (ti.ry[ii] - uy0) * uw + (ti.rx[ii] - ux0);
                        rn[r] = ti.green[ii] ? n8[pe] : n16[pe];
                        gmask[r] = -ti.green[ii];
                    }
                }
            }
            // A wave takes one block of 16 columns of the union and every so-many-th row, so that all
            // addresses step by constants and the columns of the windows are tested once.  In the
            // union's coordinates the references 4 q + r lie in row q and column r of the tile, so the
            // rows of their windows go with q and the columns with r; position (dy, dx) of reference
            // 4 q + r is table byte 4 (dy ww + dx) of its row.
            // TURN: where few columns are left over, a lane takes a row of one of them instead.
            const bool turned = TURN && turn_columns(uh, uw);
            const int ncb = turned ? uw >> 4 : (uw + 15) >> 4;   // 0 .. 4
            const int wpc = ncb <= 1 ? NW : (ncb == 2 ? NW / 2 : (ncb == 3 ? NW / 3 : NW / 4));   // waves per block of columns
            const int cb = (wave >= wpc) + (wave >= 2 * wpc) + (wave >= 3 * wpc), cr0 = wave - cb * wpc;
            const int cc0 = 16 * cb + i16, cc = min(cc0, uw - 1);
            const int wy = ti.wy0[4 * q] - uy0, wh = ti.ry[4 * q] >= 0 ? ti.wh[4 * q] : 0;
            bool inside[4];
            int step4[4];
            unsigned char *at[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int dx = cc0 - (ti.wx0[r] - ux0), ww = ti.ry[r] >= 0 ? ti.ww[r] : 0;
                inside[r] = (unsigned)dx < (unsigned)ww;
                at[r] = reinterpret_cast<unsigned char *>(tab + (4 * q + r) * TAB + ((ONE ? slot * wh : 0) + cr0 - wy) * ww + dx);
                step4[r] = 4 * wpc * ww;
            }
            const unsigned char *c8 = p8 + (cc & 3) * plane8 + (cr0 + 2 * q) * L.pitch8 + (cc & ~3);
            // 8 halves from the copy in which they start on a dword (pitch and offsets even)
            const _Float16 *c16 = p16 + (cc & 1) * plane16 + (cr0 + q) * L.pitch16 + (cc & ~1);
            const int32_t *m8 = n8 + cr0 * uw + cc, *m16 = n16 + cr0 * uw + cc;
            if (cb < ncb) {
                for (int cr = cr0; cr < uh; cr += wpc) {
                    const uint32_t *w8a = reinterpret_cast<const uint32_t *>(c8);
                    const uint32_t *w8b = reinterpret_cast<const uint32_t *>(c8 + L.pitch8);
                    const v4i b8 = {(int)w8a[0], (int)w8a[1], (int)w8b[0], (int)w8b[1]};
                    const v4i acc8 = __builtin_amdgcn_mfma_i32_16x16x64_i8(a8, b8, (v4i){0, 0, 0, 0}, 0, 0, 0);
                    // d = |a|^2 + |b|^2 - 2 a.b with |a.b| <= 64 384^2 < 2^24
                    int d[4];
                    if (any_sum) {
                        const uint32_t *ra = reinterpret_cast<const uint32_t *>(c16);
                        const uint32_t *rb = reinterpret_cast<const uint32_t *>(c16 + 4 * L.pitch16);
                        const v8h b16a = __builtin_bit_cast(v8h, make_uint4(ra[0], ra[1], ra[2], ra[3]));
                        const v8h b16b = __builtin_bit_cast(v8h, make_uint4(rb[0], rb[1], rb[2], rb[3]));
                        v4f acc16 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a16a, b16a, (v4f){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                        acc16 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a16b, b16b, acc16, 0, 0, 0);
                        const int nb8 = *m8, nb16 = *m16;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int dot = (gmask[r] & acc8[r]) | (~gmask[r] & (int)acc16[r]);
                            const int nb = (gmask[r] & nb8) | (~gmask[r] & nb16);
                            d[r] = nb + rn[r] - 2 * dot;
                        }
                    } else {
                        const int nb8 = *m8;
#pragma unroll
                        for (int r = 0; r < 4; ++r) d[r] = nb8 + rn[r] - 2 * acc8[r];
                    }
                    if ((unsigned)(cr - wy) < (unsigned)wh) {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (inside[r]) *reinterpret_cast<uint32_t *>(at[r]) = (uint32_t)d[r];
                    }
                    c8 += wpc * L.pitch8;
                    c16 += wpc * L.pitch16;
                    m8 += wpc * uw;
                    m16 += wpc * uw;
#pragma unroll
                    for (int r = 0; r < 4; ++r) at[r] += step4[r];
                }
            }
            if (TURN && turned) {
                const int rows16 = (uh + 15) >> 4;
#pragma unroll 1
                for (int it = NW - 1 - wave; it < (uw & 15) * rows16; it += NW) {
                    int i16 = lane & 15, q = lane >> 4;
                    asm volatile("" : "+v"(i16), "+v"(q));   // nothing of this is made before the loop above
                    const int c = (uw & ~15) + it / rows16, row = 16 * (it % rows16) + i16, cr = min(row, uh - 1);
                    const unsigned char *t8 = p8 + (c & 3) * plane8 + (cr + 2 * q) * L.pitch8 + (c & ~3);
                    const uint32_t *w8a = reinterpret_cast<const uint32_t *>(t8);
                    const uint32_t *w8b = reinterpret_cast<const uint32_t *>(t8 + L.pitch8);
                    const v4i b8 = {(int)w8a[0], (int)w8a[1], (int)w8b[0], (int)w8b[1]};
                    const v4i acc8 = __builtin_amdgcn_mfma_i32_16x16x64_i8(a8, b8, (v4i){0, 0, 0, 0}, 0, 0, 0);
                    v4f acc16 = {0.f, 0.f, 0.f, 0.f};
                    if (any_sum) {
                        const _Float16 *t16 = p16 + (c & 1) * plane16 + (cr + q) * L.pitch16 + (c & ~1);
                        const uint32_t *ra = reinterpret_cast<const uint32_t *>(t16);
                        const uint32_t *rb = reinterpret_cast<const uint32_t *>(t16 + 4 * L.pitch16);
                        const v8h b16a = __builtin_bit_cast(v8h, make_uint4(ra[0], ra[1], ra[2], ra[3]));
                        const v8h b16b = __builtin_bit_cast(v8h, make_uint4(rb[0], rb[1], rb[2], rb[3]));
                        acc16 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a16a, b16a, acc16, 0, 0, 0);
                        acc16 = __builtin_amdgcn_mfma_f32_16x16x32_f16(a16b, b16b, acc16, 0, 0, 0);
                    }
                    const int nb8 = n8[cr * uw + c], nb16 = any_sum ? n16[cr * uw + c] : 0;
                    if ((unsigned)(row - wy) < (unsigned)wh) {   // the windows end within the union
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int dx = c - (ti.wx0[r] - ux0), ww = ti.ry[r] >= 0 ? ti.ww[r] : 0;
                            const int dot = (gmask[r] & acc8[r]) | (~gmask[r] & (int)acc16[r]);
                            const int nb = (gmask[r] & nb8) | (~gmask[r] & nb16);
                            if ((unsigned)dx < (unsigned)ww)
                                tab[(4 * q + r) * TAB + (row - wy) * ww + dx] = (uint32_t)(nb + rn[r] - 2 * dot);
                        }
                    }
                }
            }
        }
        if (ONE && fi + 1 < nf) continue;   // the next frame's staging begins with a barrier
        __syncthreads();

        // ---- top-K per reference ----
        for (int ii = wave; ii < NR; ii += NW) {
            if (ti.ry[ii] < 0) continue;
            const int ww = __builtin_amdgcn_readfirstlane(ti.ww[ii]);
            const int n = __builtin_amdgcn_readfirstlane(ti.wh[ii]) * ww * (ONE ? nf : 1);
            uint32_t *row = tab + ii * TAB;
            // this lane's candidates p = lane + 64 i, read once (past the window: whatever is there)
            uint32_t dv[NPL];
#pragma unroll
            for (int i = 0; i < NPL; ++i) dv[i] = row[lane + 64 * i];
            const bool small = __builtin_amdgcn_readfirstlane(ti.green[ii]) != 0;
            if constexpr (VIDEO && !ONE) {
                if (fi > 0) {
                    // Only keys below the running K-th can enter the list; its slot is another one,
                    // so the distance decides alone.  When at most 64 - K of this frame's candidates
                    // are, one sort of them with the list is the merge.
                    const uint64_t th = run[ii * RUN_K + K - 1];
                    const uint32_t below = (uint32_t)(th >> 16) + ((uint32_t)slot < ((uint32_t)(th >> 10) & 63u) ? 1u : 0u);
                    uint32_t in = 0;   // bit i: dv[i] qualifies
                    int total = 0;
#pragma unroll
                    for (int i = 0; i < NPL; ++i) {
                        const bool q1 = lane + 64 * i < n && dv[i] < below;
                        in |= (uint32_t)q1 << i;
                        total += __popcll(__builtin_amdgcn_ballot_w64(q1));
                    }
                    if (total == 0) continue;
                    if (total <= 64 - K) {
                        uint64_t *sel = reinterpret_cast<uint64_t *>(row);
                        int at0 = 0;
#pragma unroll
                        for (int i = 0; i < NPL; ++i) {
                            const bool q1 = (in >> i) & 1u;
                            const uint64_t mask = __builtin_amdgcn_ballot_w64(q1);
                            if (q1)
                                sel[at0 + bits_below(mask)] = ((uint64_t)dv[i] << 16) | ((uint64_t)slot << 10) |
                                                              (uint64_t)(lane + 64 * i);
                            at0 += __popcll(mask);
                        }
                        wave_lds_sync();
                        uint64_t v = lane < total ? sel[lane]
                                                  : (lane < total + K ? run[ii * RUN_K + lane - total] : ~0ull);
                        v = wave_sort64(v, lane);
                        if (lane < K) run[ii * RUN_K + lane] = v;
                        wave_lds_sync();
                        continue;
                    }
                }
            }
            const uint64_t mine = select_k<NPL>(dv, n, K, small, row, lane);
            if constexpr (VIDEO && !ONE) {
                // merge into the running list: keys (distance, frame slot, position); only this wave
                // touches reference ii's list
                uint64_t v = lane < K ? (((mine >> 10) << 16) | ((uint64_t)slot << 10) | (mine & 1023u)) : ~0ull;
                if (fi > 0) {
                    if (lane >= K && lane < 2 * K) v = run[ii * RUN_K + lane - K];
                    v = wave_sort64(v, lane);
                }
                if (lane < K) run[ii * RUN_K + lane] = v;
            } else if (lane < K) {
                const int p = (int)(mine & 1023u);
                const int py = (int)((uint32_t)p * (65536u / (uint32_t)ww + 1u) >> 16);   // p / ww for p < 1024
                int y = ti.wy0[ii] + py;
                const int x = ti.wx0[ii] + p - py * ww;
                const int iy = iya + ii / REF_TILE, ix = txi * REF_TILE + ii % REF_TILE;
                int64_t r = (int64_t)iy * g.nx + ix;
                if constexpr (ONE) {   // py runs through the rows of all frames' windows
                    const int wh = ti.wh[ii], f = py / wh;
                    y += (f_lo + f) * g.h - f * wh;
                    r += (int64_t)t * g.ny * g.nx;
                }
                idx_out[r * K + lane] = y * g.w + x;
                if (dist_out) dist_out[r * K + lane] = (int32_t)(mine >> 10);
            }
            wave_lds_sync();
        }
        if constexpr (ONE) break;
    }   // frames

    if constexpr (VIDEO && !ONE) {
        for (int ii = wave; ii < NR; ii += NW) {
            if (ti.ry[ii] < 0 || lane >= K) continue;
            const uint64_t key = run[ii * RUN_K + lane];
            const int p = (int)(key & 1023u), f = f_lo + (int)((key >> 10) & 63u);
            const int y = ti.wy0[ii] + p / ti.ww[ii], x = ti.wx0[ii] + p % ti.ww[ii];
            const int iy = iya + ii / REF_TILE, ix = txi * REF_TILE + ii % REF_TILE;
            const int64_t r = ((int64_t)t * g.ny + iy) * g.nx + ix;
            idx_out[r * K + lane] = (f * g.h + y) * g.w + x;
            if (dist_out) dist_out[r * K + lane] = (int32_t)(key >> 16);
        }
    }
}

// MANY: the form of 64 registers for many tiles of which two share a CU; only this one has the rows per
// lane for the columns left over, whose registers cost the others more than they gain.
template <int NPL, int TR = REF_TILE, bool MANY = false>
__global__ __launch_bounds__(256 * TR, MANY ? 8 : (TR == REF_TILE ? 4 : 6)) void bm_kernel(ImageGeom g, MethodParams mp, int tiles_x, int n_tiles,
                                                 BmLds L, int32_t *__restrict__ idx_out,
                                                 int32_t *__restrict__ dist_out, BmExtra extra) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ TileInfo ti;
    // XCD-aware order: consecutive workgroups are dealt round-robin over the 8 XCDs; give
    // each XCD a contiguous run of tiles so neighbouring tiles share its L2.
    // The grid has 8*ceil(n_tiles/8) workgroups; b -> (b%8)*per + b/8 is a bijection on it.
    const int per = (n_tiles + 7) / 8;
    const int b = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (b >= n_tiles) return;
    if (extra.guard && blockIdx.x == 0 && threadIdx.x < 2) extra.guard[threadIdx.x] = 0;
    if (extra.tau && threadIdx.x < 4 * TR) {
        const int iy = b / tiles_x * TR + threadIdx.x / REF_TILE, ix = b % tiles_x * REF_TILE + threadIdx.x % REF_TILE;
        if (iy < g.ny && ix < g.nx) extra.tau[(int64_t)iy * g.nx + ix] = extra.value;
    }
    bm_tile<false, NPL, false, TR, MANY>(g, mp, tiles_x, b, L, idx_out, dist_out, smem, ti, VideoArgs{});
}

// Spatio-temporal form: n_tiles covers the tiles of all frames.
// 64 registers, so that two workgroups share a CU where the LDS allows: while one waits at a barrier
// the other works.  Rows of 16 keys per lane do not fit them.
template <int NPL, bool ONE>
__global__ __launch_bounds__(BMT, ONE && NPL < 16 ? 8 : 4) void bm_video_kernel(ImageGeom g, MethodParams mp, int tiles_x, int n_tiles,
                                                       VideoArgs va, BmLds L, int32_t *__restrict__ idx_out,
                                                       int32_t *__restrict__ dist_out) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ TileInfo ti;
    const int per = (n_tiles + 7) / 8;
    const int b = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (b >= n_tiles) return;
    bm_tile<true, NPL, ONE>(g, mp, tiles_x, b, L, idx_out, dist_out, smem, ti, va);
}

// Persistent form over many images: each workgroup pulls (image, tile) units from a queue.
template <int NPL, int TR = REF_TILE>
__global__ __launch_bounds__(256 * TR, NPL < 16 ? 8 : (TR < REF_TILE ? 6 : 4)) void bm_kernel_batched(
    const BatchItem *__restrict__ items, int n_items, const int *__restrict__ unit_start, BmLds L,
    int *__restrict__ queue) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ TileInfo ti;
    __shared__ int s_u;
    const int total = unit_start[n_items];
    for (;;) {
        if (threadIdx.x == 0) s_u = atomicAdd(queue, 1);
        __syncthreads();
        const int u = s_u;
        __syncthreads();
        if (u >= total) break;
        const int i = find_unit(unit_start, n_items, u);
        const BatchItem it = items[i];
        bm_tile<false, NPL, false, TR>(it.g, it.mp, it.bm_tiles_x, u - unit_start[i], L, it.idx, nullptr, smem, ti, VideoArgs{});
        __syncthreads();
    }
}

// Register rows of the table (tab_stride) that windows of up to n positions need.
int bm_npl(int n) { return n <= 256 ? 4 : (n <= 448 ? 7 : (n <= 640 ? 10 : 16)); }
int bm_tab_stride(int npl) { return npl == 11 ? tab_stride<11>() : npl == 4 ? tab_stride<4>() : (npl == 7 ? tab_stride<7>() : (npl == 10 ? tab_stride<10>() : tab_stride<16>())); }

BmLds bm_lds_layout(int uh_max, int uw_max, int npl, bool video = false, bool one = false, int tile_rows = REF_TILE) {
    BmLds L;
    L.rows = uh_max + PS - 1;
    // The int8 planes: rows of 96 bytes (enough for a union of 64 columns plus the patch and the
    // dword reads past it) and copies 16 bytes past a row multiple apart.  With these offsets the
    // 64 lanes' dword reads of a distance step (16 consecutive candidates x 4 row pairs, each
    // candidate in the copy where it starts on a dword) spread over the LDS banks (at most 1.5
    // reads per bank against 2 to 4 for tightly packed rows, whether 32 or 64 banks serve a
    // half or a whole wave).
    const int pitch_min = ((uw_max + PS + 3) / 4) * 4 + 4;
    L.pitch8 = pitch_min > 96 || tile_rows < REF_TILE ? pitch_min : 96;
    L.plane8 = L.rows * L.pitch8 + 16;
    L.pitch16 = ((uw_max + PS + 1) / 2) * 2 + 2;
    int off = 0;
    L.off_p8 = off;  off += 4 * L.plane8;
    off = (off + 15) & ~15;
    L.off_p16 = off; off += 2 * L.rows * L.pitch16 * 2;
    off = (off + 15) & ~15;
    L.off_n8 = off;  off += uh_max * uw_max * 4;
    L.off_n16 = off; off += uh_max * uw_max * 4;
    off = (off + 15) & ~15;
    L.off_tab = off;
    // the last row is read to 64 npl words
    int tab_bytes = ((4 * tile_rows - 1) * bm_tab_stride(npl) + std::max(bm_tab_stride(npl), 64 * npl)) * 4;
    // row sums of the norm pass live in the table, unless that holds the windows of earlier frames;
    // its columns read up to 3 rows past the last
    const int rs_bytes = (2 * L.rows + 3) * uw_max * 4;
    if (!one && tab_bytes < rs_bytes) tab_bytes = rs_bytes;
    off += (tab_bytes + 15) & ~15;
    L.off_rs = off;
    if (one) off += (rs_bytes + 15) & ~15;
    if (video && !one) off += NREF * RUN_K * 8;   // the running lists of the video search
    L.total = off;
    return L;
}

}  // namespace

namespace {

// Launch shape for images up to h x w, steps up to s and windows up to W: register rows, rows of
// references per tile, LDS layout and whether two workgroups fit a CU.
struct BmShape {
    int npl, rows;
    BmLds L;
    bool two;
};

BmShape bm_shape(int s, int W, int h, int w) {
    BmShape r;
    // largest union of windows over a tile: 3 grid steps plus the window, capped by the image
    const int uw = min((REF_TILE - 1) * s + W, w - PS + 1);
    r.npl = bm_npl(min(W, h - PS + 1) * min(W, w - PS + 1));
    auto layout = [&](int rows) {
        r.rows = rows;
        r.L = bm_lds_layout(min((rows - 1) * s + W, h - PS + 1), uw, r.npl, false, false, rows);
        r.two = 2 * (r.L.total + (int)sizeof(TileInfo) + 64) <= 160 * 1024;
    };
    // The phases of a tile are separated by barriers, and only another workgroup fills the waits
    // behind them.  The table of 16 references with windows past 640 positions takes 62 KB and leaves no
    // room for a second one; 12 references with 12 waves do up to step 4: 12 MP, window 31, step 3, 4.15 ->
    // 3.44 ms, 512 x 512, step 4, 87 -> 68 us, though a tile's staging and matrix products serve fewer.
    // Where two tiles of 12 do not fit either, 16 references share the staging.
    if (r.npl == 16) layout(3);
    if (r.npl < 16 || !r.two) layout(REF_TILE);
    return r;
}

}  // namespace

int bm_tile_rows(int s, int W, int h, int w) { return bm_shape(s, W, h, w).rows; }

hipError_t launch_block_match(const ImageGeom &g, const MethodParams &mp, int32_t *idx, int32_t *dist,
                              hipStream_t st, const BmExtra &extra) {
    const BmShape sh = bm_shape(g.s, mp.W, g.h, g.w);
    const int tiles_x = (g.nx + REF_TILE - 1) / REF_TILE;
    const int n_tiles = (g.ny + sh.rows - 1) / sh.rows * tiles_x;
    // round the grid up to a multiple of 8 so the XCD remap is a bijection onto [0, 8*per)
    const int per = (n_tiles + 7) / 8;
    auto go = [&](auto kernel) {
        const hipError_t e = prepare_dynamic_lds((const void *)kernel, sh.L.total, (int)sizeof(TileInfo));
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(8 * per), dim3(256 * sh.rows), sh.L.total, st, g, mp, tiles_x, n_tiles, sh.L, idx,
                           dist, extra);
        return hipGetLastError();
    };
    // The form of 64 registers lets two workgroups share a CU where the LDS does: 509 x 763 RGB, window 21,
    // 91 us instead of 118, and with the column left over of a union of 33 (window 21 at step 4) 1536 x 2048
    // gray 322 instead of 425.  It spills 7 to 11 registers, which costs a workgroup alone on its CU more
    // than it gains: 256 x 256 gray 16.2 us against 15.3 (so it takes more than two rounds, 512 tiles), and
    // tiles of more than 80 KB (900 x 900 gray, window 25, step 6) 73.8 against 69.1.
    const bool many = n_tiles > 512 && sh.two;
    switch (sh.npl) {
        case 4: return many ? go(bm_kernel<4, REF_TILE, true>) : go(bm_kernel<4>);
        case 7: return many ? go(bm_kernel<7, REF_TILE, true>) : go(bm_kernel<7>);
        case 10: return many ? go(bm_kernel<10, REF_TILE, true>) : go(bm_kernel<10>);
        default: return sh.rows == 3 ? go(bm_kernel<16, 3>) : go(bm_kernel<16>);
    }
}

// Spatio-temporal block matching of T frames of g.h rows stacked from g.img (Sec. IV-C): the
// candidates of a reference in frame t are its clipped window in frames t - radius .. t + radius
// (within [0, T)).  idx/dist: T * ny * nx references, frame-major; idx = (f*h + y)*w + x.
hipError_t launch_block_match_video(const ImageGeom &g, const MethodParams &mp, int T, int radius, int32_t *idx,
                                    int32_t *dist, hipStream_t st) {
    const int tiles_y = (g.ny + REF_TILE - 1) / REF_TILE, tiles_x = (g.nx + REF_TILE - 1) / REF_TILE;
    const int64_t n_tiles64 = (int64_t)tiles_y * tiles_x * T;
    if (T < 1 || radius < 0 || radius > 31 || mp.K > RUN_K || n_tiles64 > (int64_t)1 << 30)
        return hipErrorInvalidValue;
    const int n_tiles = (int)n_tiles64;
    const int span = (REF_TILE - 1) * g.s + mp.W;
    const int uh = span < g.h - PS + 1 ? span : g.h - PS + 1;
    const int uw = span < g.w - PS + 1 ? span : g.w - PS + 1;
    const int window = min(mp.W, g.h - PS + 1) * min(mp.W, g.w - PS + 1), frames = min(2 * radius + 1, T);
    // One selection from the windows of all frames where they fit a row of the table and the table fits
    // beside the planes: 981 us against 1,761 us with a selection per frame and merged lists (four 720 x
    // 1280 frames, radius 1, window 15), of which 380 us are the second workgroup on a CU.
    const bool fits = window * frames <= MAX_CAND;
    const int npl_one = window * frames > 640 && window * frames <= 704 ? 11 : bm_npl(window * frames);
    const BmLds L_one = bm_lds_layout(uh, uw, fits ? npl_one : 4, true, true);
    const bool one = fits && L_one.total + (int)sizeof(TileInfo) <= 160 * 1024;
    const int npl = one ? npl_one : bm_npl(window);
    const BmLds L = one ? L_one : bm_lds_layout(uh, uw, npl, true);
    VideoArgs va{T, radius, (int64_t)g.h * g.stride};
    const int per = (n_tiles + 7) / 8;
    auto go = [&](auto kernel) {
        const hipError_t e = prepare_dynamic_lds((const void *)kernel, L.total, (int)sizeof(TileInfo));
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(8 * per), dim3(BMT), L.total, st, g, mp, tiles_x, n_tiles, va, L, idx, dist);
        return hipGetLastError();
    };
    if (one)
        switch (npl) {
            case 4: return go(bm_video_kernel<4, true>);
            case 7: return go(bm_video_kernel<7, true>);
            case 10: return go(bm_video_kernel<10, true>);
            case 11: return go(bm_video_kernel<11, true>);
            default: return go(bm_video_kernel<16, true>);
        }
    return npl == 4 ? go(bm_video_kernel<4, false>)
                    : (npl == 7 ? go(bm_video_kernel<7, false>)
                                : (npl == 10 ? go(bm_video_kernel<10, false>) : go(bm_video_kernel<16, false>)));
}

// Batched block matching: one persistent launch over the tiles of all images (bm_tile_rows of the
// same limits to a tile), `grid` workgroups or, where two fit a CU, twice as many; the LDS layout is
// the largest any image of the batch needs.
hipError_t launch_block_match_batched(const BatchItem *items, int n_items, const int *unit_start, int max_s,
                                      int max_W, int max_h, int max_w, int *queue, int grid, int units, hipStream_t st) {
    const BmShape sh = bm_shape(max_s, max_W, max_h, max_w);
    const int n = min(sh.two ? 2 * grid : grid, units);
    auto go = [&](auto kernel) {
        const hipError_t e = prepare_dynamic_lds((const void *)kernel, sh.L.total, (int)sizeof(TileInfo) + 16);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(n), dim3(256 * sh.rows), sh.L.total, st, items, n_items, unit_start, sh.L, queue);
        return hipGetLastError();
    };
    switch (sh.npl) {
        case 4: return go(bm_kernel_batched<4>);
        case 7: return go(bm_kernel_batched<7>);
        case 10: return go(bm_kernel_batched<10>);
        default: return sh.rows == 3 ? go(bm_kernel_batched<16, 3>) : go(bm_kernel_batched<16>);
    }
}

hipError_t prepare_dynamic_lds(const void *kernel, int bytes, int static_bytes) {
    int dev = 0, max_lds = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    e = hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    if (e != hipSuccess) return e;
    if (bytes + static_bytes > max_lds) return hipErrorInvalidValue;
    if (bytes > 64 * 1024) {
        // opt-in for large dynamic LDS where the runtime asks for it; a runtime that does not
        // need the opt-in may reject the attribute, which is harmless
        if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess)
            (void)hipGetLastError();
    }
    return hipSuccess;
}

}  // namespace htsvd
