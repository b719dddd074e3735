// Stand-alone tile crop for gfx950 (Section 4.3 / Table 1 "Tile" of the paper): copies the tile x tile
// window at a per-image origin out of each of the three u8 planes.  HBM-bound byte shuffling: one
// block per (image, plane); when everything is 4-byte friendly each lane assembles one aligned output
// dword from two aligned input dwords (funnel shift by the source misalignment), otherwise bytes.
// Also here: variance-based tile selection (further down).
#include <algorithm>
#include <type_traits>
#include "qrm_internal.h"

namespace qrm {

namespace {

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

template <bool WORDS>
__global__ __launch_bounds__(256) void extract_tiles_kernel(const uint8_t *__restrict__ img, int H, int W,
                                                            const int32_t *__restrict__ off, int tile,
                                                            uint8_t *__restrict__ out)
{
    const int64_t plane = blockIdx.x; // n*3 + c
    const int64_t n = plane / 3;
    int oy = 0, ox = 0;
    if (off) {
        oy = clampi(off[2 * n], 0, H - tile);
        ox = clampi(off[2 * n + 1], 0, W - tile);
    }
    const uint8_t *src = img + plane * (int64_t)H * W + (int64_t)oy * W + ox;
    uint8_t *dst = out + plane * (int64_t)tile * tile;
    if (WORDS) {
        const int wpr = tile >> 2; // dwords per output row
        const int total = wpr * tile;
        for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
            const int row = idx / wpr, col = (idx - row * wpr) << 2;
            const uint8_t *s = src + (int64_t)row * W + col;
            const uintptr_t a = (uintptr_t)s;
            const uint32_t *aligned = (const uint32_t *)(a & ~(uintptr_t)3);
            const unsigned sh = (unsigned)(a & 3u);
            uint32_t lo = aligned[0];
            uint32_t v = lo;
            if (sh) {
                uint32_t hi = aligned[1];
                v = __builtin_amdgcn_alignbyte(hi, lo, sh);
            }
            *(uint32_t *)(dst + (int64_t)row * tile + col) = v;
        }
    } else {
        const int total = tile * tile;
        for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
            const int row = idx / tile, col = idx - row * tile;
            dst[idx] = src[(int64_t)row * W + col];
        }
    }
}

// Tile crops out of images in page-locked HOST memory, read over the link by the kernel itself: a tile's rows are all
// that crosses it, not the image (1/16 of it for 64 x 64 tiles of 256 x 256 images).  What bounds it: the link, which
// carries whole lines, a row of 64 bytes touching up to two of them: 1024 such tiles take 0.63 ms, the copy of
// the images 3.52 ms (57 GB/s).  It runs beside the convolutions of the chunk before, whose workgroups fill a compute
// unit each, so it is a few large workgroups (kGatherLds of LDS: one to a compute unit) on compute units those
// leave free, a dword per lane, every lane of the workgroup with a request on its way: 8 workgroups take 0.59 / 0.93 / 2.5
// ms for 1024 tiles of 32 / 64 / 128, 16 of them 0.32 / 0.65 / 1.78, 256 no less than that.
constexpr int kGatherThreads = 1024;
constexpr int kGatherLds = 84 * 1024; // more than half of a compute unit's
template <bool WORDS>
__global__ __launch_bounds__(kGatherThreads) void gather_host_tiles_kernel(const uint8_t *__restrict__ img, int planes, int H, int W,
                                                                const int32_t *__restrict__ off, int tile,
                                                                uint8_t *__restrict__ out)
{
    typedef const uint32_t __attribute__((address_space(1))) *host_word_t;
    const uint32_t wpr = WORDS ? tile >> 2 : tile; // dwords / bytes per output row
    const uint32_t row0 = threadIdx.x / wpr, col0 = threadIdx.x - row0 * wpr;
    const uint32_t drow = kGatherThreads / wpr, dcol = kGatherThreads - drow * wpr; // what that many more dwords are
    for (int p = blockIdx.x; p < planes; p += gridDim.x) {
        int oy = 0, ox = 0;
        if (off) {
            oy = clampi(off[2 * (p / 3)], 0, H - tile);
            ox = clampi(off[2 * (p / 3) + 1], 0, W - tile);
        }
        // the tile's first byte as an aligned dword (the same for the whole workgroup) + byte offset
        const uintptr_t first = (uintptr_t)(img + p * (int64_t)H * W + (int64_t)oy * W + ox);
        const uintptr_t base = first & ~(uintptr_t)3;
        const uint32_t skew = (uint32_t)first & 3u;
        uint8_t *dst = out + p * (int64_t)tile * tile;
        uint32_t row = row0, col = col0;
        for (uint32_t idx = threadIdx.x; idx < wpr * tile; idx += kGatherThreads) {
            const uint32_t o = row * W + (WORDS ? col * 4 : col) + skew;
            const uint32_t lo = *(host_word_t)(base + (o & ~3u));
            if (WORDS) { // the second dword is another one only where the first does not hold all four bytes
                const uint32_t hi = *(host_word_t)(base + ((o + 3) & ~3u));
                *(uint32_t *)(dst + idx * 4) = __builtin_amdgcn_alignbyte(hi, lo, o & 3u);
            } else {
                dst[idx] = (uint8_t)(lo >> (8 * (o & 3u)));
            }
            col += dcol;
            row += drow;
            if (col >= wpr) {
                col -= wpr;
                ++row;
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// Variance-based tile selection (Listing 1 of the paper, `select_patch`): windows of win x win pixels at
// a stride that divides win; score of a window = sum over channels of w_c * (n S2_c - S1_c^2), i.e. the
// channel's unbiased variance up to the common factor n (n-1); the first window with the largest score
// is the tile.  HBM-bound: every pixel that lies in some window is read exactly once.
//
// One workgroup per image, of THREADS threads.  The image is cut into cells of stride x stride pixels; a window is a square of
// (win / stride)^2 cells.  Phase 1: every lane walks down a run of rows of one 16-byte (or 1-byte) column
// chunk, of one colour or of all three, sums x (v_sad_u8) and x^2 (v_dot4_u32_u8) in registers and
// adds them to the cell's 32-bit sums in LDS when it crosses into the next cell row.  Phase 2: one lane per window adds up its cells (64 bit),
// forms the exact integers n S2 - S1^2, and the score in float64 in a fixed order with no fused
// multiply-add; a workgroup reduction picks the first maximum.
// A launch of fewer images than compute units waits for the round trips of its only wave of workgroups: 1024 threads an image
// instead of 256 where that is the faster way (select_threads).  Its length is then a chain: quotients by small products instead
// of integer divisions, a window's six look-ups at a time and the best window by DPP moves instead of shuffles took one image of
// 256 x 256, windows of 64 at strides of 32, from 5.9 to 4.7 us, 16 of 384 x 384 at 16 from 14.6 to 12.9, 600 of 256 x 256 from
// 20.5 to 19.7.
// ------------------------------------------------------------------------------------------------
constexpr int kMaxCells = 1024; // cells per channel a workgroup can hold

struct SelectArgs {
    int H, W, win, stride;
    int nH, nW;     // windows
    int nCy, nCx;   // cells that lie in some window
    int tx, rows;   // column chunks that THREADS lanes walk down at a time, rows of a run
    float inv_tx, inv_stride, inv_nW;
    double w[3];    // channel weights
};

// a / d for 0 <= a < 2^22 from the rounded 1 / d: a + 0.5 is at least 0.5 / d away from the next whole quotient, the two roundings
// change it by less than a 2^-23 / d.  (An integer division is some forty instructions, and this kernel has one after the other
// before its first load.)
__device__ __forceinline__ int small_quotient(int a, float inv_d) { return (int)(((float)a + 0.5f) * inv_d); }

template <int VEC, int THREADS>
__global__ __launch_bounds__(THREADS) void tile_variance_kernel(const uint8_t *__restrict__ img, SelectArgs a,
                                                            int32_t *__restrict__ off_yx, double *__restrict__ scores)
{
    __shared__ uint32_t s_sum[3][kMaxCells], s_sq[3][kMaxCells];
    __shared__ double s_best[THREADS / 64];
    __shared__ int s_idx[THREADS / 64];
    const int tid = threadIdx.x;
    const int64_t n = blockIdx.x;
    for (int i = tid; i < 3 * kMaxCells; i += THREADS) {
        (&s_sum[0][0])[i] = 0u;
        (&s_sq[0][0])[i] = 0u;
    }
    __syncthreads();

    // ---- phase 1: cell sums
    const int Hc = a.nCy * a.stride, Wc = a.nCx * a.stride; // the part of the image that windows cover
    const int ncx = Wc / VEC;                                // column chunks per row
    const int TX = a.tx, R = a.rows;
    const int rg = small_quotient(tid, a.inv_tx);            // row group
    const int64_t plane = (int64_t)a.H * a.W;
    const uint8_t *base = img + n * 3 * plane;
    // colours a lane has on their way together: all of them where few bytes are (bytes instead of 16 at a time, few images)
    constexpr int TOGETHER = VEC == 1 || THREADS > 256 ? 3 : 1;
    if (rg * R < Hc && (rg + 1) * TX <= THREADS) { // (a rest of the lanes makes no group)
        const int r0 = rg * R, r1 = min(Hc, r0 + R);
        for (int c0 = 0; c0 < 3; c0 += TOGETHER)
            for (int cx = tid - rg * TX; cx < ncx; cx += TX) {
                const int cellx = small_quotient(cx * VEC, a.inv_stride);
                const uint8_t *col = base + c0 * plane + cx * VEC;
                for (int seg = r0; seg < r1;) { // the run's rows, one cell row at a time
                    const int cy = small_quotient(seg, a.inv_stride);
                    const int seg_end = min(r1, (cy + 1) * a.stride);
                    uint32_t s1[TOGETHER] = {}, s2[TOGETHER] = {};
#pragma unroll 4
                    for (int r = seg; r < seg_end; ++r) { // independent loads: several in flight per lane
#pragma unroll
                        for (int c = 0; c < TOGETHER; ++c) {
                            const uint8_t *p = col + c * plane + (int64_t)r * a.W;
                            if (VEC == 16) {
                                const uint4 v = *(const uint4 *)p;
                                s1[c] = __builtin_amdgcn_sad_u8(v.x, 0u, s1[c]);
                                s1[c] = __builtin_amdgcn_sad_u8(v.y, 0u, s1[c]);
                                s1[c] = __builtin_amdgcn_sad_u8(v.z, 0u, s1[c]);
                                s1[c] = __builtin_amdgcn_sad_u8(v.w, 0u, s1[c]);
                                s2[c] = __builtin_amdgcn_udot4(v.x, v.x, s2[c], false);
                                s2[c] = __builtin_amdgcn_udot4(v.y, v.y, s2[c], false);
                                s2[c] = __builtin_amdgcn_udot4(v.z, v.z, s2[c], false);
                                s2[c] = __builtin_amdgcn_udot4(v.w, v.w, s2[c], false);
                            } else {
                                const uint32_t x = *p;
                                s1[c] += x;
                                s2[c] += x * x;
                            }
                        }
                    }
#pragma unroll
                    for (int c = 0; c < TOGETHER; ++c) {
                        atomicAdd(&s_sum[c0 + c][cy * a.nCx + cellx], s1[c]);
                        atomicAdd(&s_sq[c0 + c][cy * a.nCx + cellx], s2[c]);
                    }
                    seg = seg_end;
                }
            }
    }
    __syncthreads();

    // ---- phase 2: window scores, first maximum
    const int k = a.win / a.stride;
    double best = -1.0;                               // scores are >= 0
    int best_idx = 0x7fffffff;
    for (int wi = tid; wi < a.nH * a.nW; wi += THREADS) {
        const int wy = small_quotient(wi, a.inv_nW), wx = wi - wy * a.nW;
        unsigned long long S1[3] = {}, S2[3] = {};
        for (int dy = 0; dy < k; ++dy)
#pragma unroll 2
            for (int dx = 0; dx < k; ++dx) {
                const int cell = (wy + dy) * a.nCx + wx + dx;
#pragma unroll
                for (int c = 0; c < 3; ++c) { // (six look-ups at a time)
                    S1[c] += s_sum[c][cell];
                    S2[c] += s_sq[c][cell];
                }
            }
        double score = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
#pragma clang fp contract(off) // each product and each sum is rounded on its own: no fused multiply-add
            const unsigned long long v = (unsigned long long)(a.win * a.win) * S2[c] - S1[c] * S1[c]; // exact, < 2^53
            const double term = (double)v * a.w[c];
            score = c == 0 ? term : score + term;
        }
        if (scores) scores[n * (int64_t)(a.nH * a.nW) + wi] = score;
        if (score > best) { // ascending wi: the first maximum stays
            best = score;
            best_idx = wi;
        }
    }
    auto take = [&](double o, int oi) {
        if (o > best || (o == best && oi < best_idx)) {
            best = o;
            best_idx = oi;
        }
    };
    // The wavefront's best ends up in its last lane: a lane may meet a candidate twice
    auto step = [&](auto ctrl, auto row_mask) {
        constexpr int CTRL = decltype(ctrl)::value, MASK = decltype(row_mask)::value;
        const uint64_t bits = __builtin_bit_cast(uint64_t, best);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)bits, (int)(uint32_t)bits, CTRL, MASK, 0xf, false);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(bits >> 32), (int)(bits >> 32), CTRL, MASK, 0xf, false);
        const int oi = __builtin_amdgcn_update_dpp(best_idx, best_idx, CTRL, MASK, 0xf, false);
        take(__builtin_bit_cast(double, (uint64_t)hi << 32 | lo), oi);
    };
    typedef std::integral_constant<int, 0xf> AllRows;
    step(std::integral_constant<int, 0xB1>{}, AllRows{});  // quad_perm [1,0,3,2]
    step(std::integral_constant<int, 0x4E>{}, AllRows{});  // quad_perm [2,3,0,1]
    step(std::integral_constant<int, 0x141>{}, AllRows{}); // row_half_mirror
    step(std::integral_constant<int, 0x140>{}, AllRows{}); // row_mirror
    step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{}); // row_bcast:15 into rows 1 and 3
    step(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{}); // row_bcast:31 into rows 2 and 3
    const int used = min(THREADS / 64, (a.nH * a.nW + 63) / 64); // wavefronts with a window
    if (used > 1) {
        if ((tid & 63) == 63) {
            s_best[tid >> 6] = best;
            s_idx[tid >> 6] = best_idx;
        }
        __syncthreads();
    }
    if (tid == 63) {
        for (int v = 1; v < used; ++v) take(s_best[v], s_idx[v]);
        off_yx[2 * n] = best_idx / a.nW * a.stride;
        off_yx[2 * n + 1] = best_idx % a.nW * a.stride;
    }
}

// ------------------------------------------------------------------------------------------------
// Fused pre-processing (Table 1 of the paper: resize to x, centre crop x, to tensor; Appendix A: one pass
// from the raw buffer): raw u8 images, height x width x 3 interleaved, -> planar u8 [3][T][T], where the
// T x T window is either the whole centre crop (T = x) or one tile of it at a per-image origin: only the
// source pixels under that window are touched.  Bilinear, pixel centres at half-integers, fixed point:
// the fraction of a source coordinate is rounded to 11 bits, the four products are exact integers, the
// sum is rounded half up (>> 22).  Integer arithmetic only: the bytes do not depend on the hardware.
//
// One workgroup per (image, strip of rows).  The column taps of the window are computed once into LDS
// (two integer divisions per column), a lane then produces four neighbouring pixels of a row for the
// three colours and writes one dword per plane.  18 KB of tables: eight workgroups a compute unit.  Workgroups take an image's
// strips one after the other, so that what the chip reads at a time lies together: 600 images of 480 x 640 to 256 x 256, with the
// selection and crop behind it, 164.2 -> 159.8 us (all images' first strips, then all their second ones, before).
//
// Enlarging, or making less than half as large, it is bound by the L1's address side: lanes that load from odd addresses are
// served one after the other (52 accesses a load of eight bytes a lane, 27 a load of twelve at multiples of four, which then
// shifts the taps into place: LOAD, preprocess_load).  The 600 images above 132 -> 111 us with the strips below (5.0 TB/s read
// and written: memory), 1024 of 300 x 300 to 128 x 128 windows 34.1 -> 26.7, 4096 of 256 x 256 to windows of 64 31.1 -> 25.1,
// 400 of 300 x 300 to 384 x 384 140 -> 88.  Dropped: the rows' spans staged in LDS by 16-byte loads (111 on the 600 images, slower
// on windows of 64 and 12.3 instead of 11.6 on 64 images); a wavefront's lanes on neighbouring pixels, the bytes dealt to dword stores
// afterwards (as fast on the 600, 104 instead of 88 on the 400: more instructions).
// ------------------------------------------------------------------------------------------------
constexpr int kCoefBits = 11;
constexpr int kTopShift = 32 - 8 - 2 * kCoefBits; // of the vertical weights: the sum's byte comes to the top
constexpr int kMaxTile = 1024; // columns of a window

struct PreArgs {
    int H_in, W_in, x, T;  // raw size, size after resize + crop, window
    int Hr, Wr, cy, cx;    // resized size, origin of the centre crop in it
    float inv_H, inv_W;    // 1 / (2 Hr), 1 / (2 Wr)
    int groups, d_row;     // pixel groups of a row, whole rows that 256 of them are
    float inv_groups;
    int rows_per_block;
    uint32_t strips; // of rows_per_block rows
    uint32_t pitch;  // bytes of a raw row
    int64_t images;  // from the launch's first one to the buffer's end
};

// num / den for 0 <= num < 2^31 and quotients up to 2^15, from the rounded 1 / den: the estimate is off by less than one (three
// roundings of 2^-24 of it).  A third of an integer division's instructions, which a strip's tables mostly were: one image of
// 480 x 640 to 256 x 256 3.69 -> 3.54 us, 1024 of 300 x 300 to windows of 128 x 128 27.3 -> 26.2, 3000 of 100 x 100, windows of 30 x 30, 11.1 ->
// 10.7; launches that memory bounds are the same.
__device__ __forceinline__ int quotient(int num, int den, float inv_den, int &rest)
{
    int q = (int)((float)num * inv_den);
    rest = num - q * den;
    const int up = rest >= den, down = rest < 0;
    q += up - down;
    rest += down ? den : up ? -den : 0;
    return q;
}

// inv_den: 1 / (2 n_res)
__device__ __forceinline__ void source_taps(int dst, int n_in, int n_res, float inv_den, int &i0, int &i1, int &w1)
{
    int num = (2 * dst + 1) * n_in - n_res; // numerator of the source coordinate over 2 * n_res
    const int den = 2 * n_res;
    num = num < 0 ? 0 : num;
    int a, rest;
    i0 = quotient(num, den, inv_den, a);
    if (i0 >= n_in - 1) {
        i0 = n_in - 1;
        a = 0;
    }
    i1 = min(i0 + 1, n_in - 1);
    w1 = quotient(a * (1 << kCoefBits) + n_res, den, inv_den, rest); // round(fraction * 2048)
}

typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));

// One colour of one window pixel, in the top byte, from the eight bytes of either row that hold its taps (top0 top1 above bot0
// bot1).  sel picks the colour's byte of the left tap (low half) and of the right tap (high half), wx = wx0 | wx1 << 16.  The
// horizontal pass is a two-term dot product of 16-bit fields (< 2^19), the vertical pass two 24-bit products with weights of four
// times the size (the sum < 2^32): all full-rate instructions, and the same integers as the plain formula; the byte at the top
// saves the shift, as a permute puts four of them together.
__device__ __forceinline__ uint32_t bilinear_top_byte(uint32_t top0, uint32_t top1, uint32_t bot0, uint32_t bot1, uint32_t sel,
                                                      uint32_t wx, uint32_t wy0, uint32_t wy1)
{
    const uint32_t t = __builtin_amdgcn_perm(top1, top0, sel), b = __builtin_amdgcn_perm(bot1, bot0, sel);
    const uint32_t top = __builtin_amdgcn_udot2(__builtin_bit_cast(ushort2_t, t), __builtin_bit_cast(ushort2_t, wx), 0u, false);
    const uint32_t bot = __builtin_amdgcn_udot2(__builtin_bit_cast(ushort2_t, b), __builtin_bit_cast(ushort2_t, wx), 0u, false);
    return __umul24(top, wy0) + (__umul24(bot, wy1) + (1u << (2 * kCoefBits + kTopShift - 1)));
}
constexpr uint32_t kSelect = 0x0c000c00u; // a byte to bits 0..7 (its number 0..7 is added), one to bits 16..23, zeros between

// Walks the (row, pixel group) pairs of a strip, 256 at a time, without a division per step.
struct StripWalk {
    int row, grp, d_row, d_grp, groups;
    __device__ StripWalk(int tid, const PreArgs &a) : d_row(a.d_row), groups(a.groups)
    {
        row = small_quotient(tid, a.inv_groups);
        grp = tid - row * groups;
        d_grp = 256 - d_row * groups;
    }
    __device__ void next()
    {
        row += d_row;
        grp += d_grp;
        if (grp >= groups) {
            grp -= groups;
            ++row;
        }
    }
};

// LOAD: bytes that a load of a row's taps takes: 12 (whole dwords, shifted into place; eight where those would end behind the
// buffer), 8, 4 (a load for either tap) or 1 (rows of one pixel)
template <int VEC, int LOAD>
__global__ __launch_bounds__(256) void preprocess_kernel(const uint8_t *__restrict__ raw, PreArgs a,
                                                         const int32_t *__restrict__ off, uint8_t *__restrict__ out)
{
    __shared__ uint32_t s_x[kMaxTile], s_y[kMaxTile]; // byte offsets, of a column in a row and of a row in an image (of less than 2^30 bytes)
    __shared__ uint32_t s_wx[kMaxTile], s_sel[kMaxTile];
    __shared__ uint16_t s_wy[kMaxTile];
    const int tid = threadIdx.x;
    const int64_t n = blockIdx.x / a.strips; // an image's strips follow each other
    const int strip = (int)(blockIdx.x - (uint32_t)n * a.strips);
    int oy = 0, ox = 0;
    if (off && a.T < a.x) {
        oy = clampi(off[2 * n], 0, a.x - a.T);
        ox = clampi(off[2 * n + 1], 0, a.x - a.T);
    }
    const int r_begin = strip * a.rows_per_block, r_end = min(a.T, r_begin + a.rows_per_block);
    for (int t = tid; t < a.T; t += 256) {
        int i0, i1, w1;
        source_taps(a.cx + ox + t, a.W_in, a.Wr, a.inv_W, i0, i1, w1);
        // The six bytes of both taps come with ONE (unaligned) load of eight, from the left tap's first byte on or, at the row's
        // end, its last eight: always inside the row.  The byte selector carries where the taps lie in them.  Short rows: a load
        // of four bytes for either tap, the row's last four at its end (preprocess_load).
        const int at = LOAD > 1 ? min(3 * i0, 3 * a.W_in - min(LOAD, 8)) : 3 * i0;
        const int right = LOAD == 4 ? 4 + 3 * i1 - min(at + 3, 3 * a.W_in - 4) : LOAD >= 8 ? 3 * i1 - at : 3;
        s_x[t] = (uint32_t)at;
        s_sel[t] = kSelect + ((uint32_t)(3 * i0 - at) | (uint32_t)right << 16);
        s_wx[t] = (uint32_t)((1 << kCoefBits) - w1) | (uint32_t)w1 << 16;
    }
    for (int t = tid; t < r_end - r_begin; t += 256) {
        int y0, y1, wy1;
        source_taps(a.cy + oy + r_begin + t, a.H_in, a.Hr, a.inv_H, y0, y1, wy1);
        s_y[t] = (uint32_t)y0 * a.pitch;
        s_wy[t] = (uint16_t)(wy1 << kTopShift);
    }
    __syncthreads();
    const int64_t image = (int64_t)a.H_in * a.W_in * 3;
    const uint8_t *img = raw + n * image;
    uint8_t *dst = out + n * 3 * (int64_t)a.T * a.T;
    const int64_t plane = (int64_t)a.T * a.T;
    // Byte offsets count from the dword that the image begins in (LOAD == 12; the buffer begins with one), and so many bytes are there
    const uint32_t head = LOAD == 12 ? (uint32_t)(uintptr_t)img & 3u : 0u;
    const uint8_t *base = img - head;
    const uint32_t there = (uint32_t)min((int64_t)0x7fffffff, (a.images - n) * image + head);
    const uint32_t last_row = (uint32_t)(a.H_in - 1) * a.pitch;
    for (StripWalk w(tid, a); w.row < r_end - r_begin; w.next()) {
        const int tx = w.grp * VEC;
        const uint32_t wy1 = s_wy[w.row], wy0 = (1u << (kCoefBits + kTopShift)) - wy1;
        const uint32_t y0 = s_y[w.row] + head, y1 = min(s_y[w.row] + a.pitch, last_row) + head; // (y0 <= y1)
        uint32_t p[VEC][2][2]; // [pixel][row]: the three colours of the left tap, then of the right one, somewhere in eight bytes
        uint32_t at[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) at[v] = s_x[tx + v];
        auto eight = [&] {
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                __builtin_memcpy(p[v][0], base + (y0 + at[v]), 8);
                __builtin_memcpy(p[v][1], base + (y1 + at[v]), 8);
            }
        };
        if (LOAD == 12) {
            if (y1 + at[VEC - 1] + 12u <= there) {
                uint32_t e[VEC][2][3];
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    __builtin_memcpy(e[v][0], __builtin_assume_aligned(base + ((y0 + at[v]) & ~3u), 4), 12);
                    __builtin_memcpy(e[v][1], __builtin_assume_aligned(base + ((y1 + at[v]) & ~3u), 4), 12);
                }
#pragma unroll
                for (int v = 0; v < VEC; ++v)
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        const uint32_t shift = (r ? y1 : y0) + at[v];
                        p[v][r][0] = __builtin_amdgcn_alignbyte(e[v][r][1], e[v][r][0], shift);
                        p[v][r][1] = __builtin_amdgcn_alignbyte(e[v][r][2], e[v][r][1], shift);
                    }
            } else {
                eight();
            }
        } else if (LOAD == 8) {
            eight();
        } else if (LOAD == 4) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                const uint32_t b1 = min(at[v] + 3u, a.pitch - 4u);
                __builtin_memcpy(&p[v][0][0], base + (y0 + at[v]), 4);
                __builtin_memcpy(&p[v][0][1], base + (y0 + b1), 4);
                __builtin_memcpy(&p[v][1][0], base + (y1 + at[v]), 4);
                __builtin_memcpy(&p[v][1][1], base + (y1 + b1), 4);
            }
        } else {
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                const uint32_t b1 = min(at[v] + 3u, a.pitch - 3u);
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const uint8_t *left = base + ((r ? y1 : y0) + at[v]), *right = base + ((r ? y1 : y0) + b1);
                    p[v][r][0] = left[0] | left[1] << 8 | left[2] << 16 | (uint32_t)right[0] << 24;
                    p[v][r][1] = right[1] | right[2] << 8;
                }
            }
        }
        uint32_t q[3][VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            const uint32_t wx = s_wx[tx + v], sel = s_sel[tx + v];
#pragma unroll
            for (int c = 0; c < 3; ++c) q[c][v] = bilinear_top_byte(p[v][0][0], p[v][0][1], p[v][1][0], p[v][1][1], sel + c * 0x10001u, wx, wy0, wy1);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            uint8_t *to = dst + c * plane + (int64_t)(r_begin + w.row) * a.T + tx;
            if (VEC == 4) {
                const uint32_t low = __builtin_amdgcn_perm(q[c][1 % VEC], q[c][0], 0x0c0c0703u), high = __builtin_amdgcn_perm(q[c][3 % VEC], q[c][2 % VEC], 0x07030c0cu);
                *(uint32_t *)to = low | high;
            } else {
                *to = (uint8_t)(q[c][0] >> 24);
            }
        }
    }
}

} // namespace

void preprocess_resized_shape(int H_in, int W_in, int x, int *Hr, int *Wr)
{
    if (H_in <= W_in) {
        *Hr = x;
        *Wr = (int)std::max<int64_t>(x, (int64_t)x * W_in / H_in);
    } else {
        *Hr = (int)std::max<int64_t>(x, (int64_t)x * H_in / W_in);
        *Wr = x;
    }
}

bool preprocess_supported(int H_in, int W_in, int x, int T)
{
    if (H_in <= 0 || W_in <= 0 || x <= 0 || T <= 0 || T > x || T > kMaxTile) return false;
    if (H_in > 16384 || W_in > 16384) return false;
    int Hr, Wr;
    preprocess_resized_shape(H_in, W_in, x, &Hr, &Wr);
    // (2 * dst + 1) * n_in and fraction * 2048 must stay below 2^31
    return Hr <= 16384 && Wr <= 16384 && (int64_t)(2 * (int64_t)std::max(Hr, Wr) + 1) * std::max(H_in, W_in) < (1LL << 31) &&
           (int64_t)2 * std::max(Hr, Wr) * 2048 < (1LL << 31);
}

// Strips a T x T window is cut into when a launch has N of them.  Enough workgroups for one wave over the chip (eight fit a compute
// unit); beyond it short strips, so that the rows that are read at a time lie together and no last wave is nearly empty: 600
// images of 480 x 640 to 256 x 256 125 us in 4 strips, 121 in 8, 115 in 16, 111 in 32.
// But a strip's column taps are its own: two turns of 256 pixel groups for each, four where a window has less than 16 (1024
// windows of 64 x 64 out of 512 x 512 13.7 us in 1 to 4 strips, 14.8 in 8; 2048 of them 17.8 in one, 23.3 in 8; 3000 of 30 x 30
// 10.4 in one, 12.0 in two; 1024 of 128 x 128 out of 300 x 300 24.5 in 4, 25.3 in 8, 29.8 in 16, out of 480 x 480 44.0, 42.3, 38.4).
int preprocess_strips(int64_t N, int T, bool vec)
{
    const int64_t turns = (int64_t)T * (vec ? T / 4 : T) / 256;
    const int64_t one_wave = 2048 / N, several = turns >= 16 ? turns / 2 : turns / 4;
    const int strips = (int)std::min<int64_t>((T + 7) / 8, std::max<int64_t>(1, std::max(one_wave, several)));
    const int rows = (T + strips - 1) / strips;
    return (T + rows - 1) / rows;
}

// Bytes per load of the taps.  Rows of two pixels have no room for eight, rows of one none for four.  1000 images to 256 x 256, four /
// eight bytes: images of 2 x 3 112 / 123 us, 3 x 4 104 / 90; of 2 x 2, one byte / four: 125 / 84.  Dwords (12 bytes) as long as
// neighbouring left taps lie less than two pixels apart: eight / twelve bytes, 1024 windows of 128 x 128 out of 256 columns of 200
// raw ones 34 / 25, of 400 40 / 31, of 500 53 / 47, of 512 47 / 48; further apart there is no difference up to 700 and then the
// longer load touches more lines: 1000 24 / 25, 1500 16 / 18.5.
static int preprocess_load(int W_in, int Wr, const uint8_t *raw)
{
    if (W_in < 4) return W_in >= 2 ? 4 : 1;
    return W_in < 2 * Wr && (uintptr_t)raw % 4 == 0 ? 12 : 8;
}

hipError_t launch_preprocess(const uint8_t *raw, int64_t N, int H_in, int W_in, int x, const int32_t *off, int T,
                             uint8_t *out, hipStream_t s)
{
    if (N <= 0) return hipSuccess;
    PreArgs a{};
    a.H_in = H_in; a.W_in = W_in; a.x = x; a.T = T;
    preprocess_resized_shape(H_in, W_in, x, &a.Hr, &a.Wr);
    a.cy = (a.Hr - x) / 2;
    a.cx = (a.Wr - x) / 2;
    const bool vec = T % 4 == 0 && ((uintptr_t)out & 3u) == 0;
    const int strips = preprocess_strips(N, T, vec);
    a.rows_per_block = (T + strips - 1) / strips;
    a.strips = (uint32_t)strips;
    a.groups = vec ? T / 4 : T;
    a.d_row = 256 / a.groups;
    a.inv_groups = 1.0f / (float)a.groups;
    a.inv_H = 1.0f / (float)(2 * a.Hr);
    a.inv_W = 1.0f / (float)(2 * a.Wr);
    a.pitch = 3u * (uint32_t)W_in;
    const int64_t kMaxGrid = (1LL << 30) / strips;
    for (int64_t n0 = 0; n0 < N; n0 += kMaxGrid) {
        const int64_t cnt = N - n0 < kMaxGrid ? N - n0 : kMaxGrid;
        const uint8_t *raw0 = raw + n0 * (int64_t)H_in * W_in * 3;
        const int32_t *off0 = off ? off + 2 * n0 : nullptr;
        uint8_t *out0 = out + n0 * 3 * (int64_t)T * T;
        const dim3 grid((unsigned)(cnt * strips));
        a.images = N - n0;
        auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, raw0, a, off0, out0); };
        const int load = preprocess_load(W_in, a.Wr, raw0);
        if (load == 12) launch(vec ? preprocess_kernel<4, 12> : preprocess_kernel<1, 12>);
        else if (load == 8) launch(vec ? preprocess_kernel<4, 8> : preprocess_kernel<1, 8>);
        else if (load == 4) launch(vec ? preprocess_kernel<4, 4> : preprocess_kernel<1, 4>);
        else launch(vec ? preprocess_kernel<4, 1> : preprocess_kernel<1, 1>);
    }
    return hipGetLastError();
}

bool select_tiles_supported(int H, int W, int win, int stride)
{
    if (win <= 0 || stride <= 0 || win > H || win > W || win % stride != 0 || win > 512 || stride > 256) return false;
    const int nH = (H - win) / stride + 1, nW = (W - win) / stride + 1, k = win / stride;
    return (int64_t)(nH - 1 + k) * (nW - 1 + k) <= kMaxCells;
}

// Threads an image.  256 / 1024 threads, us: byte by byte 256 images of 250 x 250 66 / 19, 256 of 500 x 500 242 / 41.  16 bytes at a time:
// one image of 320 x 320 14.3 / 9.8, 32 of 512 x 512 13.2 / 10.7, 256 of 224 x 224 16.8 / 9.2, 256 of 384 x 384 31.6 / 26.0, of 416 x
// 416 34.4 / 28.1.  Images that are larger, or wide, and more than the L2s hold fill the memory's queues with 256 threads: 200 of
// 512 x 512 27.2 / 29.8, 64 of 480 x 640 33.8 / 38.8, 64 of 768 x 768 61.3 / 71.2, 200 of 288 x 512 18.9 / 22.4.  (Within the L2s, of
// 28 sizes one loses by 1024 threads: 720 x 1280, 37.0 / 39.2.)
static int select_threads(int64_t N, int H, int W, bool wide)
{
    if (N > 256) return 256;
    if (!wide) return 1024;
    const bool small = W <= 416 && (int64_t)H * W <= 416 * 416, cached = 3 * N * H * W <= 24 << 20;
    return small || cached ? 1024 : 256;
}

hipError_t launch_select_tiles_variance(const uint8_t *img, int64_t N, int H, int W, int win, int stride,
                                        const double w[3], int32_t *off_yx, double *scores, hipStream_t s)
{
    if (N <= 0) return hipSuccess;
    SelectArgs a{};
    a.H = H; a.W = W; a.win = win; a.stride = stride;
    a.nH = (H - win) / stride + 1;
    a.nW = (W - win) / stride + 1;
    const int k = win / stride;
    a.nCy = a.nH - 1 + k;
    a.nCx = a.nW - 1 + k;
    a.inv_stride = 1.0f / (float)stride;
    a.inv_nW = 1.0f / (float)a.nW;
    for (int c = 0; c < 3; ++c) a.w[c] = w[c];
    // 16-byte loads: chunks must not straddle cells and every row of every image must start 16-byte aligned
    const bool wide = stride % 16 == 0 && W % 16 == 0 && ((uintptr_t)img & 15u) == 0;
    const int64_t kMaxGrid = 1LL << 30;
    for (int64_t n0 = 0; n0 < N; n0 += kMaxGrid) {
        const int64_t cnt = N - n0 < kMaxGrid ? N - n0 : kMaxGrid;
        const uint8_t *img0 = img + n0 * 3 * (int64_t)H * W;
        double *sc0 = scores ? scores + n0 * (int64_t)(a.nH * a.nW) : nullptr;
        auto launch = [&](auto kernel, int threads) {
            const int chunks = a.nCx * stride / (wide ? 16 : 1), groups = threads / std::min(chunks, threads);
            a.tx = std::min(chunks, threads);
            a.rows = (a.nCy * stride + groups - 1) / groups;
            a.inv_tx = 1.0f / (float)a.tx;
            hipLaunchKernelGGL(kernel, dim3((unsigned)cnt), dim3(threads), 0, s, img0, a, off_yx + 2 * n0, sc0);
        };
        if (select_threads(N, H, W, wide) == 1024) launch(wide ? tile_variance_kernel<16, 1024> : tile_variance_kernel<1, 1024>, 1024);
        else launch(wide ? tile_variance_kernel<16, 256> : tile_variance_kernel<1, 256>, 256);
    }
    return hipGetLastError();
}

HostPlan plan_host_upload(int C, int n_blocks, int final_slices, int H, int W, int tile, int chunk_images, int used, int num_cu)
{
    HostPlan p{};
    p.first_workgroups = 32;
    // Bytes a tile's rows touch on average, in pieces of 64, against the image's: 64 x 64 tiles of 256 x 256 images 0.12 (0.63 ms
    // for 1024 against 3.52 for the copy), 128: 0.37 (1.75), 192: 0.75 (2.66), 256: 1.2 (3.50).  The copy needs no compute units:
    // the gather has to halve the bytes.
    if (2 * (int64_t)tile * (tile + 63) > (int64_t)H * W) return p;
    p.first = true; // nothing runs beside it
    if (used < 2) {
        p.rest = true;
        p.rest_workgroups = p.first_workgroups;
        return p;
    }
    // The gather of a later chunk runs beside the kernels of the chunk before, which leave it its compute units and take 1.07 ..
    // 1.16 times as long for it: it is worth having only where the copy takes longer than that, i.e. where the link is the
    // bound.  (Six chunks, later ones copied / gathered, ms: 1024 images of 256 x 256 with tiles of 64 20.1 / 11.3, of 65 21.6 / 20.5, of 72
    // 22.0 / 22.8, of 80 24.5 / 25.1; 512 of 512 x 512, 160 42.8 / 39.9, 176 43.6 / 45.0.)  The estimate: picoseconds per block and
    // pixel of the tiles' column blocks, 57 GB/s.
    const double columns = 64.0 * ((tile + 63) / 64);
    const double tile_s = tile * columns * 1e-12 * (n_blocks * (C == 64 ? 50.0 : 26.0) + final_slices * (C == 64 ? 50.0 : 32.0));
    p.rest = num_cu >= 64 && 1.1 * tile_s * chunk_images < 3.0 * H * W * chunk_images / 57e9;
    // 8 or 16 workgroups (figures above): 8 where the work on a tile's own pixels takes longer than they do.  (On the column
    // blocks tiles of 32 would get 8 as well: 6 chunks of 1024 5.84 ms instead of 5.53 with 16.)
    if (p.rest) p.rest_workgroups = p.lent_cu = tile_s * tile / columns > 3.0 * tile * 5.5e-9 ? 8 : 16;
    return p;
}

hipError_t launch_gather_host_tiles(const uint8_t *img, int64_t N, int H, int W, const int32_t *off, int tile, uint8_t *out,
                                    int workgroups, hipStream_t s)
{
    if (N <= 0) return hipSuccess;
    if (N > (1 << 29)) return hipErrorInvalidValue;
    const int planes = (int)N * 3;
    const dim3 grid((unsigned)std::min(planes, workgroups));
    // (dwords: the output is dword aligned; an aligned dword that holds a byte of the images never leaves its page)
    if (tile % 4 == 0 && ((uintptr_t)out & 3u) == 0)
        hipLaunchKernelGGL(gather_host_tiles_kernel<true>, grid, dim3(kGatherThreads), kGatherLds, s, img, planes, H, W, off, tile, out);
    else
        hipLaunchKernelGGL(gather_host_tiles_kernel<false>, grid, dim3(kGatherThreads), kGatherLds, s, img, planes, H, W, off, tile, out);
    return hipGetLastError();
}

hipError_t launch_extract_tiles(const uint8_t *img, int64_t N, int H, int W, const int32_t *off, int tile,
                                uint8_t *out, hipStream_t s)
{
    if (N <= 0) return hipSuccess;
    // dword path: output rows are whole dwords, the output is dword aligned, and every aligned input
    // dword that overlaps the image buffer lies inside it (base aligned, total size a multiple of 4)
    const bool words = (tile % 4 == 0) && (((uintptr_t)out & 3u) == 0) && (((uintptr_t)img & 3u) == 0) &&
                       (((int64_t)N * 3 * H * W) % 4 == 0);
    const int64_t planes = N * 3;
    // grid.x is limited to 2^31-1; batches beyond that are split
    const int64_t kMaxGrid = 3LL << 28; // whole images per launch
    for (int64_t p0 = 0; p0 < planes; p0 += kMaxGrid) {
        const int64_t cnt = planes - p0 < kMaxGrid ? planes - p0 : kMaxGrid;
        const uint8_t *img0 = img + p0 * (int64_t)H * W;
        const int32_t *off0 = off ? off + 2 * (p0 / 3) : nullptr;
        uint8_t *out0 = out + p0 * (int64_t)tile * tile;
        if (words)
            hipLaunchKernelGGL(extract_tiles_kernel<true>, dim3((unsigned)cnt), dim3(256), 0, s, img0, H, W, off0,
                               tile, out0);
        else
            hipLaunchKernelGGL(extract_tiles_kernel<false>, dim3((unsigned)cnt), dim3(256), 0, s, img0, H, W, off0,
                               tile, out0);
    }
    return hipGetLastError();
}

} // namespace qrm
