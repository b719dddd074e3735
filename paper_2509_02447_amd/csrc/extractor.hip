// Convolutional bit-extractor H_D (Section 4.1 / 4.3 of the paper) for gfx950.
//
// Every 3x3 convolution is an implicit GEMM on the bf16 matrix cores:
//     D[cout][pixel] += W[cout][k] * X[k][pixel],   k = (tap, cin)
// with v_mfma_f32_32x32x16_bf16: A = a 32(cout) x 16(k) weight fragment, B = a 16(k) x 32(pixel)
// activation fragment, D = 32 x 32 fp32 accumulators.  Activations travel between layers as bf16 NHWC,
// so the 8 consecutive channels a lane feeds to the matrix core are one 16-byte load.
//
//  * Weights are stationary in registers: a wavefront owns 32 output channels and keeps all
//    9 * C/16 of their A fragments (144 VGPRs at C = 64) for the lifetime of a persistent workgroup.
//    The folded batch-norm scale is multiplied into the weights at context creation; bias and ReLU are
//    applied to the accumulators on the way out, before the single bf16 rounding per layer.
//  * Workgroups are persistent (one per compute unit, eight wavefronts in two groups of four) and stage
//    rows of pixels in LDS rings with direct-to-LDS loads: a pixel takes C * 2 + 16 bytes, so that the
//    16-byte fragment reads are bank-conflict free, and whatever lies outside the tile arrives as zeros (the
//    bounds check of buffer loads, RowLoader).  Each fragment read from LDS feeds up to three matrix instructions (the three
//    vertical taps that touch that input row).  conv_mid_kernel computes one block per launch (strips of
//    4 rows x 64 columns, the two groups in opposite phases); conv_pair_kernel computes two consecutive
//    blocks per launch and keeps the activations between them in a second LDS ring.
//  * Rows of the weight fragments are permuted so that a lane ends up with 16 consecutive output
//    channels of one pixel: the epilogue writes two 16-byte stores per lane.
//  * The first layer reads the u8 image directly (tile crop + normalisation fused: zero padding is
//    applied in the normalised domain and never looks outside the tile); K = 9 taps x 4 channels (r, g,
//    b, 1 inside the tile) = 36, with the weights as bf16 high part + bf16 residual: 72 of 80.
//  * The last block writes no activations when the final convolution has no ReLU: final conv + global
//    average pool are linear, so nine border-aware channel sums per image are all head_kernel needs to
//    apply the final convolution (fp32 weights), the linear layer, the threshold and the symbol packing.
//    With a final ReLU, conv_mid_kernel<64, MODE_FINAL> or conv_final32_kernel sums the final convolution's output
//    over the pixels.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "qrm_internal.h"
#include "rs_lane.h"

namespace qrm {

namespace {

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// XCD-aware block order: hardware deals consecutive workgroups round-robin to the 8 XCDs; give each XCD
// a contiguous range of work so that neighbouring strips (which share halo rows) meet in one L2.
__device__ __forceinline__ int xcd_virtual_block(int b, int nblocks)
{
    if (nblocks % 8) return b;
    return (b % 8) * (nblocks / 8) + b / 8;
}

// s_waitcnt immediates (gfx9 layout: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt_hi[15:14]).  kWaitVm0
// waits for vmcnt(0) only, OR-ing in n <= 15 gives vmcnt(n); kWaitLgkm0 waits for lgkmcnt(0) only.  The
// builtin, unlike an asm statement, is seen by the compiler's own wait-count bookkeeping, which then does
// not add a full drain of its own later.
constexpr int kWaitVm0 = (7 << 4) | (15 << 8);
constexpr int kWaitLgkm0 = 15 | (3 << 14) | (7 << 4);

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also waits for every outstanding
// global store of the wavefront (a workgroup-scope fence counts direct-to-LDS loads as LDS writes and
// drains the whole vector-memory queue), which would put the write latency of a strip's output on the
// critical path of the next strip.  Callers wait for their direct-to-LDS loads themselves.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0); // own LDS reads / writes are done
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Passes a per-lane value through an empty asm statement: what is derived from the result is recomputed
// where it is used instead of being hoisted and kept in registers across the matrix loop.
__device__ __forceinline__ int pin_in_loop(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x2 __attribute__((ext_vector_type(2)));

// Activations are rounded to bf16 once per layer.  Round-to-nearest makes the same error wherever the value
// is the same: on a flat or smooth image every pixel of a channel is off in the same direction, and that part
// of the error survives the global average pool (measured: up to 3.4e-2 of a logit on one-colour images,
// against 2e-3 on noise).  The rounding is therefore dithered by position: a pixel adds a fraction u(x, y) of a
// bf16 step to the value's bits and truncates, u in [0, 1) a fixed pseudo-random function of the pixel's place
// in the tile (an integer hash: an ordered pattern would line up with regular image content such as a
// checkerboard).  Single values are off by up to one step instead of half a step; sums over pixels, which is
// all the method looks at, come out unbiased.  Deterministic: the same pixel always gets the same u.
// One hash per group of rows a wavefront finishes together (the group's first row; the only full 32-bit multiply
// is the column's share, the row's share is the same for the whole wavefront and lives on the scalar unit); the
// other rows of the group take the same fraction shifted by a half or by quarters of a step, which spreads the
// fractions of vertically neighbouring pixels evenly.
__device__ __forceinline__ uint32_t dither16(int x, int y)
{
    uint32_t h = (uint32_t)x * 0x9E3779B1u + (uint32_t)y * 0x85EBCA77u;
    h ^= h >> 15;
    h = __umul24(h, 0x00C1B3C5u); // low 24 bits x 24 bits: the product's upper half depends on all of them
    return h >> 16;
}

// 16 consecutive floats of LDS, e.g. a lane's biases
__device__ __forceinline__ f32x16 load16(const float *p)
{
    f32x16 v;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const f32x4 w = *(const f32x4 *)(p + 4 * q);
        v[4 * q] = w[0]; v[4 * q + 1] = w[1]; v[4 * q + 2] = w[2]; v[4 * q + 3] = w[3];
    }
    return v;
}

// two fp32 -> packed bf16, each truncated after `dither` (< 2^16) has been added to its bits, with ReLU
// applied on the packed pair: a negative bf16 has its sign bit set, i.e. is negative as a 16-bit integer, so
// max(.,0) on the halves clamps it.  (Plain instructions: the compiler puts the wait states a matrix result
// needs in front of its own instructions only, never in front of an asm statement.)
__device__ __forceinline__ uint32_t pack_bf16_relu(float a, float b, uint32_t dither, bool relu)
{
    const uint32_t ua = __builtin_bit_cast(uint32_t, a) + dither, ub = __builtin_bit_cast(uint32_t, b) + dither;
    const uint32_t p = __builtin_amdgcn_perm(ub, ua, 0x07060302u); // the high halves: a's below b's
    s16x2 q = __builtin_bit_cast(s16x2, p);
    if (relu) q = __builtin_elementwise_max(q, (s16x2){0, 0});
    return __builtin_bit_cast(uint32_t, q);
}

// ------------------------------------------------------------------------------------------------
// conv3x3 C -> C on bf16 NHWC activations.  One strip = kRows x kTileW output pixels.
// ------------------------------------------------------------------------------------------------
template <int C>
struct MidCfg {
    static constexpr int KC = C / 16;                 // 16-channel k chunks per tap
    static constexpr int NCB = C / 32;                // 32-wide output channel blocks
    static constexpr int PS = C * 2 + 16;             // LDS bytes per pixel: C bf16 + one 16-byte pad slot
    static constexpr int SPP = PS / 16;               // 16-byte slots per pixel
    static constexpr int ROW_SLOTS = kHaloW * SPP;    // slots of one staged row (halo columns included)
    static constexpr int PIECES = (ROW_SLOTS + 63) / 64; // wavefront-wide direct-to-LDS loads per row
    static constexpr int ROWB = ROW_SLOTS * 16;       // LDS bytes per staged row: rows are packed, the last piece is partial
    static constexpr int QPW = (PIECES + 3) / 4;      // pieces of a row one wavefront is responsible for
};

typedef const __attribute__((address_space(1))) void *gptr_t;
typedef const __attribute__((address_space(1))) uint32_t *global_word_t;
typedef const __attribute__((address_space(4))) int32_t *scalar_ints_t; // what no launch writes while it runs, loaded into scalar registers
typedef __attribute__((address_space(3))) void *lptr_t;
typedef uint32_t lrow_t; // LDS byte address
__device__ __forceinline__ lrow_t lds_address(const void *p)
{
    return (lrow_t)(uintptr_t)(const __attribute__((address_space(3))) uint8_t *)p;
}

// Asynchronous staging of rows of activations into LDS with direct-to-LDS buffer loads.  A staged row (the halo columns
// included) is cut into PIECES pieces of 64 slots of 16 bytes; one wavefront-wide load fills one piece (1 KiB of LDS from
// row + piece * 1024 on), lane l supplying slot piece * 64 + l = (column, 8-channel chunk).  Wavefront w (0..3) of the
// loading group always handles pieces w, w + 4, ..
// Pixels outside the tile must read as zero (zero padding of the convolution).  That is the bounds check of the buffer
// instruction: what lies outside the image's buffer arrives as zeros and asks nothing of memory.  Rows above / below the tile
// see a buffer of no bytes; halo columns outside the tile and the padding slots of a pixel get an offset beyond any image
// (kOutside).  A load is then a scalar row offset and a per-lane offset that only changes with the column block: two or three
// scalar instructions where 64-bit addresses selected per lane against a block of zeros took eight vector ones, which made the
// loading group of conv_mid_kernel the longer one (3200 of a phase's 6200 cycles went into the loads of a strip): 100 tiles of
// 75 x 100, seven blocks and a final ReLU 438.0 -> 415.8 us, 333 of 64 x 64 588.6 -> 580.0, 4096 of them 6654 -> 6592.
// The caller waits (s_waitcnt vmcnt) and passes a barrier before anyone reads the rows.
constexpr uint32_t kOutside = 0x80000000u; // above kMaxImageActBytes

// one wavefront-wide load: 16 bytes per lane from offset voff (per lane) + soff of the `bytes` bytes at `buf`
__device__ __forceinline__ void load_lds16(const uint8_t *buf, uint32_t bytes, uint32_t voff, int soff, uint8_t *dst)
{
    __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(buf), 0, (int)bytes, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lptr_t)dst, 16, voff, soff, 0, 0);
}

// 16 bytes per lane to offset voff + soff of the `bytes` bytes at `buf`; what lies outside is dropped
__device__ __forceinline__ void store16(void *buf, uint32_t bytes, uint32_t voff, int soff, u32x4 v)
{
    __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(buf, 0, (int)bytes, 0x00020000);
    __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, voff, soff, 0);
}

// The loads of launches whose workgroups hand data to each other (conv_chain_kernel): at the scope of the device, so that they do not
// find what the compute unit's own cache holds of earlier contents.
constexpr int kDeviceScope = 16; // the instructions' sc1 bit
__device__ __forceinline__ void load_lds16c(const uint8_t *buf, uint32_t bytes, uint32_t voff, uint8_t *dst)
{
    __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(buf), 0, (int)bytes, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lptr_t)dst, 16, voff, 0, 0, kDeviceScope);
}
__device__ __forceinline__ u32x4 load16c(const void *buf, uint32_t bytes, uint32_t voff)
{
    __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(buf), 0, (int)bytes, 0x00020000);
    return __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, 0, kDeviceScope);
}
template <int C>
struct RowLoader {
    typedef MidCfg<C> K;
    // per lane and piece: byte offset of the lane's slot in an image row for the column block at column 0 (negative for the
    // halo column left of the tile), or far below zero: no slot (the last piece of a row is partial, the next row starts
    // right behind it), or one of a pixel's padding slots
    static constexpr int32_t kNone = INT32_MIN, kPad = INT32_MIN + 1; // (a row has at most 1900 MiB)
    int32_t off[K::QPW];
    __device__ __forceinline__ RowLoader(int w4, int lane)
    {
#pragma unroll
        for (int k = 0; k < K::QPW; ++k) {
            const int sl = (w4 + 4 * k) * 64 + lane, col = sl / K::SPP, cpos = sl - col * K::SPP;
            off[k] = sl >= K::ROW_SLOTS ? kNone : (cpos < C / 8 ? ((col - 1) * C + cpos * 8) * 2 : kPad);
        }
    }
    // the offsets for the column block at column x0 of rows of row_bytes bytes
    struct Block {
        uint32_t voff[K::QPW];
    };
    __device__ __forceinline__ Block at(int x0, uint32_t row_bytes) const
    {
        Block b;
#pragma unroll
        for (int k = 0; k < K::QPW; ++k) {
            const uint32_t o = (uint32_t)(off[k] + x0 * (C * 2)); // (the marks stay below zero)
            b.voff[k] = o < row_bytes ? o : kOutside;
        }
        return b;
    }
    // row y (of h) of the image at `img` (img_bytes bytes; all the same for the whole wavefront) -> dst
    __device__ __forceinline__ void row(const Block &b, const uint8_t *img, uint32_t img_bytes, int y, int h, uint32_t row_bytes, uint8_t *dst, int w4) const
    {
        const bool rowok = (uint32_t)y < (uint32_t)h;
        const uint32_t bytes = rowok ? img_bytes : 0;
        const int soff = rowok ? y * (int)row_bytes : 0;
#pragma unroll
        for (int k = 0; k < K::QPW; ++k) {
            const int q = w4 + 4 * k; // the same for the whole wavefront
            if (4 * k + 3 < K::PIECES - 1 || (q < K::PIECES && off[k] != kNone))
                load_lds16(img, bytes, b.voff[k], soff, dst + q * 1024);
        }
    }
    // Window rows first_row .. kRows + 1 of the strip whose first output row is y0 (window row r is image row y0 - 1 + r) into
    // row slots (ring_pos + r) mod nslot, a power of two.
    __device__ __forceinline__ void strip(uint8_t *lds, int nslot, const uint8_t *img, uint32_t img_bytes, int h, uint32_t row_bytes, int y0, int x0,
                                          int w4, int first_row = 0, int ring_pos = 0) const
    {
        const Block b = at(x0, row_bytes);
#pragma unroll
        for (int r = 0; r < kRows + 2; ++r) {
            if (r < 2 && r < first_row) continue; // already in LDS (or known to be zero there)
            row(b, img, img_bytes, y0 - 1 + r, h, row_bytes, lds + ((ring_pos + r) & (nslot - 1)) * K::ROWB, w4);
        }
    }
};

// body(std::integral_constant<int, 0>) ... body(std::integral_constant<int, N - 1>) in this order: a loop whose
// counter is a compile-time constant inside the body (assembly operands with immediate constraints need one)
template <int... I, typename F>
__device__ __forceinline__ void unrolled_impl(std::integer_sequence<int, I...>, F &&body)
{
    (body(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void unrolled(F &&body)
{
    unrolled_impl(std::make_integer_sequence<int, N>{}, body);
}

// One matrix operand (16 bytes per lane) from LDS address `row` + OFFSET, and the wait that says it has landed
// (at most PENDING later LDS operations of the wavefront outstanding).  Assembly, tied to the register: the
// compiler, not knowing which direct-to-LDS load fills which bytes, would otherwise drain the whole
// vector-memory queue (stores included) before the first read.
template <int OFFSET>
__device__ __forceinline__ void frag_read(bf16x8 &dst, lrow_t row)
{
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(row), "n"(OFFSET));
}
template <int PENDING>
__device__ __forceinline__ void frag_wait(bf16x8 &frag)
{
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(frag) : "n"(PENDING));
}

// Accumulates RW output rows of one 32-pixel x 32-channel block from the staged strip.
//
// The RW + 2 staged rows feed 1, 2, 3, .., 3, 2, 1 vertical taps; rows are paired (p, p + (RW+2)/2) so
// that every pair feeds the same number of matrix instructions.  A "set" is the four fragments
// {two rows of a pair} x {two 16-channel k chunks} of one horizontal tap: 8 (RW = 4) matrix
// instructions.  Each fragment register is refilled for set s+1 right after the matrix instructions of
// set s that read it, and the scheduler is fenced so that it keeps that order: every LDS read has the
// matrix instructions of the three other fragments (6 x 32 cycles at RW = 4) to land.  The reads and
// their waits are written as assembly: the compiler, not knowing which direct-to-LDS load fills which
// bytes, would otherwise drain the whole vector-memory queue (stores included) before the first read.
// `rowp` holds the LDS byte address of each staged row for this lane.
// The accumulators are not read; the first matrix instruction of every output row starts from `first`: zero, or the bias.
// rows_read() is called when the wavefront has read all it needs of the rows, with the last few matrix instructions still to
// be issued: a step's barrier put there lets the others go on meanwhile.
// The code begins on a boundary of 32 bytes: where its eight-byte instructions happened to straddle those of the instruction
// fetch, a launch took up to a fifth longer (the last pair of 1024 tiles of 64 x 64: 406 us, 487 without).
constexpr f32x16 kZeroAcc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
template <int C, int RW, typename F>
__device__ __forceinline__ void strip_mma(const lrow_t (&rowp)[RW + 2], const bf16x8 (&Wr)[9][C / 16],
                                          f32x16 (&acc)[RW], const f32x16 &first, F &&rows_read)
{
    asm volatile(".p2align 5");
    bool started[RW] = {};
    typedef MidCfg<C> K;
    constexpr int NP = (RW + 2) / 2;  // row pairs
    constexpr int KP = K::KC / 2;     // pairs of k chunks
    constexpr int NS = 3 * KP * NP;   // sets
    constexpr int NF = 4;                   // fragment registers = reads in flight (6 or 8 measure the same)
    constexpr int NT = 4 * NS;              // fragments, in the order they are used: set by set
    bf16x8 f[NF];
    constexpr auto set_row = [](int s2, int j) { return (s2 % NP) + (j & 1) * NP; };
    constexpr auto set_kc = [](int s2, int j) { return 2 * ((s2 / NP) % KP) + (j >> 1); };
    constexpr auto set_dx = [](int s2) { return s2 / (NP * KP); };
    unrolled<NF>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        frag_read<set_dx(t / 4) * K::PS + set_kc(t / 4, t % 4) * 32>(f[t], rowp[set_row(t / 4, t % 4)]);
    });
    __builtin_amdgcn_sched_barrier(0);
    unrolled<NT>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        constexpr int s2 = t / 4, j = t % 4;
        constexpr int dx = set_dx(s2);
        constexpr int r = set_row(s2, j), kc = set_kc(s2, j);
        bf16x8 &fr = f[t % NF];
        if constexpr (t == NT - NF + 1) {
            rows_read();
            __builtin_amdgcn_sched_barrier(0);
        }
        // LDS reads return in order: fragment t has landed once at most the NF - 1 reads issued after it
        // (fewer near the end) are outstanding
        frag_wait<(t + NF <= NT ? NF - 1 : NT - 1 - t)>(fr);
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) {
            const int orow = r - dy;
            if (orow >= 0 && orow < RW) {
                if (!started[orow]) {
                    acc[orow] = mfma32(Wr[dy * 3 + dx][kc], fr, first);
                    started[orow] = true;
                } else {
                    acc[orow] = mfma32(Wr[dy * 3 + dx][kc], fr, acc[orow]);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (t + NF < NT) { // the register is free again: refill it
            constexpr int u = t + NF;
            frag_read<set_dx(u / 4) * K::PS + set_kc(u / 4, u % 4) * 32>(fr, rowp[set_row(u / 4, u % 4)]);
        }
        __builtin_amdgcn_sched_barrier(0);
    });
}

template <int C>
__device__ __forceinline__ void load_weight_frags(bf16x8 (&Wr)[9][C / 16], const bf16_t *wfrag, int blk, int lane)
{
    typedef MidCfg<C> K;
    const bf16x8 *wp = (const bf16x8 *)wfrag + (int64_t)blk * 9 * K::KC * 64 + lane;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap)
#pragma unroll
        for (int kc = 0; kc < K::KC; ++kc) Wr[tap][kc] = wp[(tap * K::KC + kc) * 64];
}

// ---- per-image channel statistics ---------------------------------------------------------------
// Every layer hands the next one per-image channel sums of its (post-ReLU) output.  They serve two
// purposes:
//  (1) weights are bf16 on the matrix cores; the rounding residual W - bf16(W) acts on the mean
//      activation as a constant per output channel, the only part of the rounding error that global
//      average pooling does not wash out.  The consumer adds sum_c rsum[o][c] * mean[c] to its bias
//      (rsum = residual summed over the 9 taps), with mean estimated from every eighth strip of four
//      rows: strips p, p + 8, .. with p = sampled_strip(strips).  A record of C sums is written per sampled
//      piece of the image (sample_records), by whichever wavefront computes that piece; the number of pixels
//      behind an image's records is known beforehand (MeanIn::inv_cnt).  Records exist for sampled rows
//      only: a record per workgroup and wavefront, as many as 128 per image in a small launch and most of them
//      zero, took a consumer longer to read (30 of a block's 42 us for 7 tiles of 128 x 128) than its matrix work.
//  (2) the last conv (C -> n_bits, no ReLU) followed by the global average pool is linear, so it only
//      needs, per channel of the last block's output, the sums over the whole tile, its first / last
//      row, first / last column and four corners (9 numbers): the last block writes no activations but lines
//      of C sums, each over a part of the image that does not depend on how the rows were dealt to workgroups
//      (LastSums), so that its results do not either: in one schedule (a launch per block or all blocks in one, which are the same
//      bits; two blocks a launch) the same image gives the same bits whatever the batch around it and however many compute units
//      the launch has.  (A record of nine sums per workgroup, wavefront and image, the
//      alternative, also was 295 KB per image for the head to read in a launch of 7 tiles of 128 x 128; the lines are 52.)
// Accumulation order is fixed, so results do not depend on scheduling.
__host__ __device__ constexpr int sampled_strip(int strips) { return strips < 4 ? strips - 1 : 3; }

// The sampled channel means of an image, from its mi.recs records, into dst[0 .. C) (LDS) by one wavefront: 16 bytes
// per lane, four loads in flight, i.e. 16 (C = 64) or 32 (C = 32) records per round trip to memory.
template <int C>
struct ImageMeans {
    static constexpr int LPR = C / 4, RPL = 64 / LPR; // lanes per record, records per wavefront-wide load
    f32x4 v[4];
    __device__ __forceinline__ void load(const MeanIn &mi, int n, int lane, int r0)
    {
        const f32x4 *p = (const f32x4 *)(mi.rec + (int64_t)n * mi.recs * C) + lane % LPR;
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = p[min(r0 + u * RPL + lane / LPR, mi.recs - 1) * LPR];
    }
    // load(.., 0) has been called
    __device__ __forceinline__ void finish(const MeanIn &mi, int n, float *dst, int lane)
    {
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int r0 = 0;;) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool ok = r0 + u * RPL + lane / LPR < mi.recs;
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[e] += ok ? v[u][e] : 0.f;
            }
            r0 += 4 * RPL;
            if (r0 >= mi.recs) break;
            load(mi, n, lane, r0);
        }
#pragma unroll
        for (int sh = LPR; sh < 64; sh <<= 1)
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] += __shfl_xor(sum[e], sh);
        if (lane < LPR) {
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] *= mi.inv_cnt;
            *(f32x4 *)(dst + 4 * lane) = sum;
        }
    }
};

// What a workgroup's first image needs before its first step: bias + sum_c rsum[c][o] * mean_n[c] (see MeanIn), by four
// wavefronts, each C/4 outputs, its lanes splitting the sum over c in 64 / (C/4) parts.  Every load is asked for in start(),
// before the wavefront asks for its weights, so that a launch opens with one round trip to memory and not with one for the
// weights, one for the records and four for the residual sums, one after the other; and the group that multiplies later asks
// for its weights only behind the first barrier (72 KiB for either group of two wavefronts, the bulk of what a launch of few
// strips waits for).  7 tiles of 128 x 128, ten launches: 124.5 -> 117.5 us.
template <int C>
struct FirstInit {
    static constexpr int OPW = C / 4, PARTS = 64 / OPW, CP = C / PARTS;
    ImageMeans<C> means;
    float rs[CP], b;
    __device__ __forceinline__ void start(const MeanIn &mi, const float *rsum, const float *bias, int n, int w4, int lane)
    {
        const int o = w4 * OPW + lane % OPW, part = lane / OPW;
        b = bias ? bias[o] : 0.f;
        if (mi.rec && rsum) {
            means.load(mi, n, lane, 0);
#pragma unroll
            for (int k = 0; k < CP; ++k) rs[k] = rsum[(part * CP + k) * C + o];
        }
        asm volatile("" ::: "memory"); // what is asked for behind this stays behind it
    }
    __device__ __forceinline__ void finish(const MeanIn &mi, const float *rsum, int n, int w4, int lane, float *s_mean, float *s_init)
    {
        const int o = w4 * OPW + lane % OPW, part = lane / OPW;
        float d = 0.f;
        if (mi.rec && rsum) {
            means.finish(mi, n, s_mean, lane);
#pragma unroll
            for (int k = 0; k < CP; ++k) d = fmaf(rs[k], s_mean[part * CP + k], d);
#pragma unroll
            for (int sh = OPW; sh < 64; sh <<= 1) d += __shfl_xor(d, sh);
        }
        if (part == 0) s_init[o] = b + d;
    }
};

// Sum over the 32 pixel lanes of one half-wavefront with DPP lane permutes (no LDS traffic, no waits).
// After the four butterfly steps every lane holds the sum of its row of 16 lanes; the last step adds the
// sum of row 0 (2) into row 1 (3).  The total is valid in lanes with px >= 16 only: kSumLane reads it.
constexpr int kSumLane = 16;
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_f(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xf, false));
}
__device__ __forceinline__ float half_sum(float v)
{
    v += dpp_f<0xB1, 0xf>(v);  // quad_perm [1,0,3,2]
    v += dpp_f<0x4E, 0xf>(v);  // quad_perm [2,3,0,1]
    v += dpp_f<0x141, 0xf>(v); // row_half_mirror
    v += dpp_f<0x140, 0xf>(v); // row_mirror
    v += dpp_f<0x142, 0xa>(v); // row_bcast:15 into rows 1 and 3
    return v;
}

// Sums of 16 values per lane over the 32 pixel lanes of one half-wavefront, handed out one value per lane: a
// butterfly that halves the number of values a lane holds while it doubles the number of lanes summed (rows of
// 16 lanes are paired with v_permlane16_swap, then lanes p and 15-p, p and 7-p within 8, p and p^2, p and p^1 with
// DPP moves), 38 instructions instead of 80 for sixteen separate 32-lane sums.  Lane (pxl) ends up with the sum of
// value number reduce16_index(pxl); lanes p and p^1 hold the same one.
__device__ __forceinline__ int reduce16_index(int pxl) { return ((pxl >> 4) & 1) * 8 + ((pxl >> 3) & 1) * 4 + ((pxl >> 2) & 1) * 2 + ((pxl >> 1) & 1); }
__device__ __forceinline__ float reduce16_over_half(const float (&t)[16], int pxl)
{
    float u[8], w[4], x2[2], lo[8], hi[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) { lo[j] = t[j]; hi[j] = t[j + 8]; }
    // v_permlane16_swap_b32 a, b: rows 1 and 3 of a <-> rows 0 and 2 of b.  As assembly: this compiler's builtin
    // hands back the first register for both results.  The instruction must not read a register a vector
    // instruction wrote in the two cycles before it, hence the s_nop in front (the compiler, which keeps such
    // distances for its own instructions, does not look into assembly); the operands are sums the compiler's own
    // instructions formed, so the longer distance behind a matrix instruction has been kept by then.
    asm volatile("s_nop 1\n\t"
                 "v_permlane16_swap_b32 %0, %8\n\tv_permlane16_swap_b32 %1, %9\n\t"
                 "v_permlane16_swap_b32 %2, %10\n\tv_permlane16_swap_b32 %3, %11\n\t"
                 "v_permlane16_swap_b32 %4, %12\n\tv_permlane16_swap_b32 %5, %13\n\t"
                 "v_permlane16_swap_b32 %6, %14\n\tv_permlane16_swap_b32 %7, %15\n\t"
                 "s_nop 1"
                 : "+v"(lo[0]), "+v"(lo[1]), "+v"(lo[2]), "+v"(lo[3]), "+v"(lo[4]), "+v"(lo[5]), "+v"(lo[6]), "+v"(lo[7]),
                   "+v"(hi[0]), "+v"(hi[1]), "+v"(hi[2]), "+v"(hi[3]), "+v"(hi[4]), "+v"(hi[5]), "+v"(hi[6]), "+v"(hi[7]));
#pragma unroll
    for (int j = 0; j < 8; ++j) u[j] = lo[j] + hi[j]; // rows 0, 2: value j over both rows; rows 1, 3: value j + 8
    const bool b3 = (pxl & 8) != 0, b2 = (pxl & 4) != 0, b1 = (pxl & 2) != 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = (b3 ? u[j + 4] : u[j]) + dpp_f<0x140, 0xf>(b3 ? u[j] : u[j + 4]);      // row_mirror
#pragma unroll
    for (int j = 0; j < 2; ++j) x2[j] = (b2 ? w[j + 2] : w[j]) + dpp_f<0x141, 0xf>(b2 ? w[j] : w[j + 2]);    // row_half_mirror
    float y = (b1 ? x2[1] : x2[0]) + dpp_f<0x4E, 0xf>(b1 ? x2[0] : x2[1]);                                    // quad_perm [2,3,0,1]
    y += dpp_f<0xB1, 0xf>(y);                                                                                   // quad_perm [1,0,3,2]
    return y;
}

// Four values of one lane into the wavefront's accumulators with LDS add instructions that return nothing:
// no round trip to wait for (a read-modify-write costs one per call, a dozen per step in the last block).
// Every accumulator has one writer (one lane of one wavefront), LDS executes a wavefront's instructions in
// order, so the sums are formed in program order as before.
__device__ __forceinline__ void lds_accumulate4(float *slot4, const float (&tv)[4], bool pred)
{
    // (written as assembly: the compiler, not knowing which bytes the direct-to-LDS loads in flight fill, would
    // otherwise wait for all of them in front of every one of these updates)
    if (pred) {
        const lrow_t a = lds_address(slot4);
        asm volatile("ds_add_f32 %0, %1\n\tds_add_f32 %0, %2 offset:4\n\tds_add_f32 %0, %3 offset:8\n\tds_add_f32 %0, %4 offset:12"
                     :
                     : "v"(a), "v"(tv[0]), "v"(tv[1]), "v"(tv[2]), "v"(tv[3])
                     : "memory");
    }
}

// Channel sums of the RW output rows (first row yw, column x) held in `acc`, after bias `si` (this lane's
// 16 channels) and ReLU, written to the line of C sums at `dst` (global memory, already offset to the lane's 16
// channels).  Four channels at a time: registers are scarce next to weights and accumulators.  above: the lane's sums over the
// rows above that belong to the line, too.
constexpr float kNoSums[16] = {};
template <int RW>
__device__ __forceinline__ void strip_statistics(const f32x16 (&acc)[RW], const float *si, float *dst, int x, int yw,
                                                 int h, int w, int px, const float (&above)[16] = kNoSums)
{
    const bool colok = (uint32_t)x < (uint32_t)w; // (x = -1: the column left of a wide tile's first block)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const f32x4 bq = *(const f32x4 *)(si + 4 * q);
        float tv[4] = {above[4 * q], above[4 * q + 1], above[4 * q + 2], above[4 * q + 3]}; // sum over valid rows of relu(output)
#pragma unroll
        for (int r = 0; r < RW; ++r)
            if (yw + r < h) {
#pragma unroll
                for (int e = 0; e < 4; ++e) tv[e] += fmaxf(acc[r][4 * q + e] + bq[e], 0.f);
            }
        if (!colok) {
#pragma unroll
            for (int e = 0; e < 4; ++e) tv[e] = 0.f;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) tv[e] = half_sum(tv[e]);
        if (px == kSumLane) *(f32x4 *)(dst + 4 * q) = (f32x4){tv[0], tv[1], tv[2], tv[3]};
        __builtin_amdgcn_sched_barrier(0);
    }
}

// This lane's sums over the RW output rows (first row yw), after bias `si` and a lower bound `low`: 16 channels, zero in
// columns beyond the tile.
template <int RW>
__device__ __forceinline__ void column_sums(float (&t)[16], const f32x16 (&acc)[RW], const float *si, float low, bool colok, int yw, int h,
                                            const float (&above)[16] = kNoSums)
{
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const f32x4 b = *(const f32x4 *)(si + 4 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float v = above[4 * q + e];
#pragma unroll
            for (int r = 0; r < RW; ++r)
                if (yw + r < h) v += fmaxf(acc[r][4 * q + e] + b[e], low); // (the same for the whole wavefront)
            t[4 * q + e] = colok ? v : 0.f;
        }
    }
}

// Last block: the lines of channel sums (LastSums) of the RW output rows held in `acc`.  `lines`: the image's first line,
// offset to the lane's 16 channels; whole / col / row: which of its lines for the whole tile, for the first / last column
// and for the first / last row these are; the latter and the corners are written by the wavefronts that hold a border.
// A sum over the 32 pixel lanes is one butterfly for all 16 channels (reduce16_over_half), as in the fused kernel.
// above: as in strip_statistics; WHOLE false: more rows of the piece follow, only the tile's first and last row are written.
struct LinePlaces {
    int first_col, last_col, rows, last_rows, corners; // as in LastSums
    int whole, col, row;
};
template <int C, int RW, bool WHOLE = true>
__device__ __forceinline__ void last_lines(const f32x16 (&acc)[RW], const float *si, float *lines, const LinePlaces &at, int x, int x0w,
                                           int yw, int h, int w, int px, const float (&above)[16] = kNoSums)
{
    const bool colok = x < w;
    const bool has_first = x0w == 0, has_last = x0w <= w - 1 && w - 1 < x0w + 32; // same for the whole wavefront
    auto summed = [&](int line, const float (&v)[16]) {
        const float y = reduce16_over_half(v, px);
        if ((px & 1) == 0) lines[line * C + reduce16_index(px)] = y;
    };
    auto single = [&](int line, const float (&v)[16], bool pred) {
        if (pred) {
#pragma unroll
            for (int q = 0; q < 4; ++q) *(f32x4 *)(lines + line * C + 4 * q) = (f32x4){v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
        }
    };
    float t[16];
    if (WHOLE) {
        column_sums<RW>(t, acc, si, 0.f, colok, yw, h, above);
        if (has_first) single(at.first_col + at.col, t, x == 0);
        if (has_last) single(at.last_col + at.col, t, x == w - 1);
        summed(at.whole, t);
    }
    const int rl = h - 1 - yw; // image row h-1 relative to this wavefront's rows
    if (yw == 0 || (rl >= 0 && rl < RW)) {
#pragma unroll 1
        for (int which = 0; which < 2; ++which) { // the tile's first row, its last one
            if (which == 0 ? yw != 0 : (rl < 0 || rl >= RW)) continue;
            const int row = which == 0 ? 0 : rl;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                float a = acc[0][v];
#pragma unroll
                for (int r = 1; r < RW; ++r) a = row == r ? acc[r][v] : a;
                t[v] = colok ? fmaxf(a + si[v], 0.f) : 0.f;
            }
            summed((which ? at.last_rows : at.rows) + at.row, t);
            if (has_first) single(at.corners + 2 * which, t, x == 0);
            if (has_last) single(at.corners + 2 * which + 1, t, x == w - 1);
        }
    }
}

struct StatArgs {
    MeanIn tin;         // channel sums of the input (rec null: no correction)
    const float *rsum;  // [c_in][c_out] residual-weight sums of this layer (fp32)
    float *tout;        // lines of sums written by this launch: [n_img][out_recs][C], MODE_FINAL [n_img][out_recs][64 * slices]
    int out_recs;       // lines per image
    int per;            // strips per workgroup
    float low;          // MODE_FINAL: lower bound of an output (0: ReLU; NaN: none, fmaxf(v, NaN) is v, also where v is NaN)
};

constexpr int MODE_MID = 0;  // write activations, sample channel sums from every eighth strip
constexpr int MODE_LAST = 1; // last block: no activations, lines of channel sums (LastSums)
constexpr int MODE_FINAL = 2; // final convolution (C output channels per grid.y slice), summed over the pixels: no activations

constexpr int kMidWaves = 8; // wavefronts of a conv_mid workgroup: two groups of four

constexpr int kMidSlots = 16;   // row slots of its LDS ring (>= 12; a power of two)

// C -> C (+bias, ReLU), bf16 NHWC in / out.  One persistent workgroup of eight wavefronts per CU, two
// wavefronts per SIMD.  The workgroup walks down its run of strips; the two groups of four wavefronts
// take alternate strips and work in opposite phases: in phase p group (p & 1) runs the matrix
// instructions of strip p while the other group adds the bias to, converts and stores strip p-1 and
// issues the direct-to-LDS loads of strip p+2.  One workgroup barrier ends a phase.  The matrix cores thus always have one wavefront per SIMD feeding them while the other
// does the vector / memory work, and every load has a whole phase to land before anyone waits for it.
//
// Staged rows live in a ring of kMidSlots row slots.  Rows are loaded in the order the run needs them, so
// ring position = number of rows loaded before: strip i of the run loads nr(i) new rows at positions
// base(i).. and reads the six rows from wstart(i):
//   i = 0                      : 6 rows,             wstart = base
//   strip below the previous   : 4 rows (two rows are shared with the strip above), wstart = base - 2
//   first strip of a new image : 5 rows (the row above the tile is zero - and so is the last row the
//                                previous strip loaded, which lay below its tile), wstart = base - 1
template <int C, int MODE>
__global__ __launch_bounds__(64 * kMidWaves, 1) void conv_mid_kernel(const uint8_t *__restrict__ in,
                                                                     ConvGeom g, const bf16_t *__restrict__ wfrag,
                                                                     const float *__restrict__ bias, StatArgs st,
                                                                     bf16_t *__restrict__ out)
{
    typedef MidCfg<C> K;
    static_assert(MODE != MODE_FINAL || C == 64, "conv_final32_kernel");
    constexpr int RG = 2 / K::NCB;     // row groups among the 4 wavefronts of a group
    constexpr int RW = kRows / RG;     // output rows per wavefront
    constexpr int NSLOT = kMidSlots;
    constexpr int WIN = kRows + 2;     // staged rows one strip reads
    __shared__ __attribute__((aligned(1024))) uint8_t lds[NSLOT * K::ROWB];
    // bias + rounding-residual correction per image, indexed by image mod 4: it is written two phases
    // before the image's first strip is multiplied and read until one phase after its last, and an
    // image may be a single strip
    __shared__ __attribute__((aligned(16))) float s_init[4][C];
    __shared__ __attribute__((aligned(16))) float s_mean[kMidWaves][C];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave >> 2, w4 = wave & 3;
    const int px = lane & 31, half = lane >> 5;
    const int cb = w4 % K::NCB;
    const int xb = (w4 / K::NCB) & 1;
    const int rg = w4 / (K::NCB * 2);

    const int slice = MODE == MODE_FINAL ? blockIdx.y : 0; // C output channels of the launch

    const int tpi = g.strips * g.colblks; // tiles per image
    const int total = g.n_img * tpi;
    const int vb = xcd_virtual_block(blockIdx.x, gridDim.x);
    const int t_begin = vb * st.per;
    const int ns = min(total, t_begin + st.per) - t_begin; // strips of this workgroup's run
    if (ns <= 0) return;
    const lrow_t lbase = lds_address(lds) + (xb * 32 + px) * K::PS + half * 16;
    const size_t img_bytes = (size_t)g.h * g.w * C * 2;
    const uint32_t row_bytes = (uint32_t)(g.w * C * 2);
    const RowLoader<C> loader(w4, lane);

    // ---- geometry of the strips of the run (tile order: image, column block, strip), kept as counters
    // that are advanced once per phase; all wave-uniform
    struct Geo {
        int i;      // index in the run
        int strip;  // strip within its column of the tile
        int colblk; // column block within the image
        int n;      // image
        int base;   // ring position of its first new row
    };
    auto rows_loaded = [&](const Geo &q) { return q.i == 0 ? WIN : (q.strip == 0 ? WIN - 1 : kRows); };
    auto first_row = [&](const Geo &q) { return WIN - rows_loaded(q); }; // first window row that is loaded
    auto wstart = [&](const Geo &q) { return q.base - first_row(q); };
    auto advance = [&](Geo &q) {
        q.base += rows_loaded(q);
        ++q.i;
        if (++q.strip == g.strips) {
            q.strip = 0;
            if (++q.colblk == g.colblks) {
                q.colblk = 0;
                ++q.n;
            }
        }
    };
    Geo gc{0, t_begin % g.strips, (t_begin / g.strips) % g.colblks, t_begin / tpi, 0}; // strip p
    Geo g1 = gc;                                                                          // strip p + 1
    advance(g1);
    Geo g2 = g1;                                                                          // strip p + 2
    advance(g2);
    Geo gp = gc;                                                                          // strip p - 1 (from phase 1 on)

    auto issue = [&](const Geo &q) {
        loader.strip(lds, NSLOT, in + (size_t)q.n * img_bytes, (uint32_t)img_bytes, g.h, row_bytes, q.strip * kRows, q.colblk * kTileW, w4,
                                     first_row(q), wstart(q));
    };
    // s_init[n & 3][o] = bias[o] + sum_c rsum[c][o] * mean_n[c], by the four wavefronts of one group:
    // each takes C/4 outputs, its lanes split the sum over c in 64 / (C/4) parts
    auto prepare_init = [&](int n) {
        constexpr int OPW = C / 4, PARTS = 64 / OPW, CP = C / PARTS;
        const int lane = pin_in_loop(tid & 63);
        const int o = w4 * OPW + lane % OPW, part = lane / OPW;
        float d = 0.f;
        const float *rsum = st.rsum;
        if (MODE != MODE_FINAL && st.tin.rec && rsum) {
            ImageMeans<C> means;
            means.load(st.tin, n, lane, 0);
            means.finish(st.tin, n, s_mean[wave], lane);
#pragma unroll 4
            for (int k = 0; k < CP; ++k) { // (little unrolling: registers are scarce here)
                const int c = part * CP + k;
                d = fmaf(rsum[c * C + o], s_mean[wave][c], d);
            }
#pragma unroll
            for (int sh = OPW; sh < 64; sh <<= 1) d += __shfl_xor(d, sh);
        }
        if (part == 0) s_init[n & 3][o] = (MODE != MODE_FINAL || bias ? bias[slice * C + o] : 0.f) + d;
    };
    f32x16 acc[RW];
    const int sample_phase = sampled_strip(g.strips); // strips 3, 11, 19, .. are sampled (the last one of a short tile)
    // bias, ReLU, bf16, stores and statistics of strip i (accumulated by this wavefront)
    auto epilogue = [&](const Geo &q) {
        const int lane = pin_in_loop(tid & 63);
        const int px = lane & 31, half = lane >> 5;
        const int strip = q.strip, n = q.n, x0 = q.colblk * kTileW;
        const int y0 = strip * kRows;
        const int x = x0 + xb * 32 + px;
        const int yw = y0 + rg * RW; // first output row of this wavefront
        // The sums start from zero: bias + correction of the image (s_init, 16 channels per lane) is added
        // on the way out, never in place - the accumulators stay untouched, so that no second copy of them
        // is ever alive next to the weights.
        const float *si = &s_init[n & 3][cb * 32 + half * 16];
        if (MODE == MODE_MID) {
            // the image's activations (same for the whole workgroup) + element offset of this lane's first row
            bf16_t *out_img = out + (size_t)n * g.h * g.w * C;
            const uint32_t dbase = dither16(x, yw);
            const uint32_t e0 = (uint32_t)((yw * g.w + x) * C + cb * 32 + half * 16);
            const bool full = y0 + kRows <= g.h && x0 + kTileW <= g.w; // same for the whole workgroup
#pragma unroll
            for (int hq = 0; hq < 2; ++hq) { // 8 channels = one 16-byte store per row
                const f32x4 b0 = *(const f32x4 *)(si + 8 * hq), b1 = *(const f32x4 *)(si + 8 * hq + 4);
#pragma unroll
                for (int r = 0; r < RW; ++r) {
                    const uint32_t dth = dbase ^ ((uint32_t)r << 14); // the strip's rows: quarter steps apart
                    u32x4 pk;
                    pk[0] = pack_bf16_relu(acc[r][8 * hq + 0] + b0[0], acc[r][8 * hq + 1] + b0[1], dth, true);
                    pk[1] = pack_bf16_relu(acc[r][8 * hq + 2] + b0[2], acc[r][8 * hq + 3] + b0[3], dth, true);
                    pk[2] = pack_bf16_relu(acc[r][8 * hq + 4] + b1[0], acc[r][8 * hq + 5] + b1[1], dth, true);
                    pk[3] = pack_bf16_relu(acc[r][8 * hq + 6] + b1[2], acc[r][8 * hq + 7] + b1[3], dth, true);
                    bf16_t *dst = out_img + (e0 + (uint32_t)(r * g.w * C) + 8 * hq);
                    if (full) *(u32x4 *)dst = pk;
                    else if (yw + r < g.h && x < g.w) *(u32x4 *)dst = pk;
                    __builtin_amdgcn_sched_barrier(0); // one store at a time keeps the temporaries few
                }
            }
        }
        const int piece = rg * 2 + xb; // which of the strip's lines is this wavefront's: row group, pixel block
        if (MODE == MODE_FINAL) {
            float t[16];
            column_sums<RW>(t, acc, si, st.low, x < g.w, yw, g.h);
            const float sum = reduce16_over_half(t, px); // one channel per lane
            const int line = (q.colblk * g.strips + strip) * (2 * RG) + piece;
            float *rec = st.tout + (((int64_t)n * st.out_recs + line) * gridDim.y + slice) * C;
            if ((px & 1) == 0) rec[cb * 32 + half * 16 + reduce16_index(px)] = sum;
        } else if (st.tout) {
            float *lines = st.tout + (int64_t)n * st.out_recs * C + cb * 32 + half * 16;
            if (MODE == MODE_LAST) { // (the places are those of conv_mid_last_sums())
                LinePlaces at;
                at.first_col = tpi * 2 * RG;
                at.last_col = at.first_col + g.strips * RG;
                at.rows = at.last_col + g.strips * RG;
                at.last_rows = at.rows + 2 * g.colblks;
                at.corners = at.last_rows + 2 * g.colblks;
                at.whole = (q.colblk * g.strips + strip) * (2 * RG) + piece;
                at.col = strip * RG + rg;
                at.row = q.colblk * 2 + xb;
                last_lines<C, RW>(acc, si, lines, at, x, x0 + xb * 32, yw, g.h, g.w, px);
            } else if ((strip & 7) == sample_phase) {
                const int line = ((strip >> 3) * g.colblks + q.colblk) * (2 * RG) + piece;
                strip_statistics<RW>(acc, si, lines + line * C, x, yw, g.h, g.w, px);
            }
        }
    };

    // ---- prologue: corrections of the first image(s), strips 0 and 1 on their way.  Group 1 multiplies a phase later: its
    // weights come in while group 0 is at work.
    bf16x8 Wr[9][K::KC];
    {
        const int n = grp == 0 ? gc.n : g1.n;
        const bool mine = grp == 0 || (ns > 1 && g1.n != gc.n); // the same for the whole wavefront
        const float *bias_s = MODE != MODE_FINAL ? bias : (bias ? bias + slice * C : nullptr);
        const float *rsum = MODE != MODE_FINAL ? st.rsum : nullptr;
        FirstInit<C> init;
        if (mine) init.start(st.tin, rsum, bias_s, n, w4, lane);
        if (grp == 0) {
            load_weight_frags<C>(Wr, wfrag, slice * K::NCB + cb, lane);
        } else {
            issue(gc);
            if (ns > 1) issue(g1);
        }
        if (mine) init.finish(st.tin, rsum, n, w4, lane, s_mean[wave], s_init[n & 3]);
    }
    int issued_upto = min(1, ns - 1);
    __builtin_amdgcn_s_waitcnt(kWaitVm0); // group 0: weights; group 1: strips 0 and 1
    lds_barrier();
    if (grp == 1 && ns > 1) {
        load_weight_frags<C>(Wr, wfrag, slice * K::NCB + cb, lane);
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
    }

    for (int p = 0; p <= ns; ++p) {
        const bool mma_phase = (p & 1) == grp;
        // Loads: the group that is not multiplying issues strips p + 1 (only if it did not fit earlier) and
        // p + 2, as far as the ring has room (strip p is being read: everything from wstart(p) on is
        // live; strip p + 1 always fits).  Every wavefront keeps the count.  Before the epilogue: behind its stores the
        // loads would wait for those to be taken by the memory pipeline.
        const bool load1 = issued_upto == p && p + 1 < ns;
        if (load1) issued_upto = p + 1;
        const bool load2 = issued_upto == p + 1 && p + 2 < ns && g2.base + rows_loaded(g2) - wstart(gc) <= NSLOT;
        if (load2) issued_upto = p + 2;
        // the end of a phase: what this group issued a phase ago (or, strip p + 1, just now) has landed
        auto end_of_phase = [&](bool wait) {
            if (wait) __builtin_amdgcn_s_waitcnt(kWaitVm0);
            lds_barrier();
        };
        if (mma_phase) {
            if (p < ns) {
                lrow_t rowp[RW + 2];
                const int start = wstart(gc) + rg * RW;
#pragma unroll
                for (int r = 0; r < RW + 2; ++r) rowp[r] = lbase + (uint32_t)((start + r) & (NSLOT - 1)) * K::ROWB;
                __builtin_amdgcn_s_setprio(3); // the matrix stream goes first whenever both wavefronts of a SIMD are ready
                strip_mma<C, RW>(rowp, Wr, acc, kZeroAcc, [&]() { end_of_phase(true); });
                __builtin_amdgcn_s_setprio(0);
            } else {
                end_of_phase(true);
            }
        } else {
            if (load1) issue(g1);
            if (load2) issue(g2);
            if (p >= 1) epilogue(gp);
            if (p + 2 < ns && g2.n != g1.n) prepare_init(g2.n);
            end_of_phase(load1);
        }
        gp = gc;
        gc = g1;
        g1 = g2;
        advance(g2);
    }
}

// ------------------------------------------------------------------------------------------------
// Final convolution of 32-channel networks, 64 output channels per grid.y slice, summed over the pixels: the lines of
// conv_mid_kernel<64, MODE_FINAL>.  Half the matrix instructions of a 64-channel strip are too few for that kernel's phases,
// of which each end costs the same (51 % of the matrix pipes' rate): here two workgroups of four wavefronts share a compute
// unit, each with weights, accumulators and two strips' rows of its own, and fill each other's gaps.  A workgroup asks for
// the next strip's rows before it multiplies this one's.  The line of a strip is written behind the next strip's loads, so
// that the wait for them never waits for a store just issued.  Measured against conv_mid_kernel in that place (two blocks and
// this, us a call): 2404 tiles of 40 x 5, 107 bits 571 -> 485; 512 of 128 x 128, 60 bits 682 -> 663; 700 of 64 x 64, 120 bits 344 ->
// 331; 20 of 64 x 64, 128 bits 34.9 -> 31.5.  Loading only the rows that the strip above does not share: no gain (504, 651).
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256, 2) void conv_final32_kernel(const uint8_t *__restrict__ in, ConvGeom g,
                                                              const bf16_t *__restrict__ wfrag, const float *__restrict__ bias,
                                                              StatArgs st)
{
    constexpr int C = 32, RW = kRows, WIN = kRows + 2, kBuf = 8; // a strip's buffer has kBuf row slots, WIN of them in use
    typedef MidCfg<C> K;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[(kBuf + WIN) * K::ROWB];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int px = lane & 31, half = lane >> 5;
    const int cb = wave & 1, xb = wave >> 1, slice = blockIdx.y;
    bf16x8 Wr[9][K::KC];
    load_weight_frags<C>(Wr, wfrag, slice * 2 + cb, lane);
    float bias16[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) bias16[v] = bias ? bias[slice * 64 + cb * 32 + half * 16 + v] : 0.f;
    const int tpi = g.strips * g.colblks, total = g.n_img * tpi;
    const int t_begin = xcd_virtual_block(blockIdx.x, gridDim.x) * st.per;
    const int ns = min(total, t_begin + st.per) - t_begin; // strips of this workgroup's run
    if (ns <= 0) return;
    const lrow_t lbase = lds_address(lds) + (xb * 32 + px) * K::PS + half * 16;
    const size_t img_bytes = (size_t)g.h * g.w * C * 2;
    const uint32_t row_bytes = (uint32_t)(g.w * C * 2);
    const RowLoader<C> loader(wave, lane);
    struct Geo {
        int strip, colblk, n;
    };
    auto advance = [&](Geo &q) {
        if (++q.strip == g.strips) {
            q.strip = 0;
            if (++q.colblk == g.colblks) {
                q.colblk = 0;
                ++q.n;
            }
        }
    };
    auto issue = [&](const Geo &q, int buf) {
        loader.strip(lds + buf * kBuf * K::ROWB, kBuf, in + (size_t)q.n * img_bytes, (uint32_t)img_bytes, g.h, row_bytes, q.strip * kRows, q.colblk * kTileW, wave);
    };
    Geo gc{t_begin % g.strips, (t_begin / g.strips) % g.colblks, t_begin / tpi}, g1 = gc;
    advance(g1);
    float *rec = nullptr; // where the sums of the strip before go
    float sum = 0.f;
    auto write_line = [&]() {
        if ((px & 1) == 0) rec[cb * 32 + half * 16 + reduce16_index(px)] = sum;
    };
    issue(gc, 0);
    for (int i = 0; i < ns; ++i) {
        __builtin_amdgcn_s_waitcnt(kWaitVm0); // this strip's rows, asked for a strip ago
        lds_barrier();                        // .. by all wavefronts, which also have read the other buffer
        if (i + 1 < ns) issue(g1, (i + 1) & 1);
        if (i > 0) write_line();
        lrow_t rowp[RW + 2];
#pragma unroll
        for (int r = 0; r < RW + 2; ++r) rowp[r] = lbase + (uint32_t)((i & 1) * kBuf + r) * K::ROWB;
        f32x16 acc[RW];
        __builtin_amdgcn_s_setprio(3);
        strip_mma<C, RW>(rowp, Wr, acc, kZeroAcc, []() {});
        __builtin_amdgcn_s_setprio(0);
        float t[16];
        auto row_sums = [&](auto full) { // as column_sums(), without a test per value where the strip has all of its rows
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                t[v] = fmaxf(acc[0][v] + bias16[v], st.low);
#pragma unroll
                for (int r = 1; r < RW; ++r)
                    if (decltype(full)::value || gc.strip * kRows + r < g.h) t[v] += fmaxf(acc[r][v] + bias16[v], st.low);
            }
        };
        if (gc.strip * kRows + RW <= g.h) row_sums(std::true_type{});
        else row_sums(std::false_type{});
        const int x0 = gc.colblk * kTileW + xb * 32;
        if (x0 + 32 > g.w) { // (the same for the whole wavefront)
#pragma unroll
            for (int v = 0; v < 16; ++v) t[v] = x0 + px < g.w ? t[v] : 0.f;
        }
        sum = reduce16_over_half(t, px); // one channel per lane
        const int line = (gc.colblk * g.strips + gc.strip) * 2 + xb;
        rec = st.tout + (((int64_t)gc.n * st.out_recs + line) * gridDim.y + slice) * 64;
        gc = g1;
        advance(g1);
    }
    write_line();
}

// ------------------------------------------------------------------------------------------------
// Two consecutive C -> C blocks in one kernel (C = 64).
//
// conv_mid is bound by activation traffic as much as by the matrix cores (288 FLOP per byte against a
// machine balance of ~310).  Here the activations between the two blocks never leave the CU: a
// workgroup walks down its images, group A (wavefronts 0-3, weights of the first block) turns input rows
// into rows of the intermediate activation map, which it writes as bf16 into a second LDS ring, and
// group B (wavefronts 4-7, weights of the second block) turns those into output rows.  Global traffic
// per FLOP halves; both wavefronts of a SIMD carry matrix work, so each fills the other's gaps.
//
// Rows are processed two at a time (the two rings of 8 rows of 66 pixels x 144 bytes fill the LDS).  Step s
// of an image of h rows, S = ceil(h/2):
//   A   : s < S: intermediate rows 2s, 2s+1 from input rows 2s-1 .. 2s+2; behind its matrix instructions it
//         waits for the loads it issued a step ago and issues the direct-to-LDS loads of input rows 2s+5, 2s+6
//         (needed in step s+2); then ReLU, bf16 -> intermediate ring (zeros outside the
//         tile);  s == S: rows 2S, 2S+1 = zero padding
//   B   : first the epilogue of the rows it accumulated in step s-1 (stores behind which its matrix
//         instructions then run), then output rows 2j, 2j+1, j = s-2, from intermediate rows 2j-1 .. 2j+2
//   end : one workgroup barrier
// The sums start from bias (+ correction), which either group keeps in 16 registers: a third of an epilogue's vector
// instructions and all of its LDS reads were the bias.  The groups have loops of their own: 225 .. 241 registers instead of the
// 239 .. 256 of one loop for both, which is where the bias found room, and scalar ones (up to 24) are no longer spilled, but for six
// where a pair is first, last, wide and dealt in runs.  A step of a middle pair of 1024 tiles of 64 x 64 takes 5190 cycles
// (SQ_BUSY_CU_CYCLES), 4608 of them matrix instructions; what bounds a launch of bulk size is the clock that its power
// leaves (1.6 GHz of 2.4).
// (All loads are group A's: the vector-memory instructions of a compute unit issue in order, and loads issued
// by group B at the end of a step would sit in front of its own stores at the start of the next.)
// Row y of either map lives in ring slot (y + 2) mod 8.
// A workgroup's images follow each other without a gap: see the main loop (virtual rows).
// The second block's weights are rounded so that the rounding residuals of the nine taps of every
// (output, input) channel pair cancel (error feedback over the taps): its input never exists as a whole
// image, so there are no channel means to correct its bias with.
//
// WIDE (tiles wider than 64 columns): the rings stay 66 pixels wide and a workgroup walks through its image
// one column block of 64 after the other, left to right, each block top to bottom ("unit" = (image, column
// block); the units of a workgroup form one stream of row pairs as the images do above).  In block b group A
// computes intermediate columns [64 b, 64 b + 64) from input columns [64 b - 1, 64 b + 65), and group B computes
// output columns [64 b - 1, 64 b + 63): one column to the left, so that everything B needs lies at or left of
// A's newest column.  The two intermediate columns left of A's (64 b - 2, 64 b - 1) were computed in block
// b - 1: A writes its last two columns of every row to a small buffer in global memory (the "seam", 256 bytes a
// row, per workgroup, two of them used alternately), from which they come back into ring pixels 0 and 1 a whole
// column block later (for b = 0 those pixels are zero: the padding).  Nothing is computed twice and no
// matrix tile is partly empty.  What is left over is the tile's last column when the width is a multiple of 64:
// the intermediate columns w-2, w-1 of every row go to a per-image seam buffer and conv_seam_kernel, a small
// launch behind this one, computes output column w-1 from them.
// ------------------------------------------------------------------------------------------------
constexpr int kPairRing = 8;
constexpr int kSeamRowBytes = 2 * 64 * 2; // two pixels of 64 bf16 channels: what one row hands over

struct PairArgs {
    MeanIn tin;         // channel sums of the input (rec null: no correction)
    const float *rsum;  // [c_in][c_out] residual-weight sums of the first block (fp32)
    float *tout;        // channel sums of the output, or nullptr: [n_img][out_recs][C]
    int out_recs;       // records (LASTB: lines) per image
    int per;            // pieces (of QUANT row pairs) per workgroup
    int sum_rows;       // LASTB: LastSums::rows, the other places follow from the tile's size
    uint8_t *seam;      // WIDE: [workgroup][2][2 S rows][2 pixels][C] bf16, columns handed to the next column block
    uint8_t *seam_last; // WIDE, width a multiple of 64: [image][2 S rows][2 pixels][C], intermediate columns w-2, w-1
};
// Row pairs behind one line of the last block's sums, and the granularity at which its images are cut between
// workgroups: 1 would store four times as much (35 KB instead of 10 for a 64 x 64 tile), 8 would make the last launch of
// a single tile twice as long.  Launches of so few tiles that kChunk row pairs are more than a compute unit's share leave a line
// per row pair instead, which the head adds up in the order in which the kernel would have: the sums are the same bit for bit
// (the last pair of one tile of 64 x 64: 18.7 -> 11.8 us).
constexpr int kChunk = 4;

// FIRST: the first of the two blocks is the network's first block (3 -> C on the raw u8 tile: crop and
//        normalisation fused, weights as bf16 high part + residual, see conv_first_kernel) instead of a
//        C -> C block; `src` replaces in, wfragA holds that block's fragments.
// LASTB: the second block is the network's last block: no activations are written, but lines of its channel
//        sums (see last_block_statistics).
// WIDE : tiles of more than one column block (see above); the other instantiations keep the straight-line code
//        of the one-block case.
// QUANT: row pairs per piece dealt to workgroups, with LASTB the row pairs behind a line: kChunk or 1 there, 1 otherwise.
// PART : workgroups take runs of row pairs that begin and end inside images; otherwise every workgroup takes whole
//        images (st.per is a multiple of an image's pieces), which costs fewer scalar instructions per step.
// in: the input activations of the launch.
template <int C, bool FIRST, bool LASTB, bool WIDE, bool PART, int QUANT>
__global__ __launch_bounds__(512, 1) void conv_pair_kernel(const uint8_t *__restrict__ in, TileSrc src,
                                                           ConvGeom g, const bf16_t *__restrict__ wfragA,
                                                           const bf16_t *__restrict__ wfragB,
                                                           const float *__restrict__ biasA,
                                                           const float *__restrict__ biasB, PairArgs st,
                                                           bf16_t *__restrict__ out)
{
    typedef MidCfg<C> K;
    static_assert(K::NCB == 2, "the pair kernel is written for 64 channels");
    constexpr int RW = 2;
    constexpr int ROWB = kHaloW * K::PS;          // staged rows are packed: 66 pixels x 144 bytes
    constexpr int SLOTS = ROWB / 16;              // 16-byte slots per row
    __shared__ __attribute__((aligned(1024))) uint8_t ring_in[FIRST ? 1024 : kPairRing * ROWB];
    __shared__ __attribute__((aligned(16))) uint8_t ring_mid[kPairRing * ROWB];
    __shared__ __attribute__((aligned(16))) uint16_t s_pix[FIRST ? kPairRing : 1][kHaloW][4]; // raw pixels as bf16; channel 3 = 1 inside the tile
    __shared__ __attribute__((aligned(16))) float s_initA[C]; // first block: bias (+ rounding-residual correction of the image)
    __shared__ __attribute__((aligned(16))) float s_biasB[C];
    __shared__ __attribute__((aligned(16))) float s_zero[LASTB ? 4 : 16]; // (the sums that the statistics read hold their bias)
    __shared__ __attribute__((aligned(16))) float s_stat[LASTB ? 4 : 1][2][32]; // LASTB: sums of the first / last column
    __shared__ __attribute__((aligned(16))) float s_mean[4][C];
    // FIRST: group A has little matrix work, group B hands it the fp32 accumulators of the first of its two rows for the epilogue
    // ([buffer = row pair parity][wavefront][channel quad][lane] x 4 floats): either group then has about 3700 cycles of a
    // step's 4300 (both rows handed over: group A 4300, group B 3200 of 4400).
    constexpr bool kHandOver = FIRST && !LASTB;
    __shared__ __attribute__((aligned(16))) float s_accx[kHandOver ? 2 * 4 * 4 * 256 : 4];
    constexpr int kSkew = WIDE ? 1 : 0;         // group B's columns lie this far left of group A's

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave >> 2, w4 = wave & 3;
    const int px = lane & 31, half = lane >> 5;
    const int cb = w4 & 1, xb = w4 >> 1;

    const int vb = xcd_virtual_block(blockIdx.x, gridDim.x);
    const int S = (g.h + 1) / 2;
    const int J = WIDE ? g.colblks : 1;           // column blocks of a tile
    // The launch's row pairs, image after image, are cut into runs of st.per pieces, one run per workgroup: row pairs ja
    // of image n_begin up to (not including) jb of image n_begin + n_cnt - 1.  Whole images per workgroup left 35 % of
    // the compute units idle at 333 images (two each for 166 of them, none for the others) and all but one at 1.
    const int ppi = (S + QUANT - 1) / QUANT;      // pieces per image
    const int q0 = vb * st.per, q1 = min(g.n_img * ppi, q0 + st.per);
    if (q0 >= q1) return;
    const int n_begin = q0 / ppi, ja = PART ? (q0 - n_begin * ppi) * QUANT : 0;
    const int n_cnt = (q1 - 1) / ppi - n_begin + 1, jb = PART ? min(S, (q1 - (n_begin + n_cnt - 1) * ppi) * QUANT) : S;
    // C -> C weights (group B; group A unless FIRST).  Group A with FIRST keeps the first block's weights in
    // the same registers: Wr[p][k] = high part (p = 0) / residual (p = 1) of 16-wide k chunk k.
    bf16x8 Wr[9][K::KC];
    auto load_weights = [&]() {
        if (FIRST && grp == 0) {
#pragma unroll
            for (int f = 0; f < kFirstFrags; ++f) Wr[f / 3][f % 3] = ((const bf16x8 *)wfragA)[(cb * kFirstFrags + f) * 64 + lane];
        } else {
            load_weight_frags<C>(Wr, grp == 0 ? wfragA : wfragB, cb, lane);
        }
    };
    FirstInit<C> init; // (the correction's loads go first, then the input rows', then the weights': see below)
    if (!FIRST && grp == 0) init.start(st.tin, st.rsum, biasA, n_begin, w4, lane);
    const size_t img_bytes = (size_t)g.h * g.w * C * 2;
    const uint32_t row_bytes = (uint32_t)(g.w * C * 2);
    const lrow_t in_base = lds_address(ring_in) + (xb * 32 + px) * K::PS + half * 16;
    const lrow_t mid_base = lds_address(ring_mid) + (xb * 32 + px) * K::PS + half * 16;
    const int sample_phase = sampled_strip(g.strips);
    auto slot_of = [](int y) { return (y + 2) & (kPairRing - 1); };

    // Loads of input row y of image n into its ring slot by the four wavefronts of one group.
    const RowLoader<C> loader(w4, lane);
    auto issue_rows = [&](int n, int blk, int y, int vrow, int rows) { // vrow: the row's place in the stream of units (see the main loop)
        const auto cols = loader.at(blk * kTileW, row_bytes);
        for (int r = 0; r < rows; ++r)
            loader.row(cols, in + (size_t)n * img_bytes, (uint32_t)img_bytes, y + r, g.h, row_bytes, ring_in + slot_of(vrow + r) * ROWB, w4);
    };
    // s_initA[o] = biasA[o] + sum_c rsum[c][o] * mean_n[c], by the four wavefronts of group A
    auto prepare_init = [&](int n) {
        constexpr int OPW = C / 4, PARTS = 64 / OPW, CP = C / PARTS;
        const int ln = pin_in_loop(tid & 63);
        const int o = w4 * OPW + ln % OPW, part = ln / OPW;
        float d = 0.f;
        if (st.tin.rec && st.rsum) {
            ImageMeans<C> means;
            means.load(st.tin, n, ln, 0);
            means.finish(st.tin, n, s_mean[w4], ln);
#pragma unroll 4
            for (int k = 0; k < CP; ++k) {
                const int c = part * CP + k;
                d = fmaf(st.rsum[c * C + o], s_mean[w4][c], d);
            }
#pragma unroll
            for (int sh = OPW; sh < 64; sh <<= 1) d += __shfl_xor(d, sh);
        }
        if (part == 0) s_initA[o] = biasA[o] + d;
    };
    // FIRST: rows of the raw tile -> bf16 pixels in s_pix, by the 256 threads of group A: thread 66 c + col fetches channel c of
    // staged column col, one row per load.  What stays the same from row to row is found once per unit (pixel_unit): the
    // address in the tile's first row, and whether the column lies inside the tile.
    // The load is unconditional (coordinates clamped into the tile, the value dropped later when it lies
    // outside) and fetches the aligned dword that holds the byte (it never leaves the byte's page): a load under
    // a lane mask, or a byte load with its widening, would be waited for on the spot, and a step would then
    // contain two round trips to memory instead of hiding them behind its matrix work.
    constexpr int kRowElems = 3 * kHaloW;
    const int plane = src.H * src.W;
    const int pix_c = min(tid, kRowElems - 1) / kHaloW, pix_col = min(tid, kRowElems - 1) - pix_c * kHaloW;
    const uint8_t *pix_at = nullptr; // this thread's byte in the unit's first row
    bool pix_inside = false;
    auto pixel_unit = [&](const uint8_t *tile0, int x0) {
        const int tx = x0 + pix_col - 1;
        pix_inside = (uint32_t)tx < (uint32_t)g.w;
        pix_at = tile0 + ((int64_t)pix_c * plane + clampi(tx, 0, g.w - 1));
    };
    auto pixel_fetch = [&](int y, uint32_t &shift) -> uint32_t {
        const uintptr_t p = (uintptr_t)(pix_at + (int64_t)clampi(y, 0, g.h - 1) * src.W);
        shift = (uint32_t)p * 8u; // (the shift instruction looks at the low five bits)
        typedef const uint32_t __attribute__((address_space(1))) *global_word_t; // a global load, not a flat one
        return *(global_word_t)(p & ~(uintptr_t)3);
    };
    auto pixel_store = [&](int vrow, bool inside, uint32_t word, uint32_t shift) { // vrow: the row's place in the stream of units; inside: the pixel lies in the tile
        asm volatile("" : "+v"(word)); // the value is first looked at here, not where it was asked for
        // the byte itself, exact as bf16: the normalisation lives in the weights (see conv_first_kernel)
        const uint32_t f = __builtin_bit_cast(uint32_t, (float)((word >> (shift & 31u)) & 0xffu)) >> 16;
        uint8_t *dst = (uint8_t *)&s_pix[slot_of(vrow)][pix_col][pix_c];
        if (tid < 2 * kHaloW) *(uint16_t *)dst = (uint16_t)(inside ? f : 0u);
        else if (tid < kRowElems) *(uint32_t *)dst = inside ? f | 0x3F800000u : 0u; // the last colour and the fourth channel: 1 inside the tile
    };

    // ---- once per workgroup: biases, the halo columns of the intermediate ring, statistics
    if (LASTB && grp == 1) (&s_stat[w4][0][0])[lane] = 0.f;
    if (grp == 1) {
        if (tid - 256 < C) s_biasB[tid - 256] = biasB[tid - 256];
        if (!LASTB && tid - 256 < 16) s_zero[tid - 256] = 0.f;
    } else if (FIRST) {
        if (tid < C) s_initA[tid] = biasA[tid];
    }
    if (!WIDE) // (WIDE: pixels 0 and 1 are rewritten in every step, 2 .. 65 by group A)
    for (int i = tid; i < kPairRing * 2 * (K::PS / 16); i += 512) { // columns -1 and w.. stay zero for good
        const int row = i / (2 * (K::PS / 16)), rem = i - row * 2 * (K::PS / 16);
        const int side = rem / (K::PS / 16), sl = rem - side * (K::PS / 16);
        *(u32x4 *)(ring_mid + row * ROWB + (side ? (kHaloW - 1) : 0) * K::PS + sl * 16) = (u32x4){0u, 0u, 0u, 0u};
    }

    // The units (image, column block) of a workgroup form one stream of positions, one per step.  A unit's output row
    // pairs are lo .. hi-1 (all S of them but for the workgroup's first and last image); its positions s are
    //   an opening position: -1, or lo - 2 if the unit begins inside the image.  Nothing is computed (zeros go to
    //       the intermediate ring: the padding below the unit before and above this one), only loads are issued;
    //   lo - 1, if the unit begins inside the image: the pair whose second row is the halo row above the unit;
    //   lo .. hi - 1;
    //   hi, if the unit ends inside the image: the pair whose first row is the halo row below.
    // (The halo pairs are computed by both neighbours, to the same bits.)  The workgroup's first unit skips its opening
    // position; one more opening position follows the last unit.  At position number sg of the stream group A
    // computes intermediate rows 2s, 2s + 1 of the unit, which live in the rings as virtual rows 2 sg, 2 sg + 1;
    // group B is at position sg - 2, the epilogue of B's rows at sg - 3, the loads at sg + 2 (pixels: sg + 1):
    // nothing drains between units.
    struct Pos {
        int i, b, s; // image within the workgroup (n_cnt: none), column block within the image, position in the unit
    };
    auto lo = [ja](int i) { return PART && i == 0 ? ja : 0; };
    auto hi = [n_cnt, jb, S](int i) { return PART && i == n_cnt - 1 ? jb : S; };
    auto opening = [ja](int i) { return PART && i == 0 && ja > 0 ? ja - 2 : -1; };
    auto closing = [hi, S](int i) { return min(hi(i), S - 1); };
    auto computes = [lo](const Pos &p) { return p.s >= max(lo(p.i) - 1, 0); }; // not an opening position
    auto owns = [lo, hi](const Pos &p) { return p.s >= lo(p.i) && (!PART || p.s < hi(p.i)); };
    auto advance = [J, closing, opening](Pos &p) {
        if (__builtin_expect(++p.s > closing(p.i), 0)) { // once per unit: kept out of the way of the other steps
            if (++p.b == J) {
                p.b = 0;
                ++p.i;
            }
            p.s = opening(p.i);
        }
    };
    int n_pos = n_cnt > 2 ? (n_cnt - 2) * J * (S + 1) : 0; // positions, opening position behind the last unit included
    n_pos += J * (closing(0) - opening(0) + 1);
    if (n_cnt > 1) n_pos += J * (closing(n_cnt - 1) + 2);
    // The two groups have loops of their own, and each keeps the positions it needs, no others: the loops are short of scalar
    // registers (with six positions in every wavefront of one loop for both, up to 24 of them were spilled).
    Pos pw{0, 0, max(ja - 1, 0)}; // group A: position sg; group B: position sg - 2
    Pos p1 = pw;                  // FIRST: group A's pixel loads, position sg + 1; group B's seam loads, position sg
    if (!FIRST || grp == 0) advance(p1);
    Pos pe = pw;                  // epilogue of B's rows, position sg - 3 (group B), sg - 4 (kHandOver: group A); otherwise group A's loads, sg + 2
    if (!FIRST && grp == 0) {
        pe = p1;
        advance(pe);
    }
    auto tile_origin = [&](int n) {
        int oy = 0, ox = 0;
        if (src.off) {
            oy = clampi(src.off[2 * n], 0, src.H - g.h);
            ox = clampi(src.off[2 * n + 1], 0, src.W - g.w);
        }
        return src.img + (int64_t)n * 3 * plane + (int64_t)oy * src.W + ox;
    };

    // FIRST, group A: the unit of position p begins
    const uint8_t *tile0 = nullptr;
    auto pixel_first_unit = [&](const Pos &p) {
        if (p.b == 0) tile0 = tile_origin(n_begin + p.i); // the next image
        pixel_unit(tile0, p.b * kTileW);
    };

    // ---- before the first step: correction of the first image, its input rows -1 .. 4 (FIRST: -1 .. 2),
    //      intermediate row -1 = zero
    if (FIRST) {
        if (grp == 0) load_weights();
        tile0 = tile_origin(n_begin);
        if (grp == 0) {
            uint32_t word[4], shift[4];
            pixel_unit(tile0, 0);
#pragma unroll
            for (int k = 0; k < 4; ++k) word[k] = pixel_fetch(2 * pw.s - 1 + k, shift[k]);
#pragma unroll
            for (int k = 0; k < 4; ++k) pixel_store(-1 + k, pix_inside && (uint32_t)(2 * pw.s - 1 + k) < (uint32_t)g.h, word[k], shift[k]);
            if (p1.i < n_cnt && p1.s == opening(p1.i)) pixel_first_unit(p1);
        }
    } else {
#pragma unroll 1
        for (int v = -1 + grp; v <= 4; v += 2) { // first, so that they travel while the correction is computed
            if (v <= 2) issue_rows(n_begin, 0, 2 * pw.s + v, v, 1);
            else if (p1.i < n_cnt) issue_rows(n_begin + p1.i, p1.b, 2 * p1.s + v - 2, v, 1);
        }
    }
    if (!FIRST && grp == 0) load_weights(); // behind the loads that take another step
    if (!FIRST && grp == 0) init.finish(st.tin, st.rsum, n_begin, w4, lane, s_mean[w4], s_initA);
    if (grp == 1)
        for (int i = tid - 256; i < SLOTS; i += 256) *(u32x4 *)(ring_mid + slot_of(-1) * ROWB + i * 16) = (u32x4){0u, 0u, 0u, 0u};
    __builtin_amdgcn_s_waitcnt(kWaitVm0);
    __syncthreads();
    if (grp == 1) { // group B multiplies from step 2 on: its weights come in while group A is at work
        load_weights();
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
    }

    // LASTB: the nine border-aware channel sums of the last block's output from the two
    // rows in `a`, written as lines of C sums (LastSums).  The sum over the whole tile, the only one every pixel goes
    // into, is kept in a register per lane: the 16 channel values of a lane (both rows added) go through one butterfly
    // over the 32 pixel lanes, after which every lane holds the sum of one channel and adds it to its running total
    // (run_sum), which becomes a line at the end of a chunk.  First / last column: the one lane that holds it adds its
    // 16 values to the LDS accumulators, in the wavefronts that contain such a column only; a line per chunk.  First /
    // last row and the four corners: lines of their own, in the (two) steps that contain those rows.
    float run_sum = 0.f;
    auto last_block_statistics = [&](const f32x16 (&a)[RW], const Pos &p, int x, int x0w, int pxl, int hf) {
        const int j = p.s;
        float *stat = &s_stat[w4][0][hf * 16];
        float *lines = st.tout + (int64_t)(n_begin + p.i) * st.out_recs * C + cb * 32 + hf * 16;
        const bool colok = (uint32_t)x < (uint32_t)g.w;
        const bool allcols = x0w >= 0 && x0w + 32 <= g.w; // same for the whole wavefront
        const bool row1 = 2 * j + 1 < g.h;                // (row 2j always lies in the tile)
        const bool has_first = x0w <= 0 && x0w + 32 > 0, has_last = x0w <= g.w - 1 && g.w - 1 < x0w + 32;
        float t[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float r1 = fmaxf(a[1][v], 0.f);
            t[v] = fmaxf(a[0][v], 0.f) + (row1 ? r1 : 0.f);
        }
        if (!allcols) {
#pragma unroll
            for (int v = 0; v < 16; ++v) t[v] = colok ? t[v] : 0.f;
        }
        auto column = [&](float *dst, const float (&val)[16], bool pred) { // one lane's 16 values into 16 accumulators
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float four[4] = {val[4 * q], val[4 * q + 1], val[4 * q + 2], val[4 * q + 3]};
                lds_accumulate4(dst + 4 * q, four, pred);
            }
        };
        auto corner = [&](float *dst, const float (&val)[16], bool pred) { // the same into global memory, once
            if (pred) {
#pragma unroll
                for (int q = 0; q < 4; ++q) *(f32x4 *)(dst + 4 * q) = (f32x4){val[4 * q], val[4 * q + 1], val[4 * q + 2], val[4 * q + 3]};
            }
        };
        if (has_first) column(stat, t, x == 0);
        if (has_last) column(stat + 32, t, x == g.w - 1);
        run_sum += reduce16_over_half(t, pxl);
        if (j % QUANT == QUANT - 1 || j == S - 1) { // the chunk's lines
            const int ch = j / QUANT, blk2 = p.b * 2 + xb, chunks = ppi;
            if ((pxl & 1) == 0) lines[(ch * 2 * J + blk2) * C + reduce16_index(pxl)] = run_sum;
            run_sum = 0.f;
            if (pxl < 16) {
                if (has_first) {
                    lines[(2 * J * chunks + ch) * C + pxl] = stat[pxl];
                    stat[pxl] = 0.f;
                }
                if (has_last) {
                    lines[((2 * J + 1) * chunks + ch) * C + pxl] = stat[32 + pxl];
                    stat[32 + pxl] = 0.f;
                }
            }
        }
        const int rl = g.h - 1 - 2 * j; // the tile's last row, counted from this pair's first
        if (j == 0 || rl < RW) { // the tile's first and / or last row is one of the two
#pragma unroll 1
            for (int which = 0; which < 2; ++which) {
                if (which == 0 ? j != 0 : (rl < 0 || rl >= RW)) continue;
                const bool second = which == 1 && rl == 1;
                float rv[16];
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float av = second ? a[1][v] : a[0][v];
                    rv[v] = colok ? fmaxf(av, 0.f) : 0.f;
                }
                const float y = reduce16_over_half(rv, pxl);
                if ((pxl & 1) == 0) lines[(st.sum_rows + (which * J + p.b) * 2 + xb) * C + reduce16_index(pxl)] = y;
                if (has_first) corner(lines + (st.sum_rows + 4 * J + 2 * which) * C, rv, x == 0);
                if (has_last) corner(lines + (st.sum_rows + 4 * J + 2 * which + 1) * C, rv, x == g.w - 1);
            }
        }
    };

    // Output row 2j + r of column block blk of image n held in `a`: ReLU and bf16, then the stores.
    auto packed_row = [&](const f32x16 &a, uint32_t dither, u32x4 (&pk)[2]) {
#pragma unroll
        for (int v = 0; v < 8; ++v) pk[v / 4][v % 4] = pack_bf16_relu(a[2 * v], a[2 * v + 1], dither, true);
    };
    auto finish_pack = [&](const f32x16 &a, int r, const Pos &p, u32x4 (&pk)[2]) {
        const int ln = pin_in_loop(tid & 63);
        packed_row(a, dither16(p.b * kTileW - kSkew + xb * 32 + (ln & 31), 2 * p.s) ^ ((uint32_t)r << 15), pk); // the pair's second row: half a step apart
    };
    auto finish_store = [&](int r, const Pos &p, const u32x4 (&pk)[2]) {
        const int ln = pin_in_loop(tid & 63);
        const int x = p.b * kTileW - kSkew + xb * 32 + (ln & 31), y = 2 * p.s + r; // (x = -1 in block 0 of a wide tile)
        const uint32_t voff = (uint32_t)x < (uint32_t)g.w ? (uint32_t)((x * C + cb * 32 + (ln >> 5) * 16) * 2) : kOutside;
        uint8_t *dst = (uint8_t *)out + (size_t)(n_begin + p.i) * img_bytes; // y: the same for the whole workgroup
#pragma unroll
        for (int hq = 0; hq < 2; ++hq) store16(dst, y < g.h ? (uint32_t)img_bytes : 0, voff, y < g.h ? y * (int)row_bytes + hq * 16 : 0, pk[hq]);
    };
    // Statistics of output rows 2j, 2j+1
    auto finish_statistics = [&](const f32x16 (&a)[RW], const Pos &p) {
        const int n = n_begin + p.i, blk = p.b, j = p.s;
        const int ln = pin_in_loop(tid & 63);
        const int pxl = ln & 31, hf = ln >> 5;
        const int x_lo = blk * kTileW - kSkew;
        const int x = x_lo + xb * 32 + pxl;
        if (!st.tout) return;
        if (LASTB) last_block_statistics(a, p, x, x_lo + xb * 32, pxl, hf);
        else if (((j >> 1) & 7) == sample_phase) { // (the rows conv_mid would sample)
            const int ri = (((j >> 4) * 2 + (j & 1)) * J + blk) * 2 + xb; // sampled row pair, column block, pixel block
            strip_statistics<RW>(a, s_zero, st.tout + ((int64_t)n * st.out_recs + ri) * C + cb * 32 + hf * 16, x, 2 * j, g.h, g.w, pxl);
        }
    };

    // WIDE, group A: the last two columns (62, 63) of the intermediate rows written in this step, read back from
    // the ring (the wavefront's own writes) and stored to the seam rows at `rows` (null: nothing to hand over).
    // Issued behind the step's wait for global memory, so that the wait never has to sit out these stores.
    auto seam_flush = [&](uint8_t *rows, int sg) {
        if (!rows || xb != 1) return;
        const int ln = pin_in_loop(tid & 63);
        const int pxl = ln & 31, hf = ln >> 5;
        if (pxl >= 30) {
#pragma unroll
            for (int r = 0; r < RW; ++r)
#pragma unroll
                for (int hq = 0; hq < 2; ++hq) {
                    const u32x4 v = *(const u32x4 *)(ring_mid + slot_of(2 * sg + r) * ROWB + (1 + kSkew + 32 + pxl) * K::PS + (cb * 32 + hf * 16 + 8 * hq) * 2);
                    *(u32x4 *)(rows + r * kSeamRowBytes + (pxl - 30) * (C * 2) + (cb * 32 + hf * 16 + 8 * hq) * 2) = v;
                }
        }
    };
    // WIDE: ring pixels 0 and 1 of the intermediate rows group A writes in this step: the two columns left of its
    // block, from the seam of the block before (zeros in block 0 and at opening positions); 2 x 9 slots per row,
    // straight into LDS.  One wavefront issues them and waits for them before the step's barrier; the step in which their
    // slots were last read is the one before.
    const size_t seam_half = (size_t)(2 * S) * kSeamRowBytes; // one of a workgroup's two seam buffers
    auto seam_loads = [&](int sg, const Pos &p) {
        const int ln = pin_in_loop(tid & 63);
        const bool have = p.b > 0 && computes(p);
        const uint8_t *sp = st.seam + ((size_t)blockIdx.x * 2 + ((p.b & 1) ^ 1)) * seam_half + (size_t)(2 * (have ? p.s : 0)) * kSeamRowBytes;
        const int spx = ln / K::SPP, sslot = ln - spx * K::SPP;
        const uint32_t voff = sslot < C / 8 ? (uint32_t)(spx * (C * 2) + sslot * 16) : kOutside;
        if (ln < 2 * K::SPP) {
#pragma unroll
            for (int r = 0; r < RW; ++r)
                load_lds16(sp, have ? RW * kSeamRowBytes : 0, voff, r * kSeamRowBytes, ring_mid + slot_of(2 * sg + r) * ROWB);
        }
    };
    // !FIRST, group A, in the middle of its step (between its matrix work and its epilogue): what the wavefront
    // issued a step ago - the two input rows of the step after this one, the seam columns it handed over - is waited for, then
    // this step's seam columns and the two rows needed two steps from now are put on their way: rows 2s+1, 2s+2 of the position
    // of step sg + 2.  Their ring slots were last read in the step before this one.  In the middle of the step, not at its end:
    // the vector-memory instructions of a compute unit queue up behind each other, and group B's stores at the start of the
    // next step - the critical path - would otherwise wait behind these twenty loads.
    auto input_loads = [&](int sg) {
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
        if (WIDE && w4 == 0) seam_loads(sg, pw);
        if (pe.i < n_cnt) issue_rows(n_begin + pe.i, pe.b, 2 * pe.s + 1, 2 * sg + 5, 2);
    };
    constexpr int kFirstWaveLoads = RW * ((K::PIECES + 3) / 4); // of those, the first wavefront's for the rows
    f32x16 acc[RW];
    const int n_steps = n_pos + (kHandOver ? 3 : 2);

    if (grp == 0) {
        // ---- group A
        // !FIRST: where its rows of the step lie and whether it multiplies them.  Found before the barrier in front of the
        // step, where this group has time to spare: between the barrier and its first matrix instruction the matrix pipes
        // would stand idle for it (a step of a middle pair 5720 -> 5360 cycles; 4096 tiles of 64 x 64 6540 -> 6460 us: the clock
        // gives way as the pipes fill up).
        lrow_t rowp[RW + 2];
        bool multiplies = false;
        auto prepare_step = [&](int sg) {
#pragma unroll
            for (int r = 0; r < RW + 2; ++r) {
                rowp[r] = in_base + (uint32_t)slot_of(2 * sg - 1 + r) * ROWB;
                asm volatile("" : "+v"(rowp[r])); // here, not where it is used
            }
            multiplies = pw.i < n_cnt && computes(pw);
        };
        if (!FIRST) prepare_step(0);
        // Sums start from bias (+ correction of the image), this lane's 16 channels: kept in registers, read anew behind an opening
        // position that prepared those of the next image
        f32x16 init16 = load16(&s_initA[cb * 32 + half * 16]);
        bool new_init = false;
#pragma unroll 1
        for (int sg = 0; sg < n_steps; ++sg) {
            const int ln = pin_in_loop(tid & 63);
            const int pxl = ln & 31, hf = ln >> 5;
            const int xl = xb * 32 + pxl;          // this lane's column within the block
            // FIRST: the raw pixels of virtual rows 2sg+3, 2sg+4 (window of step sg+1) start their way into registers
            // (behind the last unit: pixels of its tile that nobody looks at, as a load under a condition would be waited for, and
            // with it the stores of the step before, where the next step sets its register)
            const int ty = 2 * p1.s + 1; // image row of the first
            uint32_t pv[2], psh[2];
            if (FIRST) {
#pragma unroll
                for (int k = 0; k < 2; ++k) pv[k] = pixel_fetch(ty + k, psh[k]);
            }
            if (FIRST) multiplies = pw.i < n_cnt && computes(pw);
            if (!FIRST && new_init) init16 = load16(&s_initA[cb * 32 + half * 16]);
            new_init = false;
            if (multiplies) {
                if (FIRST) {
                    // Operands (first_tap): the four rows of the window at this lane's column + its half, and at column + 2
                    const uint8_t *pix = (const uint8_t *)&s_pix[0][0][0] + (xb * 32 + pxl) * 8;
                    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                    u32x2 near[RW + 2], far[RW], corner[RW];
#pragma unroll
                    for (int r = 0; r < RW + 2; ++r) near[r] = *(const u32x2 *)(pix + slot_of(2 * sg - 1 + r) * (kHaloW * 8) + hf * 8);
#pragma unroll
                    for (int r = 0; r < RW; ++r) {
                        const int up = slot_of(2 * sg - 1 + r), mid = slot_of(2 * sg + r), low = slot_of(2 * sg + 1 + r); // the same for the whole wavefront
                        far[r] = *(const u32x2 *)(pix + (hf ? mid : up) * (kHaloW * 8) + 16);
                        corner[r] = *(const u32x2 *)(pix + low * (kHaloW * 8) + 16);
                    }
                    bf16x8 bfrag[RW][3];
#pragma unroll
                    for (int r = 0; r < RW; ++r) {
                        auto taps = [](u32x2 t0, u32x2 t1) { return __builtin_bit_cast(bf16x8, (u32x4){t0[0], t0[1], t1[0], t1[1]}); };
                        bfrag[r][0] = taps(near[r], near[r + 1]);
                        bfrag[r][1] = taps(near[r + 2], far[r]);
                        bfrag[r][2] = taps(corner[r], corner[r]);
                    }
#pragma unroll
                    for (int r = 0; r < RW; ++r) acc[r] = mfma32(Wr[0][0], bfrag[r][0], init16);
#pragma unroll
                    for (int f = 1; f < kFirstFrags; ++f)
#pragma unroll
                        for (int r = 0; r < RW; ++r) acc[r] = mfma32(Wr[f / 3][f % 3], bfrag[r][f % 3], acc[r]);
                } else {
                    strip_mma<C, RW>(rowp, Wr, acc, init16, []() {});
                }
            }
            if (!FIRST) input_loads(sg);
            // kHandOver: the first of the rows group B accumulated two steps ago, beside the matrix instructions just issued
            const bool fin = kHandOver && sg >= 4 && pe.i < n_cnt && owns(pe);
            u32x4 pk_b[2];
            if (fin) {
                const float *srcx = &s_accx[(((sg & 1) * 4 + w4) * 4) * 256 + ln * 4];
                f32x16 a;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 v = *(const f32x4 *)(srcx + q * 256);
                    a[4 * q] = v[0]; a[4 * q + 1] = v[1]; a[4 * q + 2] = v[2]; a[4 * q + 3] = v[3];
                }
                finish_pack(a, 0, pe, pk_b);
            }
            uint8_t *seam_rows = nullptr;          // WIDE: where the seam columns of this step's rows go, if anywhere
            if (multiplies) {
                // epilogue: ReLU, bf16 -> intermediate ring (zeros outside the tile)
                const int x = pw.b * kTileW + xl;  // this lane's column within the tile
                const uint32_t dbase = dither16(x, 2 * pw.s);
                // WIDE: the last two columns of the block also go to the seam (seam_flush below): the workgroup's
                // own (for its next column block) or the image's (the tile's last two columns, for conv_seam_kernel)
                if (WIDE) {
                    if (pw.b + 1 < J) seam_rows = st.seam + ((size_t)blockIdx.x * 2 + (pw.b & 1)) * seam_half;
                    else if (st.seam_last && owns(pw)) seam_rows = st.seam_last + (size_t)(n_begin + pw.i) * seam_half;
                    if (seam_rows) seam_rows += (size_t)(2 * pw.s) * kSeamRowBytes;
                }
#pragma unroll
                for (int r = 0; r < RW; ++r) {
                    const int y = 2 * pw.s + r;
                    u32x4 pk[2];
                    packed_row(acc[r], dbase ^ ((uint32_t)r << 15), pk);
#pragma unroll
                    for (int hq = 0; hq < 2; ++hq) {
                        if (y >= g.h || x >= g.w) pk[hq] = (u32x4){0u, 0u, 0u, 0u};
                        *(u32x4 *)(ring_mid + slot_of(2 * sg + r) * ROWB + (1 + kSkew + xl) * K::PS + (cb * 32 + hf * 16 + 8 * hq) * 2) = pk[hq];
                    }
                }
            } else { // opening position: zero padding of the second block, below the unit before and above this one
#pragma unroll
                for (int r = 0; r < RW; ++r)
#pragma unroll
                    for (int hq = 0; hq < 2; ++hq)
                        *(u32x4 *)(ring_mid + slot_of(2 * sg + r) * ROWB + (1 + kSkew + xl) * K::PS + (cb * 32 + hf * 16 + 8 * hq) * 2) =
                            (u32x4){0u, 0u, 0u, 0u};
                if (!FIRST && pw.b == 0 && pw.i < n_cnt) { // nobody reads s_initA in this step
                    prepare_init(n_begin + pw.i);
                    new_init = true;
                }
            }
            if (FIRST) {
                // WIDE: once per step this group waits for all of its global memory traffic, at a point where it has
                // to wait for its loads anyway; the stores of the previous step are then known to be done, among them
                // the seam rows, which are read back a whole unit - at least two steps - after they were written.
                if (WIDE) __builtin_amdgcn_s_waitcnt(kWaitVm0);
#pragma unroll
                for (int k = 0; k < 2; ++k) // their slots were last read two steps ago
                    pixel_store(2 * sg + 3 + k, pix_inside && (uint32_t)(ty + k) < (uint32_t)g.h, pv[k], psh[k]);
                if (fin) finish_store(0, pe, pk_b); // behind the wait for the pixels, which would sit these stores out
            }
            if (WIDE) seam_flush(seam_rows, sg);
            // the end of this group's step
            const bool rows_issued = pe.i < n_cnt;
            advance(pw);
            if (FIRST) {
                advance(p1);
                if (p1.i < n_cnt && p1.s == opening(p1.i)) pixel_first_unit(p1);
            }
            if (!FIRST || sg >= 4) advance(pe);
            if (!FIRST) {
                prepare_step(sg + 1);
                if (WIDE && w4 == 0) { // the seam columns have landed
                    if (rows_issued) __builtin_amdgcn_s_waitcnt(kWaitVm0 | kFirstWaveLoads);
                    else __builtin_amdgcn_s_waitcnt(kWaitVm0);
                }
            }
            lds_barrier();
        }
        return;
    }

    // ---- group B
    const f32x16 bias16 = load16(&s_biasB[cb * 32 + half * 16]); // the sums start from it
    bool accumulated = false; // rows of the step before wait for their epilogue
#pragma unroll 1
    for (int sg = 0; sg < n_steps; ++sg) {
        const int ln = pin_in_loop(tid & 63);
        if (accumulated) {
            if (kHandOver) { // the first row to group A, which finishes it in the next step
                float *dst = &s_accx[((((sg - 1) & 1) * 4 + w4) * 4) * 256 + ln * 4];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *(f32x4 *)(dst + q * 256) = (f32x4){acc[0][4 * q], acc[0][4 * q + 1], acc[0][4 * q + 2], acc[0][4 * q + 3]};
            }
            if (!LASTB) {
                u32x4 pk[RW][2];
#pragma unroll
                for (int r = kHandOver ? 1 : 0; r < RW; ++r) finish_pack(acc[r], r, pe, pk[r]);
#pragma unroll
                for (int r = kHandOver ? 1 : 0; r < RW; ++r) finish_store(r, pe, pk[r]);
            }
            finish_statistics(acc, pe);
        }
        if (WIDE && FIRST && w4 == 0) seam_loads(sg, p1); // (group A is the critical path of this variant)
        auto end_of_step = [&]() {
            if (WIDE && FIRST && w4 == 0) __builtin_amdgcn_s_waitcnt(kWaitVm0); // the seam columns have landed
            lds_barrier();
        };
        accumulated = sg >= 2 && pw.i < n_cnt && owns(pw);
        if (accumulated) {
            lrow_t rowp[RW + 2];
#pragma unroll
            for (int r = 0; r < RW + 2; ++r) rowp[r] = mid_base + (uint32_t)slot_of(2 * (sg - 2) - 1 + r) * ROWB;
            strip_mma<C, RW>(rowp, Wr, acc, bias16, end_of_step);
        } else {
            end_of_step();
        }
        if (sg >= 2) advance(pw);
        if (sg >= 3) advance(pe);
        if (FIRST) advance(p1);
    }
}

// The last output column of a fused launch on a tile whose width is a multiple of 64 (see conv_pair_kernel,
// WIDE): out[r][w-1] from the intermediate columns w-2, w-1 that group A left in the per-image seam buffer; the
// column right of them is the zero padding, so only the taps dx = 0, 1 count.  One workgroup of two wavefronts
// (one per 32 output channels) per 32 rows of an image; a lane's pixel is a row.  Operands come straight from
// global memory: the launch is a fraction of a percent of the fused one's work.
// LASTB: instead of activations the column's lines of the nine border-aware channel sums (LastSums).
template <int C, bool LASTB>
__global__ __launch_bounds__(128) void conv_seam_kernel(const uint8_t *__restrict__ seam_last, ConvGeom g,
                                                        const bf16_t *__restrict__ wfragB, const float *__restrict__ biasB,
                                                        float *__restrict__ tout, int out_recs, LastSums sums,
                                                        bf16_t *__restrict__ out)
{
    typedef MidCfg<C> K;
    const int lane = threadIdx.x & 63;
    const int cb = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int px = lane & 31, half = lane >> 5;
    const int tiles = (g.h + 31) / 32;
    const int n = blockIdx.x / tiles, t = blockIdx.x - n * tiles;
    const int r = t * 32 + px; // this lane's output row
    const uint8_t *sl = seam_last + (size_t)n * (2 * ((g.h + 1) / 2)) * kSeamRowBytes;
    const bf16x8 *wp = (const bf16x8 *)wfragB + (size_t)cb * 9 * K::KC * 64 + lane;
    // all operands are asked for before the first is used (unconditional loads from a clamped row; what lies
    // outside the tile is dropped afterwards): the launch is bound by memory latency, not by its 24 matrix instructions
    u32x4 bv[3][2][K::KC];
    bf16x8 av[3][2][K::KC];
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) {
        const int yc = clampi(r + dy - 1, 0, g.h - 1);
#pragma unroll
        for (int dx = 0; dx < 2; ++dx)
#pragma unroll
            for (int kc = 0; kc < K::KC; ++kc) {
                bv[dy][dx][kc] = *(const u32x4 *)(sl + (size_t)yc * kSeamRowBytes + dx * (C * 2) + (kc * 16 + half * 8) * 2);
                av[dy][dx][kc] = wp[((dy * 3 + dx) * K::KC + kc) * 64];
            }
    }
    f32x16 sum = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) {
        const int y = r + dy - 1;
        const bool ok = y >= 0 && y < g.h;
#pragma unroll
        for (int dx = 0; dx < 2; ++dx)
#pragma unroll
            for (int kc = 0; kc < K::KC; ++kc) {
                const u32x4 b = ok ? bv[dy][dx][kc] : (u32x4){0u, 0u, 0u, 0u};
                sum = mfma32(av[dy][dx][kc], __builtin_bit_cast(bf16x8, b), sum);
            }
    }
    const float *bp = biasB + cb * 32 + half * 16;
    float val[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) val[v] = sum[v] + bp[v];
    if constexpr (!LASTB) {
        if (r < g.h) {
            bf16_t *dst = out + (((size_t)n * g.h + r) * g.w + (g.w - 1)) * C + cb * 32 + half * 16;
            u32x4 lo, hi;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                lo[v] = pack_bf16_relu(val[2 * v], val[2 * v + 1], dither16(g.w - 1, r), true);
                hi[v] = pack_bf16_relu(val[8 + 2 * v], val[8 + 2 * v + 1], dither16(g.w - 1, r), true);
            }
            *(u32x4 *)dst = lo;
            *(u32x4 *)(dst + 8) = hi;
        }
    } else if (tout) {
        // a line for these rows of the last column, and the column's first / last row: the right corners
        float *lines = tout + (int64_t)n * out_recs * C + cb * 32 + half * 16;
        float col[16], tot[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            col[v] = r < g.h ? fmaxf(val[v], 0.f) : 0.f;
            tot[v] = half_sum(col[v]);
        }
        auto put = [](float *dst, const float (&src)[16]) {
#pragma unroll
            for (int q = 0; q < 4; ++q) *(f32x4 *)(dst + 4 * q) = (f32x4){src[4 * q], src[4 * q + 1], src[4 * q + 2], src[4 * q + 3]};
        };
        if (px == kSumLane) put(lines + (sums.last_col + t) * C, tot);
        if (r == 0) put(lines + (sums.corners + 1) * C, col);
        if (r == g.h - 1) put(lines + (sums.corners + 3) * C, col);
    }
}

// ------------------------------------------------------------------------------------------------
// First layer: u8 planes -> crop -> normalise -> conv3x3 (3 -> C) + bias + ReLU -> bf16 NHWC.
// The normalisation is folded into the weights, so that the operands of the matrix cores are exact:
//   sum_c w[c] * (p_c / 255 - mean_c) / std_c  =  sum_c (w[c] / (255 std_c)) * p_c  +  (- sum_c w[c] mean_c / std_c) * 1
// A workgroup stages the (4+2) x (64+2) window of the tile as pixels of 4 bf16 channels (8 bytes) in LDS: the
// three bytes as they are (0..255 are exact in bf16) and a fourth channel that is 1 inside the tile; whatever
// lies outside the tile is four zeros, which is the zero padding of the normalised domain exactly (the
// constant term vanishes with the indicator).  The weights of the four channels are kept as bf16 high part +
// bf16 residual, i.e. to about 16 bits.  K = 9 taps x 4 channels = 36, padded to 48 = three 16-wide k chunks;
// a lane's 8 k values of a chunk are two taps, i.e. two 8-byte LDS reads.  A wavefront computes one 32-channel
// output block for one (C = 32) or two (C = 64) rows of the strip.
//
// Bound by the bf16 output it writes and by vector instructions.  The raw pixels of the next strip are fetched while this one is
// multiplied, as the aligned dwords that hold a lane's four pixels of a colour, and go into the other of two windows, so that
// a strip has one barrier, which waits for LDS only; columns of 32 that lie outside the tile are left out; the output passes
// LDS, so that four lanes write 64 bytes of a pixel together.  Against single bytes, asked for and waited for between two barriers
// that also wait for the strip's stores: 2000 tiles of 32 x 32, 32 channels 56 -> 36 us (3.7 TB/s written), 500 of 100 x 100
// 109 -> 78 (4.1), 100 of 75 x 100, 64 channels 28.8 -> 22.6.  The two halves of a wavefront's pixels swapped between rows of 16
// lanes instead, each store 64 bytes of 16 pixels from lanes 16 apart: 500 of 100 x 100 171 us where two 16-byte pieces 32 bytes
// apart took 117.
// ------------------------------------------------------------------------------------------------
constexpr int kFirstPix = (kRows + 2) * kHaloW;

template <int C>
__global__ __launch_bounds__(256, 4) void conv_first_kernel(TileSrc src, ConvGeom g, const bf16_t *__restrict__ wfrag,
                                                         const float *__restrict__ bias, float *__restrict__ tout,
                                                         int out_recs, int per, bf16_t *__restrict__ out)
{
    constexpr int NCB = C / 32;
    __shared__ __attribute__((aligned(16))) uint16_t lds[2][kFirstPix * 4]; // strips in turn
    __shared__ u32x4 s_out[4][32 * 4]; // a wavefront's 32 pixels x 32 channels on their way out
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int px = lane & 31, half = lane >> 5;

    // a wavefront owns one 32-channel output block and NCB of the strip's rows
    const int cb = wave % NCB;
    const int rbase = (wave / NCB) * NCB;
    // weights as bf16 high part + bf16 residual: this layer is tiny, so it is computed to ~16 bits
    bf16x8 Wr[kFirstFrags];
#pragma unroll
    for (int f = 0; f < kFirstFrags; ++f) Wr[f] = ((const bf16x8 *)wfrag)[(cb * kFirstFrags + f) * 64 + lane];
    f32x16 bias16;
    {
        const float4 *bp = (const float4 *)(bias + cb * 32 + half * 16);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 bq = bp[q];
            bias16[4 * q] = bq.x; bias16[4 * q + 1] = bq.y; bias16[4 * q + 2] = bq.z; bias16[4 * q + 3] = bq.w;
        }
    }

    // LDS byte offsets (relative to the lane's output pixel) of the two taps of each k chunk
    int toff[3][2];
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int tap = first_tap(q, half, j);
            toff[q][j] = ((tap / 3) * kHaloW + tap % 3) * 8;
        }

    const int plane = src.H * src.W;
    const uint32_t img_bytes = (uint32_t)((size_t)g.h * g.w * C * 2);

    const int tpi = g.strips * g.colblks;
    const int total = g.n_img * tpi;
    const int t_begin = blockIdx.x * per;
    const int t_end = min(total, t_begin + per);
    if (t_begin >= t_end) return;

    // Four pixels of a row of the window are a lane's: 17 times 6, half of the wavefronts for one strip, the others for the next
    constexpr int GROUPS = (kHaloW + 3) / 4;
    static_assert(GROUPS * (kRows + 2) <= 128, "two wavefronts");
    const int unit = tid & 127, row_of = min(unit / GROUPS, kRows + 1), group = unit % GROUPS;
    struct Strip {
        int n, strip, colblk;
    };
    auto advance = [&](Strip &q) {
        if (++q.colblk == g.colblks) {
            q.colblk = 0;
            if (++q.strip == g.strips) {
                q.strip = 0;
                ++q.n;
            }
        }
    };
    uint32_t word[3][2];
    uint32_t shift[3];
    // The aligned dwords that hold the first and the last of them that lies in the tile (neither leaves the page of such a byte)
    auto fetch = [&](const Strip &q) {
        int oy = 0, ox = 0;
        if (src.off) {
            const scalar_ints_t off = (scalar_ints_t)(uintptr_t)src.off + 2 * q.n;
            oy = clampi(off[0], 0, src.H - g.h);
            ox = clampi(off[1], 0, src.W - g.w);
        }
        const uint8_t *tile0 = src.img + (int64_t)q.n * 3 * plane + (int64_t)oy * src.W + ox;
        const int x = q.colblk * kTileW - 1 + 4 * group, first = clampi(x, 0, g.w - 1), last = clampi(x + 3, 0, g.w - 1);
        const uint8_t *row = tile0 + (int64_t)clampi(q.strip * kRows - 1 + row_of, 0, g.h - 1) * src.W;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const uintptr_t at = (uintptr_t)(row + (int64_t)c * plane);
            word[c][0] = *(global_word_t)((at + first) & ~(uintptr_t)3);
            word[c][1] = *(global_word_t)((at + last) & ~(uintptr_t)3);
            shift[c] = (uint32_t)at + (uint32_t)x;
        }
    };
    // .. -> pixels in `window`
    auto stage = [&](const Strip &q, uint16_t *window) {
        const int x = q.colblk * kTileW - 1 + 4 * group;
        const bool row_inside = (uint32_t)(q.strip * kRows - 1 + row_of) < (uint32_t)g.h;
        uint32_t byte[3]; // of the four
#pragma unroll
        for (int c = 0; c < 3; ++c) byte[c] = __builtin_amdgcn_alignbyte(word[c][1], word[c][0], shift[c]);
        u32x4 to[2];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool inside = row_inside && (uint32_t)(x + i) < (uint32_t)g.w;
            uint32_t f[3]; // exact in bf16, the high half
#pragma unroll
            for (int c = 0; c < 3; ++c) f[c] = __builtin_bit_cast(uint32_t, (float)(byte[c] >> (8 * i) & 0xffu));
            to[i / 2][i % 2 * 2] = inside ? __builtin_amdgcn_perm(f[1], f[0], 0x07060302u) : 0u;
            to[i / 2][i % 2 * 2 + 1] = inside ? f[2] >> 16 | 0x3F800000u : 0u;
        }
        if (unit < GROUPS * (kRows + 2)) {
            u32x4 *at = (u32x4 *)(window + (row_of * kHaloW + 4 * group) * 4);
            at[0] = to[0];
            if (group < GROUPS - 1) at[1] = to[1]; // (a row has two columns more than whole groups)
        }
    };
    static_assert(kHaloW % 4 == 2, "the last group is two pixels");
    const int turn = wave / 2;
    Strip q{t_begin / tpi, t_begin / g.colblks % g.strips, t_begin % g.colblks}, ahead = q;
    if (turn == 0) fetch(q);
    __builtin_amdgcn_s_waitcnt(kWaitVm0); // the weights are there: a wait for them in the loop would be one for all that is under way

    for (int t = t_begin; t < t_end; ++t) {
        const int colblk = q.colblk, strip = q.strip, n = q.n;
        const int y0 = strip * kRows, x0 = colblk * kTileW;
        const int parity = (t - t_begin) & 1;
        uint16_t *window = lds[parity];
        if (turn == parity) stage(q, window);
        if (t + 1 < t_end) advance(ahead);
        if (turn != parity && t + 1 < t_end) fetch(ahead); // on their way while this strip is multiplied
        lds_barrier(); // (one a strip: whoever writes the window again has passed the next strip's, behind the last reads of this one)

        const bool sample = tout && (strip & 7) == sampled_strip(g.strips);
        float tv[16] = {}; // sampled strip: channel sums over this wavefront's rows, this lane's columns
#pragma unroll
        for (int rr = 0; rr < NCB; ++rr) {
            const int row = rbase + rr;
            const int y = y0 + row;
            if (y >= g.h) continue; // same for the whole wavefront
#pragma unroll
            for (int xb = 0; xb < 2; ++xb) {
                if (x0 + xb * 32 >= g.w) continue; // (likewise)
                const int x = x0 + xb * 32 + px;
                const uint8_t *lp = (const uint8_t *)window + (row * kHaloW + xb * 32 + px) * 8;
                bf16x8 bfrag[3];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                    const u32x2 lo = *(const u32x2 *)(lp + toff[q][0]);
                    const u32x2 hi = *(const u32x2 *)(lp + toff[q][1]);
                    const u32x4 both = {lo[0], lo[1], hi[0], hi[1]};
                    bfrag[q] = __builtin_bit_cast(bf16x8, both);
                }
                const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                f32x16 sum = mfma32(Wr[0], bfrag[0], zero);
#pragma unroll
                for (int f = 1; f < kFirstFrags; ++f) sum = mfma32(Wr[f], bfrag[f % 3], sum);
                f32x16 acc;
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[v] = sum[v] + bias16[v];
                const uint32_t dth = dither16(x, y);
                u32x4 *piece = s_out[wave] + px * 4;
#pragma unroll
                for (int hq = 0; hq < 2; ++hq) {
                    u32x4 pk;
#pragma unroll
                    for (int e = 0; e < 4; ++e) pk[e] = pack_bf16_relu(acc[8 * hq + 2 * e], acc[8 * hq + 2 * e + 1], dth, true);
                    piece[(half * 2 + hq) ^ (px >> 2 & 3)] = pk;
                }
                uint8_t *img = (uint8_t *)out + (size_t)n * img_bytes;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int p = i * 16 + (lane >> 2), xs = x0 + xb * 32 + p;
                    const u32x4 pk = s_out[wave][p * 4 + ((lane & 3) ^ (p >> 2 & 3))];
                    store16(img, img_bytes, xs < g.w ? (uint32_t)(((y * g.w + xs) * C + cb * 32 + (lane & 3) * 8) * 2) : kOutside, 0, pk);
                }
                if (sample) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) tv[v] += x < g.w ? fmaxf(acc[v], 0.f) : 0.f;
                }
            }
        }
        if (sample) { // a record per sampled strip, column block and wavefront of the same channels
            const int ri = ((strip >> 3) * g.colblks + colblk) * (4 / NCB) + wave / NCB;
            float *rec = tout + ((int64_t)n * out_recs + ri) * C + cb * 32 + half * 16;
#pragma unroll
            for (int v = 0; v < 16; ++v) tv[v] = half_sum(tv[v]);
            if (px == kSumLane) {
#pragma unroll
                for (int q = 0; q < 4; ++q) *(f32x4 *)(rec + 4 * q) = (f32x4){tv[4 * q], tv[4 * q + 1], tv[4 * q + 2], tv[4 * q + 3]};
            }
        }
        q = ahead;
    }
}

// ------------------------------------------------------------------------------------------------
// All blocks of the extractor in one launch, for batches of few tiles.
//
// A block of a small batch is a launch of 5 .. 14 us of which its matrix instructions take one to four: the rest is the launch
// itself, the round trips to memory that it begins and ends with, and the weights on their way.  Here the images are dealt to the
// XCDs, whose workgroups hand rows to each other through their L2.  A block of an image is cut into items of ROWS rows x 32
// columns (the first block: 64 columns), and the workgroups of an XCD, one to a compute unit, draw items from one counter in the
// order (chunk of images, block, image, strip, column block).  An item waits until all items of its image in the block before are
// done (a counter per block and image), since the correction of its bias takes means over the image.
//   No wait can last, whatever else runs on the device and however the workgroups are dealt to the XCDs: an item only waits for
// items with lower numbers of the same XCD, and those have been drawn by workgroups that are running; the lowest unfinished
// item waits for none.  Whoever draws a chunk's first number claims the next chunk of images for its XCD, so that an XCD without
// workgroups gets none.
//   What a later item reads has been stored in the L2 (s_waitcnt vmcnt) when the counter says so, and is loaded past the
// compute unit's own cache (load16c, load_lds16c).  A hand-over between 8 workgroups of an XCD takes 1.0 us and 1.7 through the
// memory behind the L2s, between 32 it takes 2.0 and 3.6; fences, which write back and invalidate a whole L2, made that 3 and 5.
//   Products, sums, records, lines and roundings are those of conv_first_kernel and conv_mid_kernel, in their order: the results
// are the same bit for bit, so that a tile's do not depend on whether the batch around it is small enough for this launch.  A
// wavefront therefore multiplies the rows that one of conv_mid_kernel has of a strip, or half of them in the order that they come
// in there (half_mma); one wavefront sums the image's records up, or each for itself, never several in shares.  (64 channels: pairs of
// rows instead of strips of four, records shared by the wavefronts and the correction behind the products are 3 % faster, 7 tiles of
// 128 x 128, eight blocks and the head 106.7 us instead of 110.3, but then a tile's logits change with the number of tiles.)
//   The state (ChainState) is all zeros when the launch begins; the launch behind it, which reads its results, clears it again.
//   Waits are bounded all the same.  An item whose wait has run out is not counted, nor then is any that waits for it, and the first such wait
// cuts the others short; the launch behind finds the counts wrong, gives NaN for the image's logits and tells the host (ChainState::lost).
// ------------------------------------------------------------------------------------------------
struct ChainArgs {
    TileSrc src;
    ConvGeom g;
    int blocks;               // blocks to run
    const bf16_t *w_first, *w_mid;
    const float *bias, *rsum; // [blocks][C], [blocks - 1][C][C]
    uint8_t *act[2];          // block b writes act[b & 1]
    float *rec[2];            // its channel sums: rec[b & 1]
    MeanIn first, mid;        // what a consumer has to know of those of the first block, of another one (rec unused)
    float *lines;             // what the last block leaves, or null: it writes activations as the others do
    int64_t lines_stride;     // floats from image to image
    uint32_t *state;          // ChainState
    int patience;             // looks that a wait takes
    int chunk, chunks;        // images that an XCD takes at a time, chunks of them
};
// ChainState, in words: chunks claimed; from kChainTeamAt on, for every XCD, numbers drawn, the chunks it has claimed (plus one) and, at
// kChainGaveUp, whether a wait has run out; from kChainCountAt on, for every block and image, items done.  (A line of 128 bytes for what
// is counted apart.)
constexpr int kChainTeamAt = 32, kChainTeams = 8, kChainTeam = 32, kChainCountAt = kChainTeamAt + kChainTeams * kChainTeam, kChainCount = 32;
constexpr int kChainGaveUp = 16;
constexpr int kChainCols = 32;
constexpr int kChainPatience = 1 << 22; // looks, seconds: never reached (see above), but a fault elsewhere is not to hang the device
constexpr int kChainLook = 1024;        // so many looks apart, a wait sees whether another one has run out

// WAVES of a workgroup, RW: rows that a wavefront multiplies at a time, STEPS: times it does
template <int C, int WAVES, int RW, int STEPS>
struct ChainCfg {
    typedef MidCfg<C> K;
    static constexpr int RG = WAVES / K::NCB;           // wavefronts one above the other
    static constexpr int ROWS = RG * RW * STEPS;
    static constexpr int SR = 2 * K::NCB;               // rows that a wavefront of conv_mid_kernel has of a strip,
    static constexpr int SG = kRows / SR;               // .. and how many such groups of rows a strip is: sums and dither are by them
    static constexpr bool HALVES = RW < SR;             // here such a group may be two wavefronts' (an item of few rows)
    static_assert(RW == SR || (2 * RW == SR && STEPS == 1 && (C == 64 || ROWS == kRows)), "whole groups of rows");
    static constexpr int THREADS = 64 * WAVES;
    static constexpr int HALO = kChainCols + 2;
    static constexpr int ROWB = HALO * K::PS;           // a staged row
    static constexpr int ROW_SLOTS = HALO * K::SPP;
    static constexpr int SLOTS = (ROWS + 2) * ROW_SLOTS; // of 16 bytes, all rows one behind the other
    static constexpr int LOADS = (SLOTS + THREADS - 1) / THREADS; // per thread
    static constexpr int PIX = (ROWS + 2) * kHaloW;     // first block: staged pixels of 8 bytes
    // Of the three horizontal taps, those whose weights come in through LDS while the block before is multiplied: as many as it has room for
    static constexpr int AHEAD = LOADS * THREADS * 16 + 9 * K::KC * K::NCB * 1024 <= 150 * 1024 ? 3 : 2;
    static constexpr int FRAGS = AHEAD * 3 * K::KC;     // .. and their fragments for one block of 32 output channels
    // The wavefronts that ask for them, the second ones of their SIMDs, whose turn on the matrix pipes comes later: the loads take 0.5 us to be issued
    static constexpr int LOADERS = WAVES == 4 ? 2 : C == 64 ? 4 : 3;
    static_assert(K::NCB * FRAGS % LOADERS == 0, "whole fragments to a wavefront");
};

// RW output rows of 32 pixels x 32 channels, the upper or (LOWER) the lower half of a group: their products in the order of
// strip_mma<C, 2 * RW>, whose fragments that such a half does not need are left out.
template <int C, bool LOWER, int RW>
struct HalfOrder {
    static constexpr int NT = (RW + 2) * MidCfg<C>::KC * 3; // fragments
    int row[NT], kc[NT], dx[NT];
    constexpr HalfOrder() : row(), kc(), dx()
    {
        constexpr int NP = RW + 1, KP = MidCfg<C>::KC / 2; // as there
        int t = 0;
        for (int s2 = 0; s2 < 3 * KP * NP; ++s2)
            for (int j = 0; j < 4; ++j) {
                const int r = s2 % NP + (j & 1) * NP - (LOWER ? RW : 0);
                if (r < 0 || r >= RW + 2) continue;
                row[t] = r;
                kc[t] = 2 * (s2 / NP % KP) + (j >> 1);
                dx[t++] = s2 / (NP * KP);
            }
    }
};
template <int C, bool LOWER, int RW>
__device__ __forceinline__ void half_mma(const lrow_t (&rowp)[RW + 2], const bf16x8 (&Wr)[9][C / 16], f32x16 (&acc)[RW])
{
    asm volatile(".p2align 5");
    typedef MidCfg<C> K;
    constexpr HalfOrder<C, LOWER, RW> at;
    constexpr int NF = 4, NT = at.NT;
    bool started[RW] = {};
    bf16x8 f[NF];
    unrolled<NF>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        frag_read<at.dx[t] * K::PS + at.kc[t] * 32>(f[t], rowp[at.row[t]]);
    });
    __builtin_amdgcn_sched_barrier(0);
    unrolled<NT>([&](auto tc) {
        constexpr int t = decltype(tc)::value;
        bf16x8 &fr = f[t % NF];
        frag_wait<(t + NF <= NT ? NF - 1 : NT - 1 - t)>(fr);
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) {
            const int orow = at.row[t] - dy;
            if (orow >= 0 && orow < RW) {
                acc[orow] = mfma32(Wr[dy * 3 + at.dx[t]][at.kc[t]], fr, started[orow] ? acc[orow] : kZeroAcc);
                started[orow] = true;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (t + NF < NT) {
            constexpr int u = t + NF;
            frag_read<at.dx[u] * K::PS + at.kc[u] * 32>(fr, rowp[at.row[u]]);
        }
        __builtin_amdgcn_sched_barrier(0);
    });
#pragma unroll
    for (int r = 0; r < RW; ++r) asm volatile("" : "+v"(acc[r])); // (the products stay where they are)
}

template <int C, int WAVES, int RW, int STEPS>
__global__ __launch_bounds__(64 * WAVES, 1) void conv_chain_kernel(ChainArgs a)
{
    typedef MidCfg<C> K;
    typedef ChainCfg<C, WAVES, RW, STEPS> G;
    constexpr int LDS_ROWS = G::LOADS * G::THREADS * 16;
    static_assert(G::PIX * 8 <= LDS_ROWS, "the first block's pixels take the rows' place");
    __shared__ __attribute__((aligned(1024))) uint8_t lds[LDS_ROWS];
    __shared__ __attribute__((aligned(1024))) uint8_t s_weights[K::NCB * G::FRAGS * 1024];
    __shared__ __attribute__((aligned(16))) float s_mean[C == 32 ? WAVES : 1][C]; // the image's means, 32 channels: for a wavefront's own use
    // what one wavefront of a group's halves hands the other, which sums it up: 32 channels the lower row, 64 the sums over the upper rows
    __shared__ __attribute__((aligned(16))) float s_handed[G::HALVES ? WAVES / 2 : 1][G::HALVES ? 1024 : 4];
    __shared__ __attribute__((aligned(16))) float s_init[WAVES][32];  // bias + correction of its outputs
    __shared__ __attribute__((aligned(16))) int s_next[2][8]; // the next item, by its parity within the workgroup: a slow wavefront may still read the one before

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cb = wave % K::NCB, rg = wave / K::NCB;
    const int strips = (a.g.h + G::ROWS - 1) / G::ROWS, colblks = (a.g.w + kChainCols - 1) / kChainCols;
    const int ipi0 = strips * a.g.colblks, ipi = strips * colblks;          // items of an image: first block, another one
    const int first_items = a.chunk * ipi0, block_items = a.chunk * ipi;    // of a chunk
    const uint32_t items = (uint32_t)(first_items + (a.blocks - 1) * block_items);
    const uint32_t img_bytes = (uint32_t)((size_t)a.g.h * a.g.w * C * 2);
    const int sample_phase = sampled_strip(a.g.strips);
    const int xcd = __builtin_amdgcn_s_getreg((3 << 11) | 20) % kChainTeams; // hwreg(HW_REG_XCC_ID, 0, 4)
    uint32_t *const team = a.state + kChainTeamAt + xcd * kChainTeam;

    // One lane draws the next item's number and tells the others what it is.  Between the draw and the claim of a chunk nothing is
    // waited for.
    struct Item {
        int b, n, y0, colblk; // b < 0: none, n < 0: and none will come
    };
    const bool draws = wave == WAVES - 1; // one lane of this wavefront
    // (an address per lane as far as the compiler can tell: it would look at the answer at once to hand it out to several lanes)
    auto draw = [&]() -> uint32_t {
        uint32_t t = 0;
        if ((tid & 63) == 0) t = __hip_atomic_fetch_add(team + pin_in_loop(0), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return t;
    };
    // the look number `polls` of a wait is its last one
    auto out_of_patience = [&](int polls) {
        return polls >= a.patience || (polls % kChainLook == 0 && __builtin_amdgcn_readfirstlane(__hip_atomic_load(team + kChainGaveUp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != 0);
    };
    auto give_up = [&]() {
        if ((tid & 63) == 0) __hip_atomic_store(team + kChainGaveUp, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    uint32_t my_chunk = 0, chunk_at = ~0u; // the chunk that numbers from chunk_at * items on are of, plus one
    auto drawn = [&](uint32_t answer, int to) __attribute__((always_inline)) {
        const uint32_t t = __builtin_amdgcn_readfirstlane(answer), q = t / items;
        if (q >= (uint32_t)kChainTeams) { // there are at most kChainTeams chunks, and an XCD's first ones are those that it got
            my_chunk = ~0u;
        } else if (t == q * items) { // the first of a chunk
            uint32_t c = 0;
            if ((tid & 63) == 0) {
                c = 1u + __hip_atomic_fetch_add(a.state, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(team + 1 + q, c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            my_chunk = __builtin_amdgcn_readfirstlane(c);
        } else if (q != chunk_at) {
            int polls = 0;
            do my_chunk = __builtin_amdgcn_readfirstlane(__hip_atomic_load(team + 1 + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            while (my_chunk == 0 && !out_of_patience(++polls)); // (whoever drew the chunk's first number claims it at once)
            if (my_chunk == 0) give_up(); // .. and this workgroup is done: nobody has the item
        }
        chunk_at = q;
        int i = (int)(t - q * items), b = 0, in_block = first_items, in_image = ipi0, across = a.g.colblks;
        if (i >= first_items) {
            i -= first_items;
            in_block = block_items;
            in_image = ipi;
            across = colblks;
            b = 1;
        }
        const int past = i / in_block, j = i - past * in_block, m = j / in_image, at = j - m * in_image, strip = at / across;
        const int n = (int)(my_chunk - 1) * a.chunk + m;
        const bool none = my_chunk - 1 >= (uint32_t)a.chunks;
        int *s = s_next[to];
        s[0] = !none && n < a.g.n_img ? b + past : -1;
        s[1] = none ? -1 : n;
        s[2] = strip * G::ROWS;
        s[3] = at - strip * across;
    };
    int parity = 0;
    // what has been drawn (and a barrier passed)
    auto next_item = [&]() {
        int v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_readfirstlane(s_next[parity][i]);
        parity ^= 1;
        return Item{v[0], v[1], v[2], v[3]};
    };
    auto counter = [&](int b, int n) { return a.state + kChainCountAt + ((size_t)b * a.g.n_img + n) * kChainCount; };
    // Until all items of image n in block b are done; the first wavefront knows whether they are.
    auto wait_for = [&](int b, int n) {
        bool there = true;
        if (wave == 0) {
            const uint32_t all = (uint32_t)(b == 0 ? ipi0 : ipi);
            int polls = 0;
            do there = __builtin_amdgcn_readfirstlane(__hip_atomic_load(counter(b, n), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == all;
            while (!there && !out_of_patience(++polls));
            if (!there) give_up();
        }
        lds_barrier();
        return there;
    };
    // The item is done but for its last stores; next: the answer to the draw, which is asked for when the item's rows are there: a workgroup
    // that drew before would hold two items of a block while others have none.
    auto done = [&](const Item &it, uint32_t next, bool counts) {
        asm volatile("" ::: "memory");
        if (draws) drawn(next, parity);
        __builtin_amdgcn_s_waitcnt(kWaitVm0); // the stores are in the L2
        lds_barrier();                        // .. those of all wavefronts, which also are done with what is in LDS
        if (tid == 0 && counts) __hip_atomic_fetch_add(counter(it.b, it.n), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };

    // Whether block b's rows of this strip leave sums
    auto is_last = [&](int b) { return b == a.blocks - 1 && a.lines; };
    auto leaves_sums = [&](int b, int strip) { return is_last(b) || (strip & 7) == sample_phase; };
    // Bias, ReLU, bf16 and stores of the wavefront's rows, from row yw of the image on (conv_mid_kernel's epilogue)
    auto store_rows = [&](const Item &it, int yw, const f32x16 (&acc)[RW]) __attribute__((always_inline)) {
        const int ln = pin_in_loop(tid & 63), x = it.colblk * kChainCols + (ln & 31), half = ln >> 5;
        const float *si = &s_init[wave][half * 16];
        uint8_t *out = a.act[it.b & 1] + (size_t)it.n * img_bytes;
        const uint32_t dbase = dither16(x, yw & ~(G::SR - 1)); // (its rows are quarter steps apart)
#pragma unroll
        for (int hq = 0; hq < 2; ++hq) {
            const f32x4 b0 = *(const f32x4 *)(si + 8 * hq), b1 = *(const f32x4 *)(si + 8 * hq + 4);
#pragma unroll
            for (int r = 0; r < RW; ++r) {
                const uint32_t dth = dbase ^ ((uint32_t)((RW == G::SR ? 0 : yw & (G::SR - 1)) + r) << 14);
                u32x4 pk;
                pk[0] = pack_bf16_relu(acc[r][8 * hq + 0] + b0[0], acc[r][8 * hq + 1] + b0[1], dth, true);
                pk[1] = pack_bf16_relu(acc[r][8 * hq + 2] + b0[2], acc[r][8 * hq + 3] + b0[3], dth, true);
                pk[2] = pack_bf16_relu(acc[r][8 * hq + 4] + b1[0], acc[r][8 * hq + 5] + b1[1], dth, true);
                pk[3] = pack_bf16_relu(acc[r][8 * hq + 6] + b1[2], acc[r][8 * hq + 7] + b1[3], dth, true);
                const bool inside = yw + r < a.g.h && x < a.g.w;
                store16(out, img_bytes, inside ? (uint32_t)((((yw + r) * a.g.w + x) * C + cb * 32 + half * 16 + 8 * hq) * 2) : kOutside, 0, pk);
            }
        }
    };
    // The sums of a group of SR rows, whose last ones these are (from row yw on; above: the lane's sums over the others); WHOLE false:
    // more rows follow
    auto sum_rows = [&](const Item &it, int yw, const auto &acc, auto whole, const float (&above)[16]) __attribute__((always_inline)) {
        constexpr bool WHOLE = decltype(whole)::value;
        constexpr int N = sizeof acc / sizeof acc[0];
        const int ln = pin_in_loop(tid & 63), px = ln & 31, half = ln >> 5;
        const int x0 = it.colblk * kChainCols, x = x0 + px, strip = yw / kRows, group = yw / G::SR % G::SG, blk = it.colblk / 2, xb = it.colblk % 2;
        const float *si = &s_init[wave][half * 16];
        const int piece = group * 2 + xb;
        // a last block of 32 columns that stands alone also leaves the (empty) sums of the one beside it
        const bool alone = xb == 0 && x0 + kChainCols >= a.g.w;
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        if (is_last(it.b)) {
            float *lines = a.lines + it.n * a.lines_stride + cb * 32 + half * 16;
            LinePlaces p; // those of conv_mid_last_sums()
            p.first_col = a.g.strips * a.g.colblks * 2 * G::SG;
            p.last_col = p.first_col + a.g.strips * G::SG;
            p.rows = p.last_col + a.g.strips * G::SG;
            p.last_rows = p.rows + 2 * a.g.colblks;
            p.corners = p.last_rows + 2 * a.g.colblks;
            p.whole = (blk * a.g.strips + strip) * (2 * G::SG) + piece;
            p.col = strip * G::SG + group;
            p.row = blk * 2 + xb;
            last_lines<C, N, WHOLE>(acc, si, lines, p, x, x0, yw, a.g.h, a.g.w, px, above);
            if (alone && px < 4) {
                if (WHOLE) *(f32x4 *)(lines + (p.whole + 1) * C + 4 * px) = zero;
                if (yw == 0) *(f32x4 *)(lines + (p.rows + p.row + 1) * C + 4 * px) = zero;
                if (a.g.h - 1 - yw >= 0 && a.g.h - 1 - yw < N) *(f32x4 *)(lines + (p.last_rows + p.row + 1) * C + 4 * px) = zero;
            }
        } else if (WHOLE) {
            float *rec = a.rec[it.b & 1] + ((int64_t)it.n * a.mid.recs + ((strip >> 3) * a.g.colblks + blk) * (2 * G::SG) + piece) * C + cb * 32 + half * 16;
            strip_statistics<N>(acc, si, rec, x, yw, a.g.h, a.g.w, px, above);
            if (alone && px < 4) *(f32x4 *)(rec + C + 4 * px) = zero;
        }
    };

    // The weights of a block, 74 KB at 64 channels, come to the compute unit once, into LDS and while the block before is multiplied;
    // into registers they go while the block before is waited for.  (From memory for every wavefront they are 147 or 295 KB,
    // 1 .. 2 us, and the flags that are asked for behind them come in behind them.)
    int lds_of = 0; // the block whose weights s_weights holds (0: none)
    auto weights_to_lds = [&](int b) {
        lds_of = b;
        if (wave < WAVES - G::LOADERS) return;
        const bf16_t *w = a.w_mid + (size_t)(b - 1) * 9 * C * C;
        const int lane = pin_in_loop(tid & 63);
#pragma unroll
        for (int j = 0; j < K::NCB * G::FRAGS / G::LOADERS; ++j) {
            const int f = j * G::LOADERS + wave - (WAVES - G::LOADERS);
            const int block = f / G::FRAGS, r = f - block * G::FRAGS, dx = r / (3 * K::KC), kc = r / 3 % K::KC, dy = r % 3;
            __builtin_amdgcn_global_load_lds((gptr_t)((const bf16x8 *)w + ((block * 9 + dy * 3 + dx) * K::KC + kc) * 64 + lane), (lptr_t)(s_weights + f * 1024), 16, 0, 0);
        }
    };
    {
        uint32_t first = 0;
        if (draws) first = draw();
        weights_to_lds(1);
        if (draws) drawn(first, 0);
        lds_barrier();
    }
    Item it = next_item();
    // a number without an item: the next one's
    auto skip = [&]() {
        if (draws) drawn(draw(), parity);
        __syncthreads();
        it = next_item();
    };

    // ---- the first block, on the raw tile (conv_first_kernel, whose wavefronts take NCB rows each)
    auto first_block = [&]() __attribute__((always_inline)) {
        bf16x8 Wr[kFirstFrags];
        {
            const int lane = tid & 63;
#pragma unroll
            for (int f = 0; f < kFirstFrags; ++f) Wr[f] = ((const bf16x8 *)a.w_first)[(cb * kFirstFrags + f) * 64 + lane];
            if (lane < 32) s_init[wave][lane] = a.bias[cb * 32 + lane];
        }
#pragma unroll 1
        do {
            const int tid = pin_in_loop(threadIdx.x); // (nothing that follows from it is kept over the items)
            const int lane = tid & 63, px = lane & 31, half = lane >> 5, x0 = it.colblk * kTileW;
            int oy = 0, ox = 0;
            if (a.src.off) {
                oy = clampi(a.src.off[2 * it.n], 0, a.src.H - a.g.h);
                ox = clampi(a.src.off[2 * it.n + 1], 0, a.src.W - a.g.w);
            }
            const int plane = a.src.H * a.src.W;
            const uint8_t *tile0 = a.src.img + (int64_t)it.n * 3 * plane + (int64_t)oy * a.src.W + ox;
            constexpr int NB = (G::PIX * 3 + G::THREADS - 1) / G::THREADS;
            uint32_t v[NB];
#pragma unroll
            for (int k = 0; k < NB; ++k) { // all asked for before the first is used: from a pixel of the tile in any case
                const int idx = min(tid + k * G::THREADS, G::PIX * 3 - 1);
                const int c = idx / G::PIX, p = idx - c * G::PIX, row = p / kHaloW, col = p - row * kHaloW;
                v[k] = tile0[(int64_t)c * plane + (int64_t)clampi(it.y0 - 1 + row, 0, a.g.h - 1) * a.src.W + clampi(x0 - 1 + col, 0, a.g.w - 1)];
            }
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const int idx = tid + k * G::THREADS;
                const int c = idx / G::PIX, p = idx - c * G::PIX, row = p / kHaloW, col = p - row * kHaloW;
                const bool inside = (uint32_t)(it.y0 - 1 + row) < (uint32_t)a.g.h && (uint32_t)(x0 - 1 + col) < (uint32_t)a.g.w;
                if (idx < G::PIX * 3) {
                    uint16_t *q = (uint16_t *)lds + p * 4;
                    q[c] = inside ? (uint16_t)(__builtin_bit_cast(uint32_t, (float)v[k]) >> 16) : (uint16_t)0;
                    if (c == 0) q[3] = inside ? (uint16_t)0x3F80 : (uint16_t)0;
                }
            }
            lds_barrier();
            uint32_t next = 0;
            if (draws) next = draw();
            uint8_t *out = a.act[0] + (size_t)it.n * img_bytes;
            typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
#pragma unroll 1
            for (int row0 = rg * K::NCB; row0 < G::ROWS; row0 += G::RG * K::NCB) {
                const int strip = (it.y0 + row0) / kRows;
                if (strip >= a.g.strips) break;
                const bool sample = (strip & 7) == sample_phase;
                float tv[16] = {};
                const float *si = &s_init[wave][half * 16];
#pragma unroll 1
                for (int i = 0; i < 2 * K::NCB; ++i) { // rows, blocks of 32 columns
                    const int row = row0 + i / 2, y = it.y0 + row, x = x0 + i % 2 * 32 + px;
                    if (y >= a.g.h || x0 + i % 2 * 32 >= a.g.w) continue; // the same for the whole wavefront
                    const uint8_t *lp = lds + (row * kHaloW + i % 2 * 32 + px) * 8;
                    bf16x8 bfrag[3];
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        auto tap_at = [&](int j) { // (the halves of a wavefront may read different taps)
                            const int tap = half ? first_tap(q, 1, j) : first_tap(q, 0, j);
                            return *(const u32x2 *)(lp + ((tap / 3) * kHaloW + tap % 3) * 8);
                        };
                        const u32x2 t0 = tap_at(0), t1 = tap_at(1);
                        bfrag[q] = __builtin_bit_cast(bf16x8, (u32x4){t0[0], t0[1], t1[0], t1[1]});
                    }
                    f32x16 acc = kZeroAcc;
#pragma unroll
                    for (int f = 0; f < kFirstFrags; ++f) acc = mfma32(Wr[f], bfrag[f % 3], acc);
                    const uint32_t dth = dither16(x, y);
                    const uint32_t vo = x < a.g.w ? (uint32_t)(((y * a.g.w + x) * C + cb * 32 + half * 16) * 2) : kOutside;
#pragma unroll
                    for (int hq = 0; hq < 2; ++hq) {
                        u32x4 pk;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            acc[8 * hq + 2 * e] += si[8 * hq + 2 * e];
                            acc[8 * hq + 2 * e + 1] += si[8 * hq + 2 * e + 1];
                            pk[e] = pack_bf16_relu(acc[8 * hq + 2 * e], acc[8 * hq + 2 * e + 1], dth, true);
                        }
                        store16(out, img_bytes, vo + hq * 16, 0, pk); // (kOutside + 16 is outside, too)
                    }
                    if (sample) {
#pragma unroll
                        for (int v = 0; v < 16; ++v) tv[v] += x < a.g.w ? fmaxf(acc[v], 0.f) : 0.f;
                    }
                }
                if (sample) {
                    const int ri = ((strip >> 3) * a.g.colblks + it.colblk) * (kRows / K::NCB) + (it.y0 + row0) % kRows / K::NCB;
                    float *rec = a.rec[0] + ((int64_t)it.n * a.first.recs + ri) * C + cb * 32 + half * 16;
#pragma unroll
                    for (int v = 0; v < 16; ++v) tv[v] = half_sum(tv[v]);
                    if (px == kSumLane) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) *(f32x4 *)(rec + 4 * q) = (f32x4){tv[4 * q], tv[4 * q + 1], tv[4 * q + 2], tv[4 * q + 3]};
                    }
                }
            }
            done(it, next, true);
            it = next_item();
        } while (it.b == 0);
    };

    // ---- a block behind it
    auto later_blocks = [&]() __attribute__((always_inline)) {
        bf16x8 Wr[9][K::KC];
        int w_of = 0; // the block whose weights the registers hold (0: none)
        __builtin_amdgcn_s_waitcnt(kWaitVm0); // what has been asked for in the beginning (later on, done() waits for all that is under way)
        lds_barrier();
#pragma unroll 1
        do {
            const int tid = pin_in_loop(threadIdx.x);
            const int lane = tid & 63;
            if (w_of != it.b) {
                if (lds_of != it.b) {
                    weights_to_lds(it.b);
                    __builtin_amdgcn_s_waitcnt(kWaitVm0);
                    lds_barrier();
                }
#pragma unroll
                for (int dx = 0; dx < G::AHEAD; ++dx)
#pragma unroll
                    for (int kc = 0; kc < K::KC; ++kc)
#pragma unroll
                        for (int dy = 0; dy < 3; ++dy)
                            Wr[dy * 3 + dx][kc] = *(const bf16x8 *)(s_weights + (cb * G::FRAGS + (dx * K::KC + kc) * 3 + dy) * 1024 + lane * 16);
                w_of = it.b;
            }
            uint32_t voff[G::LOADS];
#pragma unroll
            for (int k = 0; k < G::LOADS; ++k) {
                const int sl = tid + k * G::THREADS, row = sl / G::ROW_SLOTS, rem = sl - row * G::ROW_SLOTS;
                const int col = rem / K::SPP, cpos = rem - col * K::SPP;
                const int y = it.y0 - 1 + row, x = it.colblk * kChainCols - 1 + col;
                const bool ok = sl < G::SLOTS && cpos < C / 8 && (uint32_t)y < (uint32_t)a.g.h && (uint32_t)x < (uint32_t)a.g.w;
                voff[k] = ok ? (uint32_t)((y * a.g.w + x) * (C * 2) + cpos * 16) : kOutside;
            }
            const bool there = wait_for(it.b - 1, it.n); // (if not, what follows is of no use, but within its bounds)
            // The rows, the records of the image, the other weights: in the order in which they are looked at (loads of a wavefront return
            // in order).
            const uint8_t *in = a.act[(it.b - 1) & 1] + (size_t)it.n * img_bytes;
#pragma unroll
            for (int k = 0; k < G::LOADS; ++k) load_lds16c(in, img_bytes, voff[k], lds + (k * WAVES + wave) * 1024);
            asm volatile("" ::: "memory");
            // (as ImageMeans; 32 channels: every wavefront all of them, 64: the first one, for all: the others see a buffer of no bytes)
            const bool reads = C == 32 || wave == 0;
            constexpr int LPR = C / 4, RPL = 64 / LPR, INF = 4; // lanes per record, records per load, loads in flight
            const int recs = it.b == 1 ? a.first.recs : a.mid.recs;
            const float *rec = a.rec[(it.b - 1) & 1] + (int64_t)it.n * recs * C;
            f32x4 v[INF];
            auto records = [&](int r0) {
#pragma unroll
                for (int u = 0; u < INF; ++u)
                    v[u] = __builtin_bit_cast(f32x4, load16c(rec, reads ? (uint32_t)recs * C * 4 : 0u, (uint32_t)(min(r0 + u * RPL + lane / LPR, recs - 1) * LPR + lane % LPR) * 16));
            };
            records(0);
            asm volatile("" ::: "memory");
            // What the correction of this wavefront's outputs needs: four outputs to a lane, eight lanes to an output with an eighth of the
            // input channels each.
            constexpr int CP = C / 8;
            const float *rsum = a.rsum + (size_t)(it.b - 1) * C * C + (lane >> 3) * CP * C + cb * 32 + 4 * (lane & 7);
            const f32x4 bias = *(const f32x4 *)(a.bias + it.b * C + cb * 32 + 4 * (lane & 7));
            f32x4 rs[CP];
#pragma unroll
            for (int k = 0; k < CP; ++k) rs[k] = *(const f32x4 *)(rsum + k * C);
            asm volatile("" ::: "memory");
#pragma unroll
            for (int dx = G::AHEAD; dx < 3; ++dx) {
                const bf16x8 *wp = (const bf16x8 *)(a.w_mid + (size_t)(it.b - 1) * 9 * C * C) + cb * 9 * K::KC * 64 + lane;
#pragma unroll
                for (int kc = 0; kc < K::KC; ++kc)
#pragma unroll
                    for (int dy = 0; dy < 3; ++dy) Wr[dy * 3 + dx][kc] = wp[((dy * 3 + dx) * K::KC + kc) * 64];
            }
            asm volatile("" ::: "memory");
            auto correct = [&](int ln) __attribute__((always_inline)) {
                f32x4 d = {0.f, 0.f, 0.f, 0.f};
                auto part = [&]() {
#pragma unroll
                    for (int k = 0; k < CP; ++k) {
                        const float mk = s_mean[C == 32 ? wave : 0][(ln >> 3) * CP + k];
#pragma unroll
                        for (int e = 0; e < 4; ++e) d[e] = fmaf(rs[k][e], mk, d[e]);
                    }
                };
                part();
                // FirstInit sums over parts of 64 / (C / 4): eighths at 32 channels, quarters at 64, the second half of each behind the first
                if (C == 64) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) d[e] = dpp_f<0x118, 0xf>(d[e]); // row_shr:8
                    part();
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) d[e] += dpp_f<0x128, 0xf>(d[e]); // row_ror:8
                }
#pragma unroll
                for (int sh = 16; sh < 64; sh <<= 1)
#pragma unroll
                    for (int e = 0; e < 4; ++e) d[e] += __shfl_xor(d[e], sh);
                if (ln >> 3 == (C == 64 ? 1 : 0)) *(f32x4 *)&s_init[wave][4 * (ln & 7)] = bias + d;
            };
            {
                f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int u = 0; u < INF; ++u) asm volatile("" : "+v"(v[u])); // the records are first looked at here
                auto add = [&](int r0) {
#pragma unroll
                    for (int u = 0; u < INF; ++u) {
                        const bool ok = r0 + u * RPL + lane / LPR < recs;
#pragma unroll
                        for (int e = 0; e < 4; ++e) sum[e] += ok ? v[u][e] : 0.f;
                    }
                };
                add(0);
#pragma unroll 1
                for (int r0 = INF * RPL; r0 < recs; r0 += INF * RPL) {
                    records(r0);
                    add(r0);
                }
#pragma unroll
                for (int sh = LPR; sh < 64; sh <<= 1)
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[e] += __shfl_xor(sum[e], sh);
                const float inv_cnt = it.b == 1 ? a.first.inv_cnt : a.mid.inv_cnt;
                if (reads && lane < LPR) *(f32x4 *)&s_mean[C == 32 ? wave : 0][4 * lane] = (f32x4){sum[0] * inv_cnt, sum[1] * inv_cnt, sum[2] * inv_cnt, sum[3] * inv_cnt};
            }
            lds_barrier(); // (the records have landed, and before them the rows)
            if (C == 64) correct(lane); // (no registers are left for what it needs while a product is formed)
            uint32_t next = 0;
            if (draws) next = draw();
            if (lds_of == it.b && it.b + 1 < a.blocks) weights_to_lds(it.b + 1);
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                const int ln = pin_in_loop(tid & 63), px = ln & 31, half = ln >> 5;
                const int row = (s * G::RG + rg) * RW; // the first of the wavefront's
                lrow_t rowp[RW + 2];
#pragma unroll
                for (int r = 0; r < RW + 2; ++r) rowp[r] = lds_address(lds) + (uint32_t)((row + r) * G::ROWB + px * K::PS + half * 16);
                f32x16 acc[RW];
                if constexpr (!G::HALVES) {
                    strip_mma<C, RW>(rowp, Wr, acc, kZeroAcc, []() {});
#pragma unroll
                    for (int r = 0; r < RW; ++r) asm volatile("" : "+v"(acc[r])); // (the products stay where they are)
                } else if (rg & 1) {
                    half_mma<C, true, RW>(rowp, Wr, acc);
                } else {
                    half_mma<C, false, RW>(rowp, Wr, acc);
                }
                if (C == 32 && s == 0) correct(ln);
                const int yw = it.y0 + row, strip = yw / kRows;
                const bool inside = strip < a.g.strips; // (the same for the whole wavefront)
                if (inside && !is_last(it.b)) store_rows(it, yw, acc);
                const bool sums = inside && leaves_sums(it.b, strip);
                if constexpr (!G::HALVES || G::ROWS == kRows) {
                    if (!sums) continue;
                } else { // (a barrier follows: the same for the whole workgroup, of whose strips one at least may be inside)
                    if (!leaves_sums(it.b, it.y0 / kRows) && !leaves_sums(it.b, it.y0 / kRows + 1)) continue;
                }
                float *handed = &s_handed[rg / 2 * K::NCB + cb][ln * 4];
                if constexpr (!G::HALVES) {
                    sum_rows(it, yw, acc, std::true_type{}, kNoSums);
                } else if constexpr (C == 32) {
                    if (rg & 1) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) *(f32x4 *)(handed + q * 256) = (f32x4){acc[0][4 * q], acc[0][4 * q + 1], acc[0][4 * q + 2], acc[0][4 * q + 3]};
                    }
                    lds_barrier();
                    if (!(rg & 1)) {
                        f32x16 pair[2] = {acc[0], {}};
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const f32x4 v = *(const f32x4 *)(handed + q * 256);
                            pair[1][4 * q] = v[0]; pair[1][4 * q + 1] = v[1]; pair[1][4 * q + 2] = v[2]; pair[1][4 * q + 3] = v[3];
                        }
                        sum_rows(it, yw, pair, std::true_type{}, kNoSums);
                    }
                } else {
                    float above[16];
                    if (sums && !(rg & 1)) {
                        column_sums<RW>(above, acc, &s_init[wave][half * 16], 0.f, true, yw, a.g.h);
#pragma unroll
                        for (int q = 0; q < 4; ++q) *(f32x4 *)(handed + q * 256) = (f32x4){above[4 * q], above[4 * q + 1], above[4 * q + 2], above[4 * q + 3]};
                    }
                    lds_barrier();
                    if (sums && !(rg & 1) && is_last(it.b)) sum_rows(it, yw, acc, std::false_type{}, kNoSums);
                    if (sums && (rg & 1)) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const f32x4 v = *(const f32x4 *)(handed + q * 256);
                            above[4 * q] = v[0]; above[4 * q + 1] = v[1]; above[4 * q + 2] = v[2]; above[4 * q + 3] = v[3];
                        }
                        sum_rows(it, yw, acc, std::true_type{}, above);
                    }
                }
            }
            done(it, next, there);
            it = next_item();
        } while (it.b > 0);
    };
#pragma unroll 1
    for (;;) {
        if (it.b == 0) first_block();
        else if (it.b > 0) later_blocks();
        else if (it.n >= 0) skip();
        else break;
    }
}

// The state of conv_chain_kernel's launch back to zeros, by a wavefront of the launch behind it: image n's counters, and for n = 0 what
// else there is.  Whether items of the image are missing; the host hears of it, too.
__device__ __forceinline__ bool clear_chain(const ChainState &c, int64_t n, int lane)
{
    if (!c.words) return false;
    bool missing = false;
    if (lane < c.blocks) {
        uint32_t *counter = c.words + kChainCountAt + ((size_t)lane * c.n_img + n) * kChainCount;
        missing = *counter != (lane == 0 ? c.first_items : c.items);
        *counter = 0u;
    }
    if (n == 0)
        for (int i = lane; i < kChainCountAt; i += 64) c.words[i] = 0u;
    const bool lost = __ballot(missing) != 0;
    if (lost && lane == 0 && c.lost) __hip_atomic_store(c.lost, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    return lost;
}

// ------------------------------------------------------------------------------------------------
// Head for the linear tail: the nine border-aware channel sums of the last block -> final conv + global
// average pool in closed form (fp32 weights) -> linear -> logits -> bits -> symbols.
//   pooled[o] = 1/(h w) * sum_{c,dy,dx} Wf[o][c][dy][dx] * S[c][dy][dx],
//   S[c][dy][dx] = sum of channel c over the input pixels that tap (dy,dx) reaches with zero padding
//                = whole - excluded row - excluded column + their corner
//   (dy = 0 never reaches the last row, dy = 2 never the first; same for dx and columns).
// Few images: an image's workgroup waits for its weights (147 KB to a compute unit at 64 channels and 64 outputs), so those of the
// final convolution and of the linear layer are asked for in 16-byte pieces before the lines of sums are read, and the tables of the
// code with them where the word is decoded here (head_decodes).  Many images: the weights come out of the L2s again and again; there
// kHeadShare images share a read.  Against a workgroup per image with 4-byte weight loads inside the sums: one tile of 32 x 32,
// 32 channels 31.1 -> 29.8 us a call; the launch over 1024 tiles of 64 x 64 20.4 -> 12.6 us, over 256 of 128 x 128, 96 bits
// 16.5 -> 12.2.
// ------------------------------------------------------------------------------------------------
// Sum of the 16-byte pieces p[r * stride], r = start, start + step, .. < count, four loads in flight.
__device__ __forceinline__ f32x4 sum_lines(const f32x4 *p, int stride, int start, int step, int count)
{
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int r0 = start; r0 < count; r0 += 4 * step) {
        f32x4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = p[(int64_t)min(r0 + u * step, count - 1) * stride];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] += r0 + u * step < count ? v[u][e] : 0.f;
    }
    return sum;
}

// The same over lines r that are kChunk lines each, one per row pair (of `pairs`): what the kernel
// would have added up before it wrote them, in its order.  width: lines of one row pair.
__device__ __forceinline__ f32x4 sum_line_groups(const f32x4 *p, int stride, int start, int step, int count, int width, int pairs)
{
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int r = start; r < count; r += step) {
        const int first = r / width * kChunk, b = r % width;
        f32x4 v[kChunk];
#pragma unroll
        for (int u = 0; u < kChunk; ++u) v[u] = p[(int64_t)(min(first + u, pairs - 1) * width + b) * stride];
#pragma unroll
        for (int u = 1; u < kChunk; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[0][e] += first + u < pairs ? v[u][e] : 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] += v[0][e];
    }
    return sum;
}

// The image's word from its bits (sbit), by 16 lanes, one symbol each; the errors (a chain of table look-ups) are found by all of them
// alike.  lost: there are no bits, and no word.
__device__ __forceinline__ void decode_image_word(const WordArgs &word, const uint8_t *tab, const uint8_t *sbit, int64_t img, int i, bool lost)
{
    const RsParams &p = word.rs;
    const int ord = p.q - 1;
    const bool mine = i < p.n;
    const Gf gf{tab, (const uint16_t *)(tab + kLogAt)};
    int sym = 0;
    for (int u = 0; u < p.m; ++u) sym |= mine ? (int)sbit[i * p.m + u] << (p.m - 1 - u) : 0;
    uint32_t S = mine ? ((const uint32_t *)(tab + kCodeAt))[i * p.q + sym] : 0u;
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) S ^= (uint32_t)__shfl_xor((int)S, off, 16);
    const LaneErrors err = lane_errors(gf, tab + kQuadAt, S, p.n, ord, p.two_t);
    if (err.ok && err.count > 0) {
        const int v1 = lane_error_value(gf, err.p1, err.a1, p.fcr, ord);
        if (i == p.n - 1 - err.p1) sym ^= v1;
        if (err.count == 2) {
            const int v2 = lane_error_value(gf, err.p2, err.a2, p.fcr, ord);
            if (i == p.n - 1 - err.p2) sym ^= v2;
        }
    }
    if (mine && word.cw) word.cw[img * p.n + i] = (uint8_t)sym;
    if (i < p.k) word.msg[img * p.k + i] = (uint8_t)sym;
    if (i == 0) word.nerr[img] = (int8_t)(err.ok && !lost ? err.count : -1);
    if (word.key.matches) {
        int agree = i < p.k ? p.m - __popc((uint32_t)(sym ^ word.key.key[i]) & (uint32_t)ord) : 0;
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) agree += __shfl_xor(agree, off, 16);
        if (i == 0) {
            word.key.matches[img] = lost ? 0 : agree;
            if (word.key.detected) word.key.detected[img] = (uint8_t)(!lost && agree >= word.key.tau);
        }
    }
}

// Linear layer of NB * 64 outputs (padded with zeros, as the weights' rows are): four lanes to an output, every fourth 16-byte
// piece of its row each.  The weights are asked for at the start of a launch (weights) and used at its end (of).
template <int NB>
struct Linear {
    f32x4 w[4 * NB];
    __device__ __forceinline__ void weights(const float *lin_w, int tid)
    {
        const float *row = lin_w + min(tid >> 2, 64 * NB - 1) * (64 * NB) + 4 * (tid & 3);
#pragma unroll
        for (int j = 0; j < 4 * NB; ++j) w[j] = *(const f32x4 *)(row + 16 * j);
    }
    __device__ __forceinline__ float of(const float *pooled, int tid) const // every lane of the four has the output
    {
        float z = 0.f;
#pragma unroll
        for (int j = 0; j < 4 * NB; ++j) {
            const f32x4 v = *(const f32x4 *)&pooled[16 * j + 4 * (tid & 3)];
#pragma unroll
            for (int e = 0; e < 4; ++e) z = fmaf(w[j][e], v[e], z);
        }
        z += __shfl_xor(z, 1);
        return z + __shfl_xor(z, 2);
    }
};

constexpr int kHeadWaves = 8;
constexpr int kHeadThreads = 64 * kHeadWaves;
// A workgroup per image while all of them are resident at once (two to a compute unit), else one per two images.  One / two images a
// workgroup, whole calls of 32 x 32, 32 channels: 300 tiles 89.7 / 90.6 us, 512 119.3 / 120.0, 1024 196.4 / 192.9, 16384 2959 / 2921.
// (Four: 94.2, 123.6, 195.6, 2910, but 1024 tiles of 64 x 64 14.8 us where two take 12.6.)
constexpr int64_t kHeadAlone = 512;
constexpr int kHeadShare = 2;

// NB = nbp / 64; IPB images to a workgroup
template <int C, int NB, int IPB>
__global__ __launch_bounds__(kHeadThreads, 4) void head_kernel(const float *__restrict__ recs, LastSums sums, int n_img, int n_bits,
                                                               float inv_hw, const float *__restrict__ wft /*[C*9][nbp]*/,
                                                               const float *__restrict__ fbias, const float *__restrict__ lin_w,
                                                               const float *__restrict__ lin_b, float *__restrict__ logits,
                                                               uint8_t *__restrict__ bits, uint8_t *__restrict__ symbols, int m,
                                                               WordArgs word, ChainState chain)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t s_tab[];  // tables of the code, if the words are decoded here
    __shared__ __attribute__((aligned(16))) float Q[IPB][9 * C];     // an image's sums, [q*C + c]
    __shared__ __attribute__((aligned(16))) float Qp[IPB][4 * C];    // partial sums over the whole-tile lines
    __shared__ float S[IPB][9 * C];                                  // [c*9 + tap]
    __shared__ __attribute__((aligned(16))) float part[kHeadWaves][IPB][64 * NB];
    __shared__ __attribute__((aligned(16))) float pooled[IPB][64 * NB];
    __shared__ uint8_t sbit[IPB][64 * NB];
    __shared__ bool s_lost; // (IPB 1)
    // (128 registers, no scratch: 64 outputs of 64 channels fit with the wavefront's number in a scalar, 128 of 32 channels without)
    const int tid = threadIdx.x, wave = NB == 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6, lane = tid & 63;
    const int64_t img0 = (int64_t)blockIdx.x * IPB;
    // final conv + pool: LPO lanes share the outputs of a k = (channel, tap), four each; a part of KLEN of them
    constexpr int nbp = 64 * NB, LPO = nbp / 4, KLEN = C * 9 * LPO / kHeadThreads, PRE = IPB > 1 ? 0 : NB == 2 ? 12 : KLEN;
    const int ol = tid % LPO, k0 = tid / LPO * KLEN;
    const f32x4 *wf = (const f32x4 *)wft + (int64_t)k0 * LPO + ol;
    f32x4 wv[PRE ? PRE : 1];
#pragma unroll
    for (int j = 0; j < PRE; ++j) wv[j] = wf[j * LPO];
    Linear<NB> linear;
    if (IPB == 1) linear.weights(lin_w, tid);
    if (word.rs.tab) { // needed last: in flight meanwhile
        for (int i = tid * 16; i < word.rs.tab_bytes; i += kHeadThreads * 16)
            __builtin_amdgcn_global_load_lds((gptr_t)(word.rs.tab + i), (lptr_t)(s_tab + (i & ~1023)), 16, 0, 0);
    }
#pragma unroll 1
    for (int i = 0; i < IPB; ++i) {
        // lines -> Q: wavefronts 0 .. 3 the whole-tile lines, 4 and 5 the columns, 6 the rows, 7 the corners; 16 bytes per
        // lane, i.e. 256 / C lines per load and four loads in flight
        constexpr int LPL = C / 4, LPW = 64 / LPL; // lanes per line, lines per wavefront-wide load
        const int l = lane % LPL, sub = lane / LPL;
        const f32x4 *p = (const f32x4 *)recs + min(img0 + i, (int64_t)n_img - 1) * (sums.stride ? sums.stride : sums.lines * LPL) + l;
        auto total = [&](int first, int count, int start, int step, float *dst, int pair_lines = 0) { // pair_lines: lines per row pair, if they are
            f32x4 v;
            if (sums.pairs && pair_lines)
                v = sum_line_groups(p + first * LPL, LPL, start, step, (sums.pairs + kChunk - 1) / kChunk * pair_lines, pair_lines, sums.pairs);
            else v = sum_lines(p + first * LPL, LPL, start, step, count);
#pragma unroll
            for (int sh = LPL; sh < 64; sh <<= 1)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] += __shfl_xor(v[e], sh);
            if (sub == 0) *(f32x4 *)(dst + 4 * l) = v;
        };
        if (wave < 4) total(0, sums.first_col, wave * LPW + sub, 4 * LPW, &Qp[i][wave * C], 2);
        else if (wave == 4) total(sums.first_col, sums.last_col - sums.first_col, sub, LPW, &Q[i][3 * C], 1);
        else if (wave == 5) total(sums.last_col, sums.rows - sums.last_col, sub, LPW, &Q[i][4 * C], 1);
        else if (wave == 6) {
            const int half = (sums.corners - sums.rows) / 2;
            total(sums.rows, half, sub, LPW, &Q[i][1 * C]);
            total(sums.rows + half, half, sub, LPW, &Q[i][2 * C]);
        } else {
            if (sub < 4) *(f32x4 *)&Q[i][(5 + sub) * C + 4 * l] = p[(sums.corners + sub) * LPL];
            if (IPB == 1) { // (this wavefront has the least to do)
                const bool lost = clear_chain(chain, img0, lane);
                if (lane == 0) s_lost = lost;
            }
        }
    }
    __syncthreads();
    if (tid < IPB * C) {
        const int i = tid / C, c = tid % C;
        float T = (Qp[i][c] + Qp[i][C + c]) + (Qp[i][2 * C + c] + Qp[i][3 * C + c]), R0 = Q[i][1 * C + c], Rl = Q[i][2 * C + c];
        const float C0 = Q[i][3 * C + c], Cl = Q[i][4 * C + c];
        const float c00 = Q[i][5 * C + c], c0l = Q[i][6 * C + c], cl0 = Q[i][7 * C + c], cll = Q[i][8 * C + c];
        if (sums.seam) { // the last column was computed apart: it is not in the whole-tile and row lines yet
            T += Cl;
            R0 += c0l;
            Rl += cll;
        }
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
                const float rex = dy == 0 ? Rl : (dy == 2 ? R0 : 0.f);
                const float cex = dx == 0 ? Cl : (dx == 2 ? C0 : 0.f);
                float corner = 0.f;
                if (dy == 0 && dx == 0) corner = cll;
                if (dy == 0 && dx == 2) corner = cl0;
                if (dy == 2 && dx == 0) corner = c0l;
                if (dy == 2 && dx == 2) corner = c00;
                S[i][c * 9 + dy * 3 + dx] = T - rex - cex + corner;
            }
    }
    __syncthreads();
    {
        f32x4 acc[IPB];
#pragma unroll
        for (int i = 0; i < IPB; ++i) acc[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
        auto add = [&](f32x4 w4, int j) {
#pragma unroll
            for (int i = 0; i < IPB; ++i) {
                const float v = S[i][k0 + j];
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i][e] = fmaf(w4[e], v, acc[i][e]);
            }
        };
#pragma unroll
        for (int j = 0; j < PRE; ++j) add(wv[j], j);
        if (KLEN > PRE) {
#pragma unroll 9
            for (int j = PRE; j < KLEN; ++j) add(wf[j * LPO], j);
        }
        if (IPB > 1) linear.weights(lin_w, tid);
#pragma unroll
        for (int i = 0; i < IPB; ++i) {
#pragma unroll
            for (int sh = LPO; sh < 64; sh <<= 1)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i][e] += __shfl_xor(acc[i][e], sh);
            if (lane < LPO) *(f32x4 *)&part[wave][i][4 * ol] = acc[i];
        }
    }
    __syncthreads();
    if (tid < IPB * nbp) {
        const int i = tid / nbp, o = tid % nbp;
        float v = 0.f;
#pragma unroll
        for (int kp = 0; kp < kHeadWaves; ++kp) v += part[kp][i][o];
        if (IPB == 1 && s_lost) v = __builtin_nanf(""); // (and so is every logit)
        pooled[i][o] = o < n_bits ? v * inv_hw + (fbias ? fbias[o] : 0.f) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < IPB; ++i) {
        float z = linear.of(pooled[i], tid);
        const int o = tid >> 2;
        if (o < n_bits && (tid & 3) == 0) {
            if (lin_b) z += lin_b[o];
            const uint8_t bt = z > 0.f ? 1 : 0;
            sbit[i][o] = bt;
            if (img0 + i < n_img) {
                if (logits) logits[(img0 + i) * n_bits + o] = z;
                if (bits) bits[(img0 + i) * n_bits + o] = bt;
            }
        }
    }
    __syncthreads();
    if (symbols) {
        const int nsym = n_bits / m;
        for (int idx = tid; idx < IPB * nsym; idx += kHeadThreads) {
            const int i = idx / nsym, j = idx - i * nsym;
            int sym = 0;
            for (int u = 0; u < m; ++u) sym |= (int)sbit[i][j * m + u] << (m - 1 - u);
            if (img0 + i < n_img) symbols[(img0 + i) * nsym + j] = (uint8_t)sym;
        }
    }
    if (word.rs.tab && tid < 16 * IPB && img0 + tid / 16 < n_img)
        decode_image_word(word, s_tab, sbit[tid / 16], img0 + tid / 16, tid % 16, IPB == 1 && s_lost);
}

// ------------------------------------------------------------------------------------------------
// pooled -> linear -> logits -> bits -> symbols.  One block per image; its threads share the lines of sums of the image
// (16 bytes each, four loads in flight).
// ------------------------------------------------------------------------------------------------
template <int NB>
__global__ __launch_bounds__(kHeadThreads) void linear_pack_kernel(const float *__restrict__ partial, int lines, int n_bits,
                                                                   float inv_hw, const float *__restrict__ fbias,
                                                                   const float *__restrict__ lin_w,
                                                                   const float *__restrict__ lin_b, float *__restrict__ logits,
                                                                   uint8_t *__restrict__ bits, uint8_t *__restrict__ symbols,
                                                                   int m, ChainState chain)
{
    constexpr int nbp = 64 * NB, lpl = nbp / 4, groups = kHeadThreads / lpl; // lanes per line
    __shared__ __attribute__((aligned(16))) float part[kHeadThreads * 4];
    __shared__ __attribute__((aligned(16))) float pooled[nbp];
    __shared__ uint8_t sbit[nbp];
    __shared__ bool s_lost;
    const int64_t n = blockIdx.x;
    const int tid = threadIdx.x, o = tid;
    Linear<NB> linear;
    linear.weights(lin_w, tid);
    *(f32x4 *)&part[tid * 4] = sum_lines((const f32x4 *)partial + n * lines * lpl + tid % lpl, lpl, tid / lpl, groups, lines);
    if (tid < 64) {
        const bool lost = clear_chain(chain, n, tid);
        if (tid == 0) s_lost = lost;
    }
    __syncthreads();
    if (o < nbp) {
        float s = 0.f;
#pragma unroll
        for (int g2 = 0; g2 < groups; ++g2) s += part[g2 * nbp + o];
        if (s_lost) s = __builtin_nanf(""); // (and so is every logit)
        pooled[o] = o < n_bits ? s * inv_hw + (fbias ? fbias[o] : 0.f) : 0.f;
    }
    __syncthreads();
    {
        float z = linear.of(pooled, tid);
        const int out = tid >> 2;
        if (out < n_bits && (tid & 3) == 0) {
            if (lin_b) z += lin_b[out];
            const uint8_t b = z > 0.f ? 1 : 0;
            if (logits) logits[n * n_bits + out] = z;
            if (bits) bits[n * n_bits + out] = b;
            sbit[out] = b;
        }
    }
    __syncthreads();
    if (symbols && o < n_bits / m) {
        int sym = 0;
        for (int u = 0; u < m; ++u) sym |= (int)sbit[o * m + u] << (m - 1 - u);
        symbols[n * (n_bits / m) + o] = (uint8_t)sym;
    }
}

__global__ __launch_bounds__(256) void clear_chain_kernel(uint32_t *state)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < kChainStateBytes / 4; i += (size_t)gridDim.x * 256) state[i] = 0u;
}

__global__ __launch_bounds__(256) void nhwc_to_nchw_kernel(const bf16_t *__restrict__ in, int64_t total, int hw, int C,
                                                           float *__restrict__ out, ChainState chain)
{
    if (blockIdx.x == 0 && threadIdx.x < 64)
        for (int n = 0; n < chain.n_img; ++n) clear_chain(chain, n, threadIdx.x);
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
        const int c = (int)(i % C);
        const int64_t p = i / C; // n*hw + pixel
        const int64_t n = p / hw;
        const int pix = (int)(p % hw);
        out[(n * C + c) * hw + pix] = (float)in[i];
    }
}

} // namespace

// What the consumer of a launch's sampled channel sums has to know: records per image and pixels behind them.
// `cols`: output columns the launch covers; `pieces`: records per sampled strip and column block.
static MeanIn sampled_strips(const ConvGeom &g, int cols, int pieces)
{
    const int first = sampled_strip(g.strips), count = (g.strips - 1 - first) / 8 + 1, last = first + 8 * (count - 1);
    const int rows = (count - 1) * kRows + std::min(kRows, g.h - last * kRows);
    return MeanIn{nullptr, count * g.colblks * pieces, 1.0f / ((float)rows * (float)cols)};
}

static int chain_most_rows(int C) { return C == 64 ? 16 : 32; }

MeanIn conv_first_samples(const ConvGeom &g, int C) { return sampled_strips(g, g.w, 4 / (C / 32)); }

MeanIn conv_mid_samples(const ConvGeom &g, int C) { return sampled_strips(g, g.w, 2 * (2 / (C / 32))); }

MeanIn conv_pair_samples(const ConvGeom &g)
{
    // two row pairs per strip, unless the last sampled strip is the tile's last one and has one row pair only; a wide
    // tile's last column belongs to conv_seam_kernel, which takes no samples
    const bool seam_column = g.colblks > 1 && g.w % kTileW == 0;
    MeanIn m = sampled_strips(g, g.w - (seam_column ? 1 : 0), 4);
    const int pairs = (g.h + 1) / 2;
    const bool last_sampled = ((g.strips - 1) & 7) == sampled_strip(g.strips);
    if (last_sampled && (pairs & 1)) m.recs -= 2 * g.colblks;
    return m;
}

hipError_t launch_conv_first(const TileSrc &src, const ConvGeom &g, int C, const bf16_t *wfrag, const float *bias,
                             float *tout, const Partition &part, bf16_t *out, hipStream_t s)
{
    const int recs = conv_first_samples(g, C).recs;
    if (C == 64)
        hipLaunchKernelGGL(conv_first_kernel<64>, dim3(part.blocks), dim3(256), 0, s, src, g, wfrag, bias, tout, recs, part.per, out);
    else
        hipLaunchKernelGGL(conv_first_kernel<32>, dim3(part.blocks), dim3(256), 0, s, src, g, wfrag, bias, tout, recs, part.per, out);
    return hipGetLastError();
}

// (the same places in conv_mid_kernel's epilogue)
LastSums conv_mid_last_sums(const ConvGeom &g, int C)
{
    const int row_groups = 2 / (C / 32);
    LastSums l{};
    l.first_col = g.strips * g.colblks * 2 * row_groups;
    l.last_col = l.first_col + g.strips * row_groups;
    l.rows = l.last_col + g.strips * row_groups;
    l.corners = l.rows + 4 * g.colblks;
    l.lines = l.corners + 4;
    return l;
}

int conv_final_lines(const ConvGeom &g) { return g.strips * g.colblks * 2; }

hipError_t launch_conv_mid(const uint8_t *in, const ConvGeom &g, int C, const bf16_t *wfrag,
                           const float *bias, const MeanIn &tin, const float *rsum, float *tout,
                           const Partition &part, bool last, bf16_t *out, hipStream_t s)
{
    StatArgs st{tin, rsum, tout, last ? conv_mid_last_sums(g, C).lines : conv_mid_samples(g, C).recs, part.per, 0.f};
    const dim3 grid(part.blocks), block(64 * kMidWaves);
    if (C == 64) {
        if (last) hipLaunchKernelGGL((conv_mid_kernel<64, MODE_LAST>), grid, block, 0, s, in, g, wfrag, bias, st, out);
        else hipLaunchKernelGGL((conv_mid_kernel<64, MODE_MID>), grid, block, 0, s, in, g, wfrag, bias, st, out);
    } else {
        if (last) hipLaunchKernelGGL((conv_mid_kernel<32, MODE_LAST>), grid, block, 0, s, in, g, wfrag, bias, st, out);
        else hipLaunchKernelGGL((conv_mid_kernel<32, MODE_MID>), grid, block, 0, s, in, g, wfrag, bias, st, out);
    }
    return hipGetLastError();
}

bool conv_pair_supported(int C, const ConvGeom &g) { return C == 64 && g.colblks >= 1; }

// Whether the last pair leaves a line per row pair instead of one per kChunk of them: where the longest workgroup's run of row
// pairs gets shorter for it, in launches whose chunks do not reach every compute unit, as long as an image's lines fit the place of
// its activations (64 channels, two bytes a pixel): on tiles of up to four columns they do not, and with a block of their own for
// them a batch of 24 tiles of 64 x 4 took a workspace half as large again as one of 25.
// Such a launch deals in runs: whole images cost the same in pieces of one row pair and of kChunk, and no split costs more.
static bool fine_lines(const ConvGeom &g, int num_cu)
{
    const int pairs = (g.h + 1) / 2, chunks = (pairs + kChunk - 1) / kChunk;
    if (g.colblks > 1 || (int64_t)g.n_img * chunks >= num_cu) return false;
    if ((int64_t)(4 * pairs + 8) * 4 > (int64_t)g.h * g.w * 2) return false; // (4 pairs + 8 lines: conv_pair_last_sums)
    return conv_pair_split(g, false, num_cu).cost < conv_pair_split(g, true, num_cu).cost;
}

LastSums conv_pair_last_sums(const ConvGeom &g, int num_cu)
{
    const bool fine = fine_lines(g, num_cu);
    const int pairs = (g.h + 1) / 2, chunks = fine ? pairs : (pairs + kChunk - 1) / kChunk;
    LastSums l{};
    l.pairs = fine ? pairs : 0;
    l.seam = g.colblks > 1 && g.w % kTileW == 0;
    l.first_col = chunks * 2 * g.colblks;
    l.last_col = l.first_col + chunks;
    l.rows = l.last_col + (l.seam ? (g.h + 31) / 32 : chunks); // (conv_seam_kernel: a line per 32 rows)
    l.corners = l.rows + 4 * g.colblks;
    l.lines = l.corners + 4;
    return l;
}

size_t conv_pair_seam_bytes(const ConvGeom &g, int num_cu)
{
    if (g.colblks <= 1) return 0;
    const size_t half = (size_t)(2 * ((g.h + 1) / 2)) * kSeamRowBytes;
    return half * (2 * (size_t)num_cu + (g.w % kTileW == 0 ? (size_t)g.n_img : 0));
}

// What the longest workgroup has to do when a launch's pieces of `quant` row pairs are dealt in runs of `per`: eight for each
// of its steps (positions of the kernel's stream and two to drain), one for each row pair that either group multiplies in them.
static int pair_cost(const ConvGeom &g, int quant, int per)
{
    const int S = (g.h + 1) / 2, ppi = (S + quant - 1) / quant;
    const int64_t pieces = (int64_t)g.n_img * ppi, runs = (pieces + per - 1) / per;
    int longest = 0;
    for (int64_t v = 0; v < std::min<int64_t>(runs, ppi); ++v) { // (where a run begins in its image repeats after ppi runs)
        const int64_t q0 = v * per, q1 = std::min(pieces, q0 + per);
        const int images = (int)((q1 - 1) / ppi - q0 / ppi) + 1;
        const int ja = (int)(q0 % ppi) * quant, jb = std::min(S, (int)((q1 - 1) % ppi + 1) * quant);
        const int own = images * S - ja - (S - jb);   // row pairs of the run, per column block
        const int halo = (ja > 0) + (jb < S);         // computed by the first group only
        longest = std::max(longest, (8 * (own + halo + images) + 2 * own + halo) * g.colblks + 16);
    }
    return longest;
}

// Whole images per workgroup, or every compute unit one run of the launch's row pairs.  A run that begins and ends inside
// images has up to two halo pairs and an opening position more than its row pairs, and its code has more scalar
// instructions a step: runs where the longest workgroup gets shorter by more than 3 %.  Short launches are bound by the
// steps' latency, which is why a step counts for more than the matrix work in it (of 101 shapes from 40 x 5 x 64 to
// 1053 x 46 x 48, up to 200 columns, the rule picks the slower way by 1.7 % at most).  Eight blocks, whole images / runs, cost of a
// middle pair: 192 tiles of 8 x 64 80 / 85 us (64 / 80), 224 of 16 x 64 123 / 129 (104 / 120), 245 of 64 x 64 411 / 424 (344 / 360), 480
// of 64 x 64 807 / 809 (672 / 658), 240 of 128 x 128 1647 / 1655 (1312 / 1284); 40 of 5 x 64 58 / 51 (54 / 52), 160 of 16 x 64 113 / 110
// (104 / 100), 333 of 16 x 64 191 / 177 (192 / 168), 300 of 64 x 64 634 / 502 (672 / 438), 200 of 128 x 128 1523 / 1413 (1312 / 1084).
PairSplit conv_pair_split(const ConvGeom &g, bool last, int num_cu)
{
    const int quant = last ? kChunk : 1;
    const int ppi = ((g.h + 1) / 2 + quant - 1) / quant;
    const int64_t pieces = (int64_t)g.n_img * ppi;
    const int whole = (g.n_img + num_cu - 1) / num_cu * ppi, run = (int)((pieces + num_cu - 1) / num_cu);
    const int whole_cost = pair_cost(g, quant, whole), run_cost = pair_cost(g, quant, run);
    PairSplit p{};
    p.part = (int64_t)103 * run_cost < (int64_t)100 * whole_cost;
    p.per = p.part ? run : whole;
    p.cost = p.part ? run_cost : whole_cost;
    p.workgroups = (int)((pieces + p.per - 1) / p.per);
    return p;
}

// Microseconds of eight blocks on tiles of more than one column block, either schedule.  Single blocks: a launch deals strips
// evenly, its workgroups pay for each strip, for the extra rows a column of strips begins with, and for the activations of
// every block; fused: a run's halo and opening positions (pair_cost), a launch for the last column of widths that are multiples
// of 64, half the activations.  Fitted to 231 shapes of 128 .. 700 tiles, 4 .. 44 rows, 66 .. 256 columns with fewer than 12 row
// pairs per compute unit, as the kernels were at commit eefb1c9 (standard deviation 3.5 and 2.6 %).  The present kernels take 5 %
// (single blocks) and 7 % (fused) less than that, standard deviation 4 and 6: on 215 such shapes the way taken is the faster one or within 3 %
// of it on 203, at worst 7.5 % slower, and then mostly single blocks, which are also the more exact (wide_tiles_fused): the line stays.
// Measured, single / fused: 256 tiles of 8 x 100 186 / 138 us, 256 of 20 x 200 584 / 528, 200 of 30 x 200 705 / 661, 128 of 24 x 66 196 /
// 194; 292 of 5 x 73, single blocks by the rule, 173 / 161; 181 of 27 x 152, fused by the rule, 433 / 454.
WideCost conv_wide_cost(const ConvGeom &g, int num_cu)
{
    const int64_t strips = (int64_t)g.n_img * g.strips * g.colblks;
    const double per = (double)((strips + num_cu - 1) / num_cu), mpx = 1e-6 * g.n_img * g.h * g.w;
    WideCost c{};
    c.single_us = 66.2 + 16.1 * per + 6.8 * per / g.strips + 174.0 * mpx;
    c.fused_us = 31.5 + 0.218 * (3 * conv_pair_split(g, false, num_cu).cost + conv_pair_split(g, true, num_cu).cost) +
                 (g.w % kTileW == 0 ? 14.5 : 0.0) + 71.6 * mpx;
    return c;
}

template <bool FIRST, bool LASTB, bool PART, int QUANT>
static void launch_pair_variant(bool wide, dim3 grid, hipStream_t s, const uint8_t *in, const TileSrc &src,
                                const ConvGeom &g, const bf16_t *wfrag_a, const bf16_t *wfrag_b, const float *bias_a,
                                const float *bias_b, const PairArgs &st, bf16_t *out)
{
    if constexpr (!LASTB || QUANT == kChunk) { // (wide tiles leave chunks: fine_lines)
        if (wide) {
            hipLaunchKernelGGL((conv_pair_kernel<64, FIRST, LASTB, true, PART, QUANT>), grid, dim3(512), 0, s, in, src, g, wfrag_a, wfrag_b, bias_a, bias_b, st, out);
            return;
        }
    }
    hipLaunchKernelGGL((conv_pair_kernel<64, FIRST, LASTB, false, PART, QUANT>), grid, dim3(512), 0, s, in, src, g, wfrag_a, wfrag_b, bias_a, bias_b, st, out);
}

hipError_t launch_conv_pair(const uint8_t *in, const TileSrc *first, const ConvGeom &g, int C,
                            const bf16_t *wfrag_a, const bf16_t *wfrag_b, const float *bias_a, const float *bias_b,
                            const MeanIn &tin, const float *rsum_a, float *tout, bool last, int num_cu,
                            uint8_t *seam, bf16_t *out, hipStream_t s)
{
    if (!conv_pair_supported(C, g)) return hipErrorInvalidValue;
    const bool wide = g.colblks > 1;
    const bool seam_column = wide && g.w % kTileW == 0;
    if (wide && !seam) return hipErrorInvalidValue;
    const LastSums sums = conv_pair_last_sums(g, num_cu);
    const bool fine = last && sums.pairs;
    const PairSplit split = conv_pair_split(g, last && !fine, num_cu);
    const dim3 grid((unsigned)split.workgroups);
    if ((int)grid.x > num_cu) return hipErrorInvalidValue; // the seam buffer holds num_cu workgroups
    if (fine && !split.part) return hipErrorInvalidValue;
    const size_t half = (size_t)(2 * ((g.h + 1) / 2)) * kSeamRowBytes;
    uint8_t *seam_last = seam_column ? seam + 2 * (size_t)num_cu * half : nullptr;
    const int out_recs = last ? sums.lines : conv_pair_samples(g).recs;
    PairArgs st{tin, rsum_a, tout, out_recs, split.per, sums.rows, seam, seam_last};
    const TileSrc src = first ? *first : TileSrc{};
    auto launch = [&](auto part) {
        constexpr bool PART = decltype(part)::value;
        auto of = [&](auto is_first) {
            constexpr bool FIRST = decltype(is_first)::value;
            if constexpr (PART) { // (whole images never leave a line per row pair: fine_lines)
                if (fine) {
                    launch_pair_variant<FIRST, true, PART, 1>(wide, grid, s, in, src, g, wfrag_a, wfrag_b, bias_a, bias_b, st, out);
                    return;
                }
            }
            if (last) launch_pair_variant<FIRST, true, PART, kChunk>(wide, grid, s, in, src, g, wfrag_a, wfrag_b, bias_a, bias_b, st, out);
            else launch_pair_variant<FIRST, false, PART, 1>(wide, grid, s, in, src, g, wfrag_a, wfrag_b, bias_a, bias_b, st, out);
        };
        if (first) of(std::true_type{});
        else of(std::false_type{});
    };
    if (split.part) launch(std::true_type{});
    else launch(std::false_type{});
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !seam_column) return e;
    const dim3 sgrid((unsigned)g.n_img * (unsigned)((g.h + 31) / 32));
    if (last) hipLaunchKernelGGL((conv_seam_kernel<64, true>), sgrid, dim3(128), 0, s, seam_last, g, wfrag_b, bias_b, tout, out_recs, sums, out);
    else hipLaunchKernelGGL((conv_seam_kernel<64, false>), sgrid, dim3(128), 0, s, seam_last, g, wfrag_b, bias_b, tout, out_recs, sums, out);
    return hipGetLastError();
}

// The word of an image in the head's launch or in one of its own behind it: a launch costs 4 us and the gap before it, the tables that
// every workgroup of the head then reads (14 KB for RS(12,8) over GF(256)) cost little by little.  Whole calls of 32 x 32, 32
// channels, own launch / with the head: 1 tile 34.4 / 30.7 us, 16 35.7 / 31.8, 512 125.3 / 120.3, 2048 386.8 / 382.1, 4096
// 753.2 / 753.1, 8192 1474 / 1477.
constexpr int64_t kHeadWords = 2048;
bool head_decodes(const RsParams &p, int64_t N) { return lane_code(p.n, p.two_t) && N <= kHeadWords; }

hipError_t launch_head(const float *recs, const LastSums &sums, int C, int64_t n_img, int n_bits, int nbp, float inv_hw,
                       const float *wft, const float *fbias, const float *lin_w, const float *lin_b, float *logits,
                       uint8_t *bits, uint8_t *symbols, int m, const WordArgs &word, const ChainState &chain, hipStream_t s)
{
    if (n_img <= 0) return hipSuccess;
    if (chain.words && n_img > kHeadAlone) return hipErrorInvalidValue; // (a workgroup per image clears it)
    const unsigned tables = word.rs.tab ? (unsigned)((word.rs.tab_bytes + 1023) / 1024 * 1024) : 0u;
    auto launch = [&](auto kernel, int per) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)((n_img + per - 1) / per)), dim3(kHeadThreads), tables, s, recs, sums, (int)n_img, n_bits,
                           inv_hw, wft, fbias, lin_w, lin_b, logits, bits, symbols, m, word, chain);
    };
    auto of = [&](auto c) {
        constexpr int CH = decltype(c)::value;
        if (n_img <= kHeadAlone) launch(nbp == 64 ? head_kernel<CH, 1, 1> : head_kernel<CH, 2, 1>, 1);
        else launch(nbp == 64 ? head_kernel<CH, 1, kHeadShare> : head_kernel<CH, 2, kHeadShare>, kHeadShare);
    };
    if (C == 64) of(std::integral_constant<int, 64>{});
    else of(std::integral_constant<int, 32>{});
    return hipGetLastError();
}

// Strips are dealt to workgroups in contiguous runs of `per` that begin and end anywhere.  (Runs that divide an image, or
// are whole images, left workgroups without work: 16 tiles of 75 x 100, 38 strips each, went to 32 of 256 compute units.)
Partition make_partition(int64_t n_img, int tiles_per_image, int target_blocks)
{
    Partition p{};
    const int64_t total = n_img * tiles_per_image;
    p.per = (int)std::max<int64_t>(1, (total + target_blocks - 1) / target_blocks);
    p.blocks = (int)((total + p.per - 1) / p.per);
    return p;
}

Partition conv_final_partition(int64_t n_img, int tiles_per_image, int num_cu, int C, int nbp)
{
    return make_partition(n_img, tiles_per_image, std::max(1, num_cu * (C == 64 ? 1 : 2) / (nbp / 64))); // (two to a compute unit)
}

hipError_t launch_conv_final(const uint8_t *in, const ConvGeom &g, int C, int nbp, const bf16_t *wfrag,
                             const float *bias, int relu, float *partial, const Partition &part, hipStream_t s)
{
    StatArgs st{MeanIn{}, nullptr, partial, conv_final_lines(g), part.per, relu ? 0.f : __builtin_nanf("")};
    const dim3 grid(part.blocks, nbp / 64);
    if (C == 64) hipLaunchKernelGGL((conv_mid_kernel<64, MODE_FINAL>), grid, dim3(64 * kMidWaves), 0, s, in, g, wfrag, bias, st, nullptr);
    else hipLaunchKernelGGL(conv_final32_kernel, grid, dim3(256), 0, s, in, g, wfrag, bias, st);
    return hipGetLastError();
}

hipError_t launch_linear_pack(const float *partial, int lines, int nbp, int64_t n_img, int n_bits, float inv_hw,
                              const float *fbias, const float *lin_w, const float *lin_b, float *logits,
                              uint8_t *bits, uint8_t *symbols, int m, const ChainState &chain, hipStream_t s)
{
    if (n_img <= 0) return hipSuccess;
    hipLaunchKernelGGL(nbp == 64 ? linear_pack_kernel<1> : linear_pack_kernel<2>, dim3((unsigned)n_img), dim3(kHeadThreads), 0, s, partial,
                       lines, n_bits, inv_hw, fbias, lin_w, lin_b, logits, bits, symbols, m, chain);
    return hipGetLastError();
}

// The rows of an item: few enough that every compute unit of an XCD gets one if there are as many.
ChainPlan conv_chain_plan(const ConvGeom &g, int C, int blocks, int num_cu)
{
    ChainPlan p{};
    const int cu = std::max(1, num_cu / kChainTeams), colblks = (g.w + kChainCols - 1) / kChainCols;
    p.chunk = (g.n_img + kChainTeams - 1) / kChainTeams;
    for (p.rows = kRows;; p.rows *= 2) {
        p.items = (int64_t)p.chunk * ((g.h + p.rows - 1) / p.rows) * colblks;
        if (p.rows == chain_most_rows(C) || p.items <= cu) break;
    }
    p.fits = blocks >= 2 && blocks <= 64 /* lanes of clear_chain */ && (int64_t)g.n_img * blocks <= kChainCounters && g.n_img <= kHeadAlone && p.items * blocks < (1 << 24) &&
             (int64_t)conv_chain_last_sums(g, C).lines * C * 4 <= (int64_t)g.h * g.w * C * 2;
    p.one_round = p.items <= cu;
    return p;
}

// Items to a compute unit of an XCD, at most (conv_chain_faster).
static int chain_rounds(int C) { return C == 32 ? 5 : 1; }

// Whether all blocks in one launch are the faster way.  As long as every compute unit of an XCD has one item at most, an item takes
// what its rows take, while a launch per block has two round trips to memory, its weights and one strip behind the other.  With more
// items it is the faster way at 32 channels where a tile of up to 32 columns is one item wide and half of a strip of 64.
//   By estimates in microseconds, fitted to whole calls of two to nine blocks, 1 .. 512 tiles of 8 x 8 to 256 x 256: 724 shapes with
// one item at most and 484 with up to five at 32 channels, 600 at 64; standard deviation 2 .. 5 % and, for more than one item, 6 .. 9 %, where the
// single blocks have to look 9 % slower (with 5 %, five of 75 calls taken were slower so, one by 10 %).  Of 534, 166 and 300 other
// shapes 179, 40 and 66 are taken, 1.19, 1.26 and 1.07 times as fast in the mean (up to 1.6); one is slower by more than 2 % (37 tiles of 57 x 72, three
// blocks, 3.5 %); of the others the chain would be faster by 1.21 at most.  The number of blocks matters: fitted to four and eight alone, the rule
// took calls of two and three that are 1.1 and 1.0 .. 1.25 times as long this way.
// Other ways / chain, us: 16 tiles of 32 x 32, 32 channels, four blocks 25.1 / 24.3, 256 of them 71.6 / 49.2; 390 of 29 x 12 90.3 / 66.7; 7 of
// 128 x 128, 64 channels, eight blocks 110.7 / 105.7.  Not by the rule: 2 of 128 x 128, 32 channels 26.2 / 35.1; 4 of 128 x 128, 64 channels
// 86.8 / 105.8 (an XCD has one image or none).  Narrow tiles at 64 channels have the fused pairs (one of 64 x 64 49.1 / 61.2, four 50.1 / 64.1).
bool conv_chain_faster(const ConvGeom &g, int C, const ChainPlan &p, int blocks, int num_cu)
{
    if ((C == 64 && g.w <= kTileW) || p.items > (int64_t)chain_rounds(C) * std::max(1, num_cu / kChainTeams)) return false;
    const double per = (double)(((int64_t)g.n_img * g.strips * g.colblks + num_cu - 1) / num_cu), mpx = 1e-6 * g.n_img * g.h * g.w;
    const double chunk_mpx = 1e-6 * p.chunk * g.h * g.w, later = blocks - 1, items = (double)p.items;
    if (C == 64) {
        const double item_us = p.rows == 4 ? 6.25 : p.rows == 8 ? 7.25 : 10.2;
        return 16.2 + later * (item_us + 70.0 * chunk_mpx) + 525.0 * chunk_mpx < 0.97 * (9.8 + 56.5 * mpx + later * (5.16 + 2.72 * per + 30.5 * mpx));
    }
    if (p.one_round) {
        const double item_us = p.rows == 4 ? 3.44 : p.rows == 8 ? 4.59 : p.rows == 16 ? 5.6 : 8.46;
        return 12.9 + later * item_us + 395.0 * chunk_mpx < 0.95 * (9.0 + 47.6 * mpx + later * (3.6 + 1.66 * per + 4.7 * mpx));
    }
    return 21.7 + 0.1 * items + later * (0.38 + 0.18 * items + 56.4 * chunk_mpx) < 0.91 * (15.6 + 16.3 * mpx + later * (4.54 + 1.36 * per + 1.0 * mpx));
}

// The lines are those of the single blocks, an image's in the place of its activations.
LastSums conv_chain_last_sums(const ConvGeom &g, int C)
{
    LastSums l = conv_mid_last_sums(g, C);
    l.stride = (int64_t)g.h * g.w * C * 2 / 16;
    return l;
}

hipError_t launch_conv_chain(const TileSrc &src, const ConvGeom &g, int C, const ChainPlan &p, int blocks, const bf16_t *w_first,
                             const bf16_t *w_mid, const float *bias, const float *rsum, uint8_t *act0, uint8_t *act1, float *rec0,
                             float *rec1, float *lines, uint32_t *state, int patience, int num_cu, hipStream_t s)
{
    if (!p.fits) return hipErrorInvalidValue;
    ChainArgs a{src, g, blocks, w_first, w_mid, bias, rsum, {act0, act1}, {rec0, rec1}, conv_first_samples(g, C), conv_mid_samples(g, C),
                lines, (int64_t)g.h * g.w * C / 2, state, patience < 0 ? kChainPatience : patience, p.chunk, (g.n_img + p.chunk - 1) / p.chunk};
    const dim3 grid((unsigned)std::min<int64_t>(p.items * kChainTeams, num_cu));
    auto launch = [&](auto kernel, int waves) { hipLaunchKernelGGL(kernel, grid, dim3(64 * waves), 0, s, a); };
    if (C == 64) {
        if (p.rows == 4) launch(conv_chain_kernel<64, 4, 2, 1>, 4);
        else if (p.rows == 8) launch(conv_chain_kernel<64, 8, 2, 1>, 8);
        else launch(conv_chain_kernel<64, 8, 4, 1>, 8);
    } else {
        if (p.rows == 4) launch(conv_chain_kernel<32, 4, 1, 1>, 4);
        else if (p.rows == 8) launch(conv_chain_kernel<32, 4, 2, 1>, 4);
        else if (p.rows == 16) launch(conv_chain_kernel<32, 8, 2, 1>, 8);
        else launch(conv_chain_kernel<32, 8, 2, 2>, 8);
    }
    return hipGetLastError();
}

uint32_t *chain_counter(uint32_t *words, int image) { return words + kChainCountAt + (size_t)image * kChainCount; }

ChainState conv_chain_state(uint32_t *words, uint32_t *lost, const ConvGeom &g, const ChainPlan &p, int blocks)
{
    const uint32_t strips = (uint32_t)((g.h + p.rows - 1) / p.rows);
    return ChainState{words, lost, blocks, g.n_img, strips * (uint32_t)g.colblks, strips * (uint32_t)((g.w + kChainCols - 1) / kChainCols)};
}

static_assert(kChainStateBytes == (size_t)(kChainCountAt + kChainCounters * kChainCount) * 4, "ChainState");

hipError_t launch_clear_chain(uint32_t *state, hipStream_t s)
{
    hipLaunchKernelGGL(clear_chain_kernel, dim3(64), dim3(256), 0, s, state);
    return hipGetLastError();
}

hipError_t launch_nhwc_to_nchw(const bf16_t *in, int64_t n_img, int h, int w, int C, float *out, const ChainState &chain, hipStream_t s)
{
    const int64_t total = n_img * h * w * C;
    if (total <= 0) return hipSuccess;
    int64_t blocks = (total + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(nhwc_to_nchw_kernel, dim3((unsigned)blocks), dim3(256), 0, s, in, total, h * w, C, out, chain);
    return hipGetLastError();
}

} // namespace qrm
