// Batched bounded-distance Reed-Solomon decoding over GF(2^m) for gfx950.
//
// Function computed (Appendix B of the paper): for every received word, the unique codeword within
// t = (n-k)/2 symbol errors, the message in its first k symbols and the number of corrected symbols,
// or a failure flag.  The paper's decoder is Berlekamp-Welch on the CPU; these kernels reach the same
// result from the 2t syndromes S_j = sum over positions of r * alpha^((fcr+j) * power):
//
//  * t <= 2, n <= 16 (rs_decode_lane_kernel): one word per lane, the error locator in closed form;
//  * every other code (rs_decode_group_kernel): 16 or 32 lanes per word (rs_lanes_per_word), Berlekamp-Massey in its
//    inversion-free systolic form with one polynomial coefficient per lane, Chien search and Forney with
//    the positions dealt to the lanes.
//
// Field arithmetic goes through tables in LDS, which qrm_create lays out once as one image per code (rs_table_image):
// the antilog table is followed by zeros and log 0 is kZeroLog, so that a product is two look-ups and an add with
// no test for zero; what is multiplied again and again by the same constant has a table of its own.
//
// Key verification (Section 4.3: the corrected message is compared with the predetermined key) rides in
// the decoder's epilogue when a key is given: the number of message bits that agree with the key's and
// (count >= tau) are written.  The same count for messages already in memory is `verify_kernel`, a plain
// streaming pass.
#include <algorithm>

#include "qrm_internal.h"
#include "rs_lane.h"

namespace qrm {

namespace {

// ---- what the table image holds behind kCodeAt for the group kernel (rs_lane.h has the rest)
//   group kernel: (SPL > 1) syndromes: u8 [SPL][q][2 TMAX], byte j of entry (s, v): v * alpha^(G (SPL - 1 - s) (fcr + j)), 0 from 2t on;
//                 (SPL > 1) Chien: u8 [TMAX][q][chien_bytes(SPL)], byte s of entry (j - 1, v): v * alpha^(G j s), 0 for j > t
//                 what differs from lane to lane: u8 [G][kLaneBytes]: exponents of alpha, (fcr + j) last_pw for j < 2 TMAX
//                 (last_pw: the power of the lane's symbol SPL - 1), then j first_x for j <= TMAX (first_x: minus the power of its
//                 symbol 0)
constexpr int kLaneBytes = 28;
// The t a kernel is made for: terms beyond the code's own t are looked up all the same, which shows where a lane has few symbols.  2^20 words
// of 17 symbols and t = 1, made for two / for four: 111 / 135 us; of 24 and t = 2 125 / 151.
constexpr int group_tmax(int two_t) { return two_t > 8 ? 8 : two_t > 4 ? 4 : 2; }
// Bytes of a table's entry.  A lane's only symbol needs no tables: its terms are its value times the lane's own powers, and a term of
// the locator at its first position is all there is (2^20 words of RS(15,9) 135 us, 153 by way of the tables).
constexpr int syn_bytes(int spl, int tmax) { return spl == 1 ? 0 : 2 * tmax; }
constexpr int chien_bytes(int spl) { return spl == 1 ? 0 : spl < 4 ? 4 : spl; }
constexpr int64_t kDecodeThreads = 2048 * 256; // lane kernel: 32 wavefronts per compute unit; a workgroup reads the tables once and takes the runs of words a grid apart
// Group kernel: three workgroups of eight wavefronts to a compute unit (up to 51 KiB of tables each), every 768th run of words.
// 20000 words of RS(255,239) 20.7 us, with two workgroups of the same size 22.
constexpr int kGroupThreads = 512;
constexpr int64_t kGroupBlocks = 768;
constexpr int64_t kSecondSplitWords = 10240;

int group_symbols(int n, int G) // SPL: symbols per lane, rounded up to a power of two
{
    int spl = 1;
    while (spl * G < n) spl *= 2;
    return spl;
}
int group_lanes(int two_t) { return two_t > 8 ? 32 : 16; } // 3t + 1 coefficients of the systolic recursion, one per lane
// Words of more than 128 symbols take 16 look-ups of a lane one behind the other, which shows where a launch has so few
// of them that every workgroup takes one run: while 32 lanes a word still fit the chip that way, they have 32.  RS(255,247), 16 /
// 32 lanes: 4096 words 8.1 / 7.9 us, 10240 10.2 / 9.8, 16000 10.7 / 12.2; RS(255,251) 7.9 / 7.9, 8.7 / 8.5, 9.1 / 10.3.
bool second_split(int n, int two_t) { return n > 128 && two_t <= 8; }
bool takes_second_split(const RsParams &p, int64_t N) { return second_split(p.n, p.two_t) && N <= kSecondSplitWords; }

// table image -> LDS, 16 bytes per lane and step
template <int THREADS>
__device__ __forceinline__ void load_tables(uint8_t *dst, const RsParams &p)
{
    for (int i = threadIdx.x * 16; i < p.tab_bytes; i += THREADS * 16) *(u32x4 *)(dst + i) = *(const u32x4 *)(p.tab + i);
}

// ------------------------------------------------------------------------------------------------
// Short codes with t <= 2: one word per lane, nothing repeated across lanes, no serial recursion.
// A lane holds its word as packed bytes (N4 = ceil(n/4) dwords).  The syndromes of a symbol at its position are ONE
// 32-bit look-up (all four in it), so the whole syndrome computation is n look-ups and n XORs; the errors follow in closed
// form (lane_errors).
// Bound by vector instructions and LDS look-ups, about 200 and 40 per word, close to what the bytes alone take.
// 2^20 words of RS(12,8) over GF(256), 34.6 MB: 12.5 -> 11.8 us a pass = 2.9 TB/s (a recursion per lane with byte-wise loads: 44.5 us), of
// which 5 are the launch, the tables and the first words, which are on their way together: every further 2^20 take 6.6 (5.2 TB/s).
// A workgroup's next words are fetched while it decodes: 2^20 of RS(15,11) 21.9 -> 20.0 us, of RS(13,9) 22.0 -> 20.8.
// WORDS: words and messages are whole aligned dwords, read and written straight from global memory; otherwise a
// workgroup's words pass through LDS so that global memory is still accessed in dwords.
// ------------------------------------------------------------------------------------------------
template <int N4, bool WORDS, int TH>
__global__ __launch_bounds__(TH) void rs_decode_lane_kernel(RsParams p, const uint8_t *__restrict__ sym, int64_t N,
                                                             uint8_t *__restrict__ msg, uint8_t *__restrict__ cw,
                                                             int8_t *__restrict__ nerr, KeyArgs key)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t s_tab[];
    __shared__ __attribute__((aligned(16))) uint8_t s_word[WORDS ? 16 : TH * 16 + 16];
    __shared__ __attribute__((aligned(16))) uint8_t s_msg[WORDS ? 16 : TH * 16];
    const int tid = threadIdx.x;
    const int n = p.n, k = p.k, ord = p.q - 1, fcr = p.fcr;
    const int64_t blocks = (N + TH - 1) / TH;
    const bool in_dwords = WORDS || ((uintptr_t)sym & 3) == 0; // TH n is a multiple of four: every workgroup's run is aligned as the first
    uint32_t in[N4]; // run b's words: the lane's own (WORDS) or dwords of all of them
    auto fetch = [&](int64_t b) {
        const int64_t w0 = b * TH;
        if (WORDS) {
            const uint32_t *src = (const uint32_t *)(sym + min(w0 + tid, N - 1) * n);
#pragma unroll
            for (int j = 0; j < N4; ++j) in[j] = src[j];
        } else if (in_dwords) {
            const uint32_t *src = (const uint32_t *)(sym + w0 * n);
            const int dwords = (int)min((int64_t)TH, N - w0) * n >> 2;
#pragma unroll
            for (int j = 0; j < N4; ++j)
                if (tid + TH * j < dwords) in[j] = src[tid + TH * j];
        }
    };
    fetch(blockIdx.x); // (there is one for every workgroup)
    load_tables<TH>(s_tab, p);
    const Gf gf{s_tab, (const uint16_t *)(s_tab + kLogAt)};
    const uint8_t *quad = s_tab + kQuadAt;
    const uint32_t *syn = (const uint32_t *)(s_tab + kCodeAt);
    const uint32_t field = (uint32_t)ord * 0x01010101u;
    uint32_t in_word[N4], in_msg[N4], keyw[N4]; // byte masks: symbols of the word, bits of the message; the key
#pragma unroll
    for (int j = 0; j < N4; ++j) {
        const int left = n - 4 * j, leftk = k - 4 * j;
        in_word[j] = field & (left >= 4 ? 0xffffffffu : (1u << (8 * left)) - 1u);
        in_msg[j] = field & (leftk >= 4 ? 0xffffffffu : leftk <= 0 ? 0u : (1u << (8 * leftk)) - 1u);
        keyw[j] = key.matches ? ((const uint32_t *)key.key)[j] : 0u;
    }
    __syncthreads();

    for (int64_t b = blockIdx.x; b < blocks; b += gridDim.x) {
        const int64_t w0 = b * TH;
        const int cnt = (int)min((int64_t)TH, N - w0);
        const bool mine = tid < cnt;
        const int64_t w = w0 + (mine ? tid : 0);
        uint32_t r[N4];
        if (WORDS) {
#pragma unroll
            for (int j = 0; j < N4; ++j) r[j] = in[j];
        } else {
            const uint8_t *src = sym + w0 * n;
            const int bytes = cnt * n;
            if (in_dwords) {
#pragma unroll
                for (int j = 0; j < N4; ++j)
                    if (tid + TH * j < bytes >> 2) ((uint32_t *)s_word)[tid + TH * j] = in[j];
                if (tid < (bytes & 3)) s_word[(bytes & ~3) + tid] = src[(bytes & ~3) + tid];
            } else {
                for (int i = tid; i < bytes; i += TH) s_word[i] = src[i];
            }
            __syncthreads();
            const int at = tid * n;
            const uint32_t *q = (const uint32_t *)s_word + (at >> 2);
            uint32_t lo = q[0];
#pragma unroll
            for (int j = 0; j < N4; ++j) {
                const uint32_t hi = q[j + 1];
                r[j] = __builtin_amdgcn_alignbyte(hi, lo, (unsigned)(at & 3));
                lo = hi;
            }
        }
#pragma unroll
        for (int j = 0; j < N4; ++j) r[j] &= in_word[j];

        if (b + gridDim.x < blocks) fetch(b + gridDim.x);

        // ---- syndromes, a byte each
        uint32_t S = 0;
#pragma unroll
        for (int i = 0; i < 4 * N4; ++i) S ^= syn[i * p.q + ((r[i / 4] >> (8 * (i % 4))) & 0xffu)];
        const LaneErrors err = lane_errors(gf, quad, S, n, ord, p.two_t);
        if (err.ok && err.count > 0) {
            auto fix = [&](int pw, int a) {
                const int i = n - 1 - pw;
                const uint32_t v = (uint32_t)lane_error_value(gf, pw, a, fcr, ord) << (8 * (i & 3));
#pragma unroll
                for (int j = 0; j < N4; ++j) r[j] ^= (i >> 2) == j ? v : 0u;
            };
            fix(err.p1, err.a1);
            if (err.count == 2) fix(err.p2, err.a2);
        }

        // ---- write back
        if (WORDS) {
            if (mine) {
                if (cw) {
                    uint32_t *d = (uint32_t *)(cw + w * n);
#pragma unroll
                    for (int j = 0; j < N4; ++j) d[j] = r[j];
                }
                uint32_t *d = (uint32_t *)(msg + w * k);
#pragma unroll
                for (int j = 0; j < N4; ++j)
                    if (4 * j < k) d[j] = r[j];
            }
        } else {
            __syncthreads(); // every lane has taken its word out of the dwords it shares with its neighbours
            if (mine) {
#pragma unroll
                for (int i = 0; i < 4 * N4; ++i) {
                    const uint8_t v = (uint8_t)(r[i / 4] >> (8 * (i % 4)));
                    if (i < n) s_word[tid * n + i] = v;
                    if (i < k) s_msg[tid * k + i] = v;
                }
            }
            __syncthreads();
            auto copy_out = [&](uint8_t *dst, const uint8_t *from, int bytes) {
                if (((uintptr_t)dst & 3) == 0) {
                    for (int i = tid; i < bytes >> 2; i += TH) ((uint32_t *)dst)[i] = ((const uint32_t *)from)[i];
                    if (tid < (bytes & 3)) dst[(bytes & ~3) + tid] = from[(bytes & ~3) + tid];
                } else {
                    for (int i = tid; i < bytes; i += TH) dst[i] = from[i];
                }
            };
            if (cw) copy_out(cw + w0 * n, s_word, cnt * n);
            copy_out(msg + w0 * k, s_msg, cnt * k);
            __syncthreads();
        }
        if (mine) {
            nerr[w] = (int8_t)(err.ok ? err.count : -1);
            if (key.matches) {
                int agree = k * p.m;
#pragma unroll
                for (int j = 0; j < N4; ++j) agree -= __popc((r[j] ^ keyw[j]) & in_msg[j]);
                key.matches[w] = agree;
                if (key.detected) key.detected[w] = (uint8_t)(agree >= key.tau);
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// All other codes: G = 16 (t <= 4) or 32 (t <= 8, or few long words) lanes per word, four or two words per wavefront.  Lane l holds the
// symbols l, l + G, l + 2G, .. (SPL of them).
//   Syndromes   symbol s of a lane enters syndrome j with alpha^((fcr + j) (last_pw + G (SPL - 1 - s))): the lane's part is
//               multiplied on at the end, the rest is the same for all lanes and ONE look-up of a symbol gives its terms of
//               all 2t syndromes, a byte each.  The lanes' terms are then added up.
//   Recursion   Berlekamp-Massey without inversions in its systolic form (the "RiBM" of Sarwate and Shanbhag): lane i
//               holds coefficient i of the 3t + 1 of one polynomial, an iteration is two products per lane and a
//               shift by one lane, and at the end lanes t .. 2t hold the locator Lambda and lanes 0 .. t-1 the
//               high part Omega_h of Lambda S = Omega + x^(2t) Omega_h.
//   Chien       likewise: ONE look-up of the term Lambda_j x^j at the lane's first position gives that term at all of the
//               lane's positions, a byte each; a byte in which the t + 1 of them cancel is an error's position.
//   Forney      at those positions only: error value X^(-fcr-2t) Omega_h(1/X) / (sum of the odd terms of Lambda at 1/X);
//               Omega(1/X) equals X^(-2t) Omega_h(1/X) because Lambda(1/X) = 0.
// A wavefront whose words are all error free stops after the syndromes.
// Bound by vector instructions and LDS look-ups, about 700 and 150 of a wavefront for its words; 20000 words of RS(255,239):
// 20.7 us a pass (with a look-up for every symbol and syndrome, every position and coefficient, and Omega_h carried along at
// every position, 1270 and 390: 37 us; the recursion repeated on all 64 lanes of a word: 388).
// ------------------------------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ uint32_t xor_dpp(uint32_t v)
{
    return v ^ (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
template <int G>
__device__ __forceinline__ uint32_t group_xor(uint32_t v)
{
    v = xor_dpp<0xB1>(v);  // quad_perm [1,0,3,2]
    v = xor_dpp<0x4E>(v);  // quad_perm [2,3,0,1]
    v = xor_dpp<0x141>(v); // row_half_mirror
    v = xor_dpp<0x140>(v); // row_mirror
    if (G == 32) v ^= (uint32_t)__shfl_xor((int)v, 16, 32);
    return v;
}

template <int G>
__device__ __forceinline__ uint32_t group_mask(bool pred, int lane) // lanes of this lane's group where pred holds
{
    const unsigned long long mask = __ballot(pred);
    return (uint32_t)(mask >> (lane / G * G)) & (uint32_t)((1ull << G) - 1ull);
}

template <int CTRL>
__device__ __forceinline__ int add_dpp(int v)
{
    return v + __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int G>
__device__ __forceinline__ int group_add(int v)
{
    v = add_dpp<0xB1>(v); // (as group_xor)
    v = add_dpp<0x4E>(v);
    v = add_dpp<0x141>(v);
    v = add_dpp<0x140>(v);
    if (G == 32) v += __shfl_xor(v, 16, 32);
    return v;
}

// The value of the lane above within the group; the top lane gets `fill`.
template <int G>
__device__ __forceinline__ int from_above(int v, int fill, int lane_g)
{
    if (G == 16) return __builtin_amdgcn_update_dpp(fill, v, 0x101, 0xf, 0xf, false); // row_shl:1
    const int up = __builtin_amdgcn_update_dpp(0, v, 0x130, 0xf, 0xf, true);         // wave_shl:1
    return lane_g == G - 1 ? fill : up;
}

// The value of the group's lane 0.
template <int G>
__device__ __forceinline__ int from_first(int v)
{
    v = __builtin_amdgcn_update_dpp(0, v, 0x150, 0xf, 0xf, true);                   // row_newbcast:0
    if (G == 32) v = __builtin_amdgcn_update_dpp(v, v, 0x142, 0xa, 0xf, false);     // row_bcast:15 into rows 1 and 3
    return v;
}

// BYTES consecutive bytes of LDS as dwords
template <int BYTES>
struct Packed {
    uint32_t d[BYTES / 4];
    __device__ __forceinline__ void load(const uint8_t *p)
    {
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        if constexpr (BYTES == 4) d[0] = *(const uint32_t *)p;
        else if constexpr (BYTES == 8) {
            const u32x2 v = *(const u32x2 *)p;
            d[0] = v[0]; d[1] = v[1];
        } else {
            const u32x4 v = *(const u32x4 *)p;
            d[0] = v[0]; d[1] = v[1]; d[2] = v[2]; d[3] = v[3];
        }
    }
};

template <int G, int TMAX, int SPL>
__global__ __launch_bounds__(kGroupThreads, 6) void rs_decode_group_kernel(RsParams p, const uint8_t *__restrict__ sym, int64_t N,
                                                                           uint8_t *__restrict__ msg, uint8_t *__restrict__ cw,
                                                                           int8_t *__restrict__ nerr, KeyArgs key)
{
    static_assert(3 * TMAX + 1 <= G, "one lane per coefficient");
    extern __shared__ __attribute__((aligned(16))) uint8_t s_tab[];
    __shared__ uint8_t s_key[256];
    const int tid = threadIdx.x, lane = tid & 63, l = tid % G;
    const int n = p.n, k = p.k, ord = p.q - 1, q = p.q, two_t = p.two_t, t = p.two_t / 2;
    const uint32_t field = (uint32_t)ord * 0x01010101u;
    const bool with_key = key.matches != nullptr;
    load_tables<kGroupThreads>(s_tab, p);
    if (tid < 256) s_key[tid] = (with_key && tid < k) ? key.key[tid] : 0;
    __syncthreads();
    const Gf gf{s_tab, (const uint16_t *)(s_tab + kLogAt)};
    constexpr int SB = 2 * TMAX, CB = chien_bytes(SPL);
    const uint8_t *syn = s_tab + kCodeAt, *chien = syn + SPL * q * syn_bytes(SPL, TMAX);

    // this lane's fixed exponents, a byte each: (fcr + j) last_pw, j first_x (1 / X of its symbol 0)
    const int lift = (p.fcr + two_t) % ord;                // X^(-fcr-2t) = x^(fcr+2t)
    const float inv_ord = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, 1.0f / (float)ord))); // (a scalar register)
    constexpr int ND = SB / 4, NL = (TMAX + 4) / 4;
    auto byte_of = [](const uint32_t *v, int j) { return (int)((v[j / 4] >> (8 * (j % 4))) & 0xffu); };
    // symbols l + s G of a word of `len` symbols: all lanes have one, some do, none does
    auto each_symbol = [&](int len, auto &&body) {
        int full = len / G;
        asm volatile("" : "+s"(full)); // compared where it is used: kept for the whole loop, the conditions would not fit the scalar registers
        const int rest = l < len - full * G ? full : -1;
#pragma unroll
        for (int s = 0; s < SPL; ++s) {
            if (s < full || s == rest) body(s);
        }
    };

    constexpr int GPB = kGroupThreads / G; // words per workgroup and iteration
    const int64_t stride = (int64_t)gridDim.x * GPB;
    const int64_t iters = (N + stride - 1) / stride; // the same for every lane: cross-lane operations see full wavefronts
    for (int64_t it = 0; it < iters; ++it) {
        auto word_index = [&]() { // found again for the write-back: the registers between are scarce
            int id = tid;
            asm volatile("" : "+v"(id));
            return it * stride + (int64_t)blockIdx.x * GPB + id / G;
        };
        const int64_t w = word_index();
        const bool valid = w < N;
        constexpr int NR = (SPL + 3) / 4;
        uint32_t r[NR] = {}; // the lane's symbols, a byte each
        {
            uint32_t one[SPL] = {};
            if (valid) {
                const uint8_t *word = sym + w * n + l;
                each_symbol(n, [&](int s) { one[s] = word[s * G]; });
            }
#pragma unroll
            for (int s = 0; s < SPL; ++s) r[s / 4] |= one[s] << (8 * (s % 4));
#pragma unroll
            for (int d = 0; d < NR; ++d) r[d] &= field;
        }
        // ---- syndromes
        uint32_t last_e[ND], first_e[NL];
        {
            int at = l * kLaneBytes;
            asm volatile("" : "+v"(at)); // read for every word: the registers are scarce
            const uint32_t *mine = (const uint32_t *)(chien + TMAX * q * CB + at);
#pragma unroll
            for (int d = 0; d < ND; ++d) last_e[d] = mine[d];
#pragma unroll
            for (int d = 0; d < NL; ++d) first_e[d] = mine[ND + d];
        }
        uint32_t Spk[ND];
        if constexpr (SPL > 1) {
#pragma unroll
            for (int s = 0; s < SPL; ++s) {
                Packed<SB> term;
                term.load(syn + (s * q + byte_of(r, s)) * SB);
#pragma unroll
                for (int d = 0; d < ND; ++d) Spk[d] = s == 0 ? term.d[d] : Spk[d] ^ term.d[d];
                if (SB == 16 && s % 4 == 3) __builtin_amdgcn_sched_barrier(0); // four look-ups of 16 bytes at a time: registers
            }
        }
        const int log_r = SPL == 1 ? gf.L((int)r[0]) : 0; // a lane's only symbol: the same in all of its terms
#pragma unroll
        for (int j0 = 0; j0 < SB; j0 += 8) { // eight at a time: registers
            constexpr int W = SB < 8 ? SB : 8;
            int v[W];
#pragma unroll
            for (int j = 0; j < W; ++j) v[j] = SPL == 1 ? log_r : gf.L(byte_of(Spk, j0 + j));
#pragma unroll
            for (int j = 0; j < W; ++j) v[j] = gf.E(v[j] + byte_of(last_e, j0 + j));
#pragma unroll
            for (int j = 0; j < W; j += 4) {
                const int d = (j0 + j) / 4, left = two_t - 4 * d; // of these four, the code has `left`
                Spk[d] = (uint32_t)v[j] | (uint32_t)v[j + 1] << 8 | (uint32_t)v[j + 2] << 16 | (uint32_t)v[j + 3] << 24;
                if (SPL == 1) Spk[d] &= left >= 4 ? 0xffffffffu : left <= 0 ? 0u : (1u << (8 * left)) - 1u;
            }
            if (SB > 8) __builtin_amdgcn_sched_barrier(0);
        }
        uint32_t any = 0;
#pragma unroll
        for (int d = 0; d < ND; ++d) {
            Spk[d] = group_xor<G>(Spk[d]);
            any |= Spk[d];
        }
        int L = 0;
        bool fail = false;
        if (__ballot(any != 0)) {
            // ---- recursion: coefficient l of this word's polynomial
            uint32_t mine = 0;
#pragma unroll
            for (int d = 0; d < ND; ++d) mine = (l >> 2) == d ? Spk[d] : mine;
            int delta = (int)((mine >> (8 * (l & 3))) & 0xffu);
            delta = l < two_t ? delta : (l == 3 * t ? 1 : 0);
            int ldelta = gf.L(delta), ltheta = ldelta, lgamma = 0, kk = 0;
            for (int rr = 0; rr < two_t; ++rr) {
                const int up = from_above<G>(ldelta, kZeroLog, l), d0 = from_first<G>(ldelta);
                int a = gf.E(lgamma + up), b = gf.E(d0 + ltheta);
                asm volatile("" : "+v"(a), "+v"(b)); // (whole registers: the compiler otherwise cuts their sum to a byte once more)
                delta = a ^ b;
                const bool grow = d0 != kZeroLog && kk >= 0;
                ltheta = grow ? up : ltheta;
                lgamma = grow ? d0 : lgamma;
                kk = grow ? -kk - 1 : kk + 1;
                ldelta = gf.L(delta);
            }
            L = (two_t - kk) >> 1; // the recursion's length; kk < 0: longer than t
            fail = kk < 0;
            // degree of Lambda must equal L (a group's lanes agree on L and fail)
            if (!fail && L > 0) fail = __shfl(ldelta, t + L, G) == kZeroLog;

            // ---- Chien: logarithms of the coefficients (zero beyond t), terms at this lane's first position, then at all of them
            int llam[TMAX + 1], lam[TMAX + 1];
            const int lhigh = l <= 2 * t ? ldelta : kZeroLog;
#pragma unroll
            for (int j = 0; j <= TMAX; ++j) {
                llam[j] = __shfl(lhigh, t + j, G);
            }
#pragma unroll
            for (int j = 0; j <= TMAX; ++j) lam[j] = gf.E(llam[j] + byte_of(first_e, j));
            uint32_t roots = 0; // bit s: symbol l + s G is in error
            if constexpr (SPL == 1) {
                int sum = lam[0];
#pragma unroll
                for (int j = 1; j <= TMAX; ++j) sum ^= lam[j];
                roots = sum == 0;
            } else {
                uint32_t sum[CB / 4];
#pragma unroll
                for (int d = 0; d < CB / 4; ++d) sum[d] = (uint32_t)lam[0] * 0x01010101u;
#pragma unroll
                for (int j = 1; j <= TMAX; ++j) {
                    Packed<CB> term;
                    term.load(chien + ((j - 1) * q + lam[j]) * CB);
#pragma unroll
                    for (int d = 0; d < CB / 4; ++d) sum[d] ^= term.d[d];
                }
#pragma unroll
                for (int d = 0; d < CB / 4; ++d) {
                    const uint32_t some = ((sum[d] & 0x7f7f7f7fu) + 0x7f7f7f7fu) | sum[d]; // bit 7 of a byte: it is not zero
                    roots |= (((~some >> 7) & 0x01010101u) * 0x01020408u >> 24) << (4 * d);
                }
            }
            const int slots = (n - l + G - 1) / G; // symbols this lane holds
            roots &= !fail && L > 0 ? (1u << max(slots, 0)) - 1u : 0u;
            if (group_add<G>(__popc(roots)) != L) fail = true;
            // ---- Forney: the lane's noted positions one after the other, all lanes together
            if (fail) roots = 0;
            bool bad = false;
            uint32_t ev[NR] = {}; // error values, a byte each
            int lom[TMAX];
            if (__ballot(roots != 0)) {
#pragma unroll
                for (int j = 0; j < TMAX; ++j) lom[j] = __shfl(l < t ? ldelta : kZeroLog, j, G);
            }
            while (__ballot(roots != 0)) {
                const bool has = roots != 0;
                const int s = has ? __ffs(roots) - 1 : 0;
                roots &= roots - 1;
                const int x = mod_once(byte_of(first_e, 1) + s * G, ord); // exponent of 1 / X
                int e = 0, odd = 0, num = 0;
#pragma unroll
                for (int j = 0; j <= TMAX; ++j) {
                    if (j < TMAX) num ^= gf.E(lom[j] + e);
                    if (j & 1) odd ^= SPL == 1 ? lam[j] : gf.E(llam[j] + e);
                    e = SPL == 1 && j < TMAX ? byte_of(first_e, j + 1) : mod_once(e + x, ord);
                }
                bad = bad || (has && (odd == 0 || num == 0));
                const int quot = gf.E(gf.L(num) + (odd ? ord - gf.L(odd) : 0));
                int lx = lift * x;                            // below 2^16: the quotient is off by one at most
                lx -= (int)((float)lx * inv_ord) * ord;
                lx = lx < 0 ? lx + ord : lx >= ord ? lx - ord : lx;
                const uint32_t v = has ? (uint32_t)gf.E(gf.L(quot) + lx) << (8 * (s & 3)) : 0u;
#pragma unroll
                for (int d = 0; d < NR; ++d) ev[d] |= (s >> 2) == d ? v : 0u;
            }
            if (group_mask<G>(bad, lane) != 0) fail = true;
            if (!fail) {
#pragma unroll
                for (int d = 0; d < NR; ++d) r[d] ^= ev[d];
            }
        }

        // ---- write back
        int agree = 0;
        const int64_t wo = word_index();
        if (wo < N) {
            if (cw) {
                uint8_t *dst = cw + wo * n + l;
                each_symbol(n, [&](int s) { dst[s * G] = (uint8_t)(r[s / 4] >> (8 * (s % 4))); });
            }
            uint8_t *dst = msg + wo * k + l;
            each_symbol(k, [&](int s) {
                const uint32_t v = r[s / 4] >> (8 * (s % 4));
                dst[s * G] = (uint8_t)v;
                if (with_key) agree += p.m - __popc((v ^ s_key[l + s * G]) & (uint32_t)ord);
            });
        }
        if (wo < N && l == 0) nerr[wo] = (int8_t)(fail ? -1 : L);
        if (with_key) {
#pragma unroll
            for (int off = G / 2; off >= 1; off >>= 1) agree += __shfl_xor(agree, off, G);
            if (wo < N && l == 0) {
                key.matches[wo] = agree;
                if (key.detected) key.detected[wo] = (uint8_t)(agree >= key.tau);
            }
        }
    }
}

// Agreement of stored messages with the key: one word per lane, V bytes of it per load.
template <typename V>
__global__ __launch_bounds__(256) void verify_kernel(const uint8_t *__restrict__ msg, int64_t N, int k, int m,
                                                     KeyArgs key)
{
    __shared__ V s_key[256 / sizeof(V)];
    const int per = k / (int)sizeof(V);
    if ((int)threadIdx.x < per) s_key[threadIdx.x] = reinterpret_cast<const V *>(key.key)[threadIdx.x];
    __syncthreads();
    V mask = 0;
#pragma unroll
    for (int b = 0; b < (int)sizeof(V); ++b) mask |= (V)((1u << m) - 1u) << (8 * b);
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t w = (int64_t)blockIdx.x * 256 + threadIdx.x; w < N; w += stride) {
        const V *src = reinterpret_cast<const V *>(msg + w * k);
        int differ = 0;
        for (int j = 0; j < per; ++j) differ += __popcll((unsigned long long)((src[j] ^ s_key[j]) & mask));
        const int agree = k * m - differ;
        key.matches[w] = agree;
        if (key.detected) key.detected[w] = (uint8_t)(agree >= key.tau);
    }
}

// G lanes a word; p's tables are the ones for G
template <int G, int TMAX, int SPL>
hipError_t launch_group(const RsParams &p, const uint8_t *sym, int64_t N, uint8_t *msg, uint8_t *cw, int8_t *nerr,
                        const KeyArgs &key, hipStream_t s)
{
    constexpr int GPB = kGroupThreads / G;
    const int64_t blocks = std::min<int64_t>((N + GPB - 1) / GPB, kGroupBlocks);
    hipLaunchKernelGGL((rs_decode_group_kernel<G, TMAX, SPL>), dim3((unsigned)blocks), dim3(kGroupThreads), (unsigned)p.tab_bytes, s, p,
                       sym, N, msg, cw, nerr, key);
    return hipGetLastError();
}

template <int N4>
hipError_t launch_lane(const RsParams &p, const uint8_t *sym, int64_t N, uint8_t *msg, uint8_t *cw, int8_t *nerr,
                       const KeyArgs &key, hipStream_t s)
{
    const bool words = p.n % 4 == 0 && p.k % 4 == 0 && (((uintptr_t)sym | (uintptr_t)msg | (uintptr_t)cw) & 3) == 0;
    auto launch = [&](auto kernel, int threads) {
        const int64_t blocks = std::min((N + threads - 1) / threads, kDecodeThreads / threads);
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(threads), (unsigned)p.tab_bytes, s, p, sym, N, msg, cw, nerr, key);
    };
    // Whole dwords over GF(256), whose tables are 10 KB and more, and a full run a workgroup: half as many copies of the tables.  RS(12,8), 256 /
    // 512 threads: 2^18 + 38 k words 5.6 / 5.7 us, 2^19 8.1 / 7.6, 786 k 10.2 / 9.4, 2^20 11.7 / 11.1, 1.5 M 14.3 / 14.5, 2^21 18.5 / 17.7, 2^22
    // 31.0 / 29.2 (28 counts of 2^19 .. 2^23: 1.025 times as fast in the mean, 0.98 .. 1.08; RS(16,12) 1.05, RS(8,4) 1.01).  Not over smaller
    // fields: over GF(16) 0.99 in the mean, 1.5 M words 12.8 / 13.6.  Nor through LDS: 2^20 of RS(15,11), 256 / 512 / 1024 threads 19.6 / 22.3 / 24.1.
    if (words && p.q == 256 && N >= kDecodeThreads) launch(rs_decode_lane_kernel<N4, true, 512>, 512);
    else if (words) launch(rs_decode_lane_kernel<N4, true, 256>, 256);
    else launch(rs_decode_lane_kernel<N4, false, 256>, 256);
    return hipGetLastError();
}

} // namespace

std::vector<uint8_t> rs_table_image(RsParams &p, const std::vector<uint8_t> &exp2, const std::vector<uint8_t> &lg)
{
    const int q = p.q, ord = q - 1;
    auto mul_pow = [&](int v, int e) { return v ? exp2[lg[v] + e % ord] : (uint8_t)0; };
    std::vector<uint8_t> img(kCodeAt, 0);
    for (int i = 0; i < 2 * ord; ++i) img[i] = exp2[i];
    for (int v = 0; v < 256; ++v) {
        const uint16_t x = v == 0 || v >= q ? (uint16_t)kZeroLog : (uint16_t)lg[v];
        img[kLogAt + 2 * v] = (uint8_t)x;
        img[kLogAt + 2 * v + 1] = (uint8_t)(x >> 8);
    }
    for (int y = q - 1; y >= 2; --y) img[kQuadAt + (mul_pow(y, lg[y]) ^ y)] = (uint8_t)y; // (0 and 1 give 0)
    if (lane_code(p.n, p.two_t)) {
        for (int i = 0; i < 4 * ((p.n + 3) / 4); ++i)
            for (int v = 0; v < q; ++v)
                for (int j = 0; j < 4; ++j)
                    img.push_back(i < p.n && j < p.two_t ? mul_pow(v, (p.fcr + j) * (p.n - 1 - i)) : (uint8_t)0);
        img.resize((img.size() + 15) / 16 * 16, 0);
        p.tab_bytes = (int)img.size();
        return img;
    }
    const std::vector<uint8_t> common = img;
    auto add_group = [&](int G) {
        const int tmax = group_tmax(p.two_t), spl = group_symbols(p.n, G);
        for (int s = 0; s < spl; ++s)
            for (int v = 0; v < q; ++v)
                for (int j = 0; j < syn_bytes(spl, tmax); ++j) img.push_back(j < p.two_t ? mul_pow(v, G * (spl - 1 - s) * (p.fcr + j)) : (uint8_t)0);
        for (int j = 1; j <= tmax; ++j)
            for (int v = 0; v < q; ++v)
                for (int s = 0; s < chien_bytes(spl); ++s) img.push_back(j <= p.two_t / 2 && s < spl ? mul_pow(v, G * j * s) : (uint8_t)0);
        for (int l = 0; l < G; ++l) {
            const int last_pw = ((p.n - 1 - l - G * (spl - 1)) % ord + ord) % ord, first_x = ((l - (p.n - 1)) % ord + ord) % ord;
            const size_t end = img.size() + kLaneBytes;
            for (int j = 0; j < 2 * tmax; ++j) img.push_back((uint8_t)((p.fcr + j) * last_pw % ord));
            for (int j = 0; j <= tmax; ++j) img.push_back((uint8_t)(j * first_x % ord));
            img.resize(end, 0);
        }
        img.resize((img.size() + 15) / 16 * 16, 0);
    };
    add_group(group_lanes(p.two_t));
    p.tab_bytes = (int)img.size();
    if (second_split(p.n, p.two_t)) { // a second image behind the first
        img.insert(img.end(), common.begin(), common.end());
        add_group(32);
        p.tab2_bytes = (int)img.size() - p.tab_bytes;
    }
    return img;
}

int rs_lanes_per_word(const RsParams &p, int64_t N)
{
    return lane_code(p.n, p.two_t) ? 1 : takes_second_split(p, N) ? 32 : group_lanes(p.two_t);
}

hipError_t launch_rs_decode(const RsParams &p, const uint8_t *sym, int64_t N, uint8_t *msg, uint8_t *cw, int8_t *nerr,
                            const KeyArgs &key, hipStream_t s)
{
    if (N <= 0) return hipSuccess;
    if (lane_code(p.n, p.two_t)) {
        switch ((p.n + 3) / 4) {
        case 1: return launch_lane<1>(p, sym, N, msg, cw, nerr, key, s);
        case 2: return launch_lane<2>(p, sym, N, msg, cw, nerr, key, s);
        case 3: return launch_lane<3>(p, sym, N, msg, cw, nerr, key, s);
        default: return launch_lane<4>(p, sym, N, msg, cw, nerr, key, s);
        }
    }
    if (takes_second_split(p, N)) {
        RsParams second = p;
        second.tab += p.tab_bytes;
        second.tab_bytes = p.tab2_bytes;
        if (group_tmax(p.two_t) == 2) return launch_group<32, 2, 8>(second, sym, N, msg, cw, nerr, key, s);
        return launch_group<32, 4, 8>(second, sym, N, msg, cw, nerr, key, s);
    }
    const int tmax = group_tmax(p.two_t);
    switch (group_symbols(p.n, group_lanes(p.two_t))) {
    case 1: return tmax == 8 ? launch_group<32, 8, 1>(p, sym, N, msg, cw, nerr, key, s) : launch_group<16, 4, 1>(p, sym, N, msg, cw, nerr, key, s);
    case 2: return tmax == 8 ? launch_group<32, 8, 2>(p, sym, N, msg, cw, nerr, key, s)
                 : tmax == 4 ? launch_group<16, 4, 2>(p, sym, N, msg, cw, nerr, key, s) : launch_group<16, 2, 2>(p, sym, N, msg, cw, nerr, key, s);
    case 4: return tmax == 8 ? launch_group<32, 8, 4>(p, sym, N, msg, cw, nerr, key, s)
                 : tmax == 4 ? launch_group<16, 4, 4>(p, sym, N, msg, cw, nerr, key, s) : launch_group<16, 2, 4>(p, sym, N, msg, cw, nerr, key, s);
    case 8: return tmax == 8 ? launch_group<32, 8, 8>(p, sym, N, msg, cw, nerr, key, s)
                 : tmax == 4 ? launch_group<16, 4, 8>(p, sym, N, msg, cw, nerr, key, s) : launch_group<16, 2, 8>(p, sym, N, msg, cw, nerr, key, s);
    default: return tmax == 4 ? launch_group<16, 4, 16>(p, sym, N, msg, cw, nerr, key, s) : launch_group<16, 2, 16>(p, sym, N, msg, cw, nerr, key, s);
    }
}

hipError_t launch_verify(const RsParams &p, const uint8_t *msg, int64_t N, const KeyArgs &key, hipStream_t s)
{
    if (N <= 0) return hipSuccess;
    int64_t blocks = (N + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    const dim3 grid((unsigned)blocks), block(256);
    // wide loads need every word (and the key) to start on a multiple of the load width
    const uintptr_t a = (uintptr_t)msg | (uintptr_t)key.key;
    if (p.k % 8 == 0 && a % 8 == 0)
        hipLaunchKernelGGL(verify_kernel<uint64_t>, grid, block, 0, s, msg, N, p.k, p.m, key);
    else if (p.k % 4 == 0 && a % 4 == 0)
        hipLaunchKernelGGL(verify_kernel<uint32_t>, grid, block, 0, s, msg, N, p.k, p.m, key);
    else
        hipLaunchKernelGGL(verify_kernel<uint8_t>, grid, block, 0, s, msg, N, p.k, p.m, key);
    return hipGetLastError();
}

} // namespace qrm
