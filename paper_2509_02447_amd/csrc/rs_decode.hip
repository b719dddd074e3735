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
#include "qrm_internal.h"

namespace qrm {

namespace {

// ---- the table image of a code, in global memory and (the same bytes) in LDS
constexpr int kZeroLog = 512;                 // log of zero: any sum with it indexes the zeros of the antilog table
constexpr int kExpBytes = 1056;               // antilogs of 0 .. 2 ord - 1, then zeros up to 2 kZeroLog
constexpr int kLogAt = kExpBytes;             // u16 [256]
constexpr int kQuadAt = kLogAt + 512;         // u8 [256]: a y with y^2 + y = index, 0 when there is none
constexpr int kCodeAt = kQuadAt + 256;        // what follows depends on the kernel:
//   lane kernel : u32 [4 ceil(n/4)][q], the (up to four) syndrome terms of symbol value v at position i, a byte each
//   group kernel: u8 [2t + t][q], v * alpha^(G (fcr + j)) for j < 2t, then v * alpha^(G j) for j = 1 .. t
constexpr int kMaxGroupTables = 24 * 256;
constexpr int64_t kDecodeBlocks = 2048; // lane kernel: eight workgroups per compute unit; each reads the tables once and takes every 2048th run of words
// Group kernel: its 56 .. 80 registers let six to eight workgroups onto a compute unit, so 2048 left some waiting for a second
// turn and others with a second run of words while the rest of the chip was done.  Five per compute unit, and every workgroup
// the same number of runs: 20000 words of RS(255,239) 50.2 -> 37.1 us, 65536 of them 117 -> 110, 100000 of RS(63,55) 37.6 ->
// 31.0, 400000 of RS(31,25) 78.8 -> 69.8, up to 13000 words unchanged; with 1024, 1536 and 2048 runs dealt evenly 45, 37 and 37
// us for the first, 113, 152 and 117 for the second.
constexpr int64_t kGroupBlocks = 1280;

bool lane_code(int n, int two_t) { return n <= 16 && two_t <= 4; }
int group_lanes(int two_t) { return two_t > 8 ? 32 : 16; } // 3t + 1 coefficients of the systolic recursion, one per lane
// Words of more than 128 symbols keep 16 lanes busy for 16 steps one after the other, which shows where a launch has so few
// of them that every workgroup takes one run: while 32 lanes a word still fit the chip that way, they have 32.  RS(255,251),
// 300 words 11.4 -> 7.8 us, 4096 11.7 -> 8.8, 8192 12.8 -> 10.6; RS(255,247) 14.3 -> 9.7, 14.7 -> 10.7, 15.7 -> 12.5; 20000
// words are 16.9 us with 16 lanes and 17.1 with 32, 21.1 and 22.3.
bool second_split(int n, int two_t) { return n > 128 && two_t <= 8; }
bool takes_second_split(const RsParams &p, int64_t N) { return second_split(p.n, p.two_t) && N <= kGroupBlocks * (256 / 32); }

struct Gf {
    const uint8_t *exp; // LDS
    const uint16_t *lg; // LDS
    __device__ __forceinline__ int E(int i) const { return exp[i]; }
    __device__ __forceinline__ int L(int a) const { return lg[a]; }
};

__device__ __forceinline__ int mod_once(int e, int ord) { return (int)min((uint32_t)e, (uint32_t)(e - ord)); } // 0 <= e < 2 ord

// table image -> LDS, 16 bytes per lane and step
__device__ __forceinline__ void load_tables(uint8_t *dst, const RsParams &p)
{
    for (int i = threadIdx.x * 16; i < p.tab_bytes; i += 256 * 16) *(u32x4 *)(dst + i) = *(const u32x4 *)(p.tab + i);
}

// ------------------------------------------------------------------------------------------------
// Short codes with t <= 2: one word per lane, nothing repeated across lanes, no serial recursion.
// A lane holds its word as packed bytes (N4 = ceil(n/4) dwords).  The syndromes of a symbol at its position are ONE
// 32-bit look-up (all four in it), so the whole syndrome computation is n look-ups and n XORs.  From S0 .. S3:
//   all zero                              no error
//   D = S1^2 + S0 S2 = 0                  one error, X = S1 / S0, if S1 S2 = S0 S3 (and S0, S1 are not zero)
//   D != 0                                two errors: sigma1 = (S1 S2 + S0 S3) / D, sigma2 = (S2^2 + S1 S3) / D,
//                                         X = sigma1 y with y^2 + y = sigma2 / sigma1^2 from a table
// and a locator outside the word, a double root or a vanishing sigma is an uncorrectable word: the same words, as
// these are exactly the cases in which the shortest recursion for S has length 1 or 2 and distinct roots.  t = 1
// is the one-error branch with S0, S1 alone.
// Bound by vector instructions and LDS look-ups, about 200 and 40 per word, close to what the bytes alone take.
// 2^20 words of RS(12,8) over GF(256), 34.6 MB: 12.5 us a pass = 2.8 TB/s (a
// recursion per lane with byte-wise loads: 44.5 us); what is left is mostly the launch and the first touch of the tables.
// WORDS: words and messages are whole aligned dwords, read and written straight from global memory; otherwise a
// workgroup's 256 words pass through LDS so that global memory is still accessed in dwords.
// ------------------------------------------------------------------------------------------------
template <int N4, bool WORDS>
__global__ __launch_bounds__(256) void rs_decode_lane_kernel(RsParams p, const uint8_t *__restrict__ sym, int64_t N,
                                                             uint8_t *__restrict__ msg, uint8_t *__restrict__ cw,
                                                             int8_t *__restrict__ nerr, KeyArgs key)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t s_tab[];
    __shared__ __attribute__((aligned(16))) uint8_t s_word[WORDS ? 16 : 256 * 16 + 16];
    __shared__ __attribute__((aligned(16))) uint8_t s_msg[WORDS ? 16 : 256 * 16];
    const int tid = threadIdx.x;
    const int n = p.n, k = p.k, ord = p.q - 1, fcr = p.fcr;
    load_tables(s_tab, p);
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

    const int64_t blocks = (N + 255) / 256;
    for (int64_t b = blockIdx.x; b < blocks; b += gridDim.x) {
        const int64_t w0 = b * 256;
        const int cnt = (int)min((int64_t)256, N - w0);
        const bool mine = tid < cnt;
        const int64_t w = w0 + (mine ? tid : 0);
        uint32_t r[N4];
        if (WORDS) {
            const uint32_t *src = (const uint32_t *)(sym + w * n);
#pragma unroll
            for (int j = 0; j < N4; ++j) r[j] = src[j];
        } else {
            const uint8_t *src = sym + w0 * n;
            const int bytes = cnt * n;
            if (((uintptr_t)sym & 3) == 0) { // 256 n is a multiple of four: every workgroup's run is aligned as the first
                for (int i = tid; i < bytes >> 2; i += 256) ((uint32_t *)s_word)[i] = ((const uint32_t *)src)[i];
                if (tid < (bytes & 3)) s_word[(bytes & ~3) + tid] = src[(bytes & ~3) + tid];
            } else {
                for (int i = tid; i < bytes; i += 256) s_word[i] = src[i];
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

        // ---- syndromes, a byte each
        uint32_t S = 0;
#pragma unroll
        for (int i = 0; i < 4 * N4; ++i) S ^= syn[i * p.q + ((r[i / 4] >> (8 * (i % 4))) & 0xffu)];
        const int S0 = S & 0xff, S1 = (S >> 8) & 0xff;
        const int l0 = gf.L(S0), l1 = gf.L(S1);
        int D = 0, lA = kZeroLog, lB = kZeroLog;
        bool one_ok = S0 && S1;
        if (p.two_t == 4) {
            const int l2 = gf.L((S >> 16) & 0xff), l3 = gf.L(S >> 24);
            D = gf.E(l1 + l1) ^ gf.E(l0 + l2);
            const int A = gf.E(l1 + l2) ^ gf.E(l0 + l3), B = gf.E(l2 + l2) ^ gf.E(l1 + l3);
            one_ok = one_ok && A == 0;
            lA = gf.L(A);
            lB = gf.L(B);
        }
        // ---- locators (as powers p1, p2) and alpha^(fcr p) weighted error values a1, a2
        int L, p1, p2 = 0, a1, a2 = 0;
        bool ok;
        if (D == 0) {
            L = S ? 1 : 0;
            ok = S == 0 || one_ok;
            p1 = one_ok ? mod_once(l1 - l0 + ord, ord) : 0;
            a1 = S0;
        } else {
            L = 2;
            ok = lA != kZeroLog && lB != kZeroLog;
            const int lD = gf.L(D);
            int e = ok ? lB + lD - 2 * lA + 2 * ord : 0; // log (sigma2 / sigma1^2), below 4 ord
            e = mod_once(e, 2 * ord);
            const int y = quad[gf.E(e)];
            ok = ok && y != 0;
            const int ls = ok ? mod_once(lA - lD + ord, ord) : 0; // log sigma1
            const int X1 = gf.E(ls + gf.L(y)), X2 = X1 ^ gf.E(ls);
            p1 = gf.L(X1);
            p2 = gf.L(X2);
            a2 = gf.E(gf.L(S1 ^ gf.E(p1 + l0)) + ord - ls); // (S1 + X1 S0) / (X1 + X2)
            a1 = S0 ^ a2;
            ok = ok && p2 < n;
        }
        ok = ok && p1 < n;
        if (ok && L > 0) {
            auto fix = [&](int pw, int a) {
                int e = pw; // error value = a * alpha^(- fcr pw)
                if (fcr != 1) e = (int)(__umul24((uint32_t)fcr, (uint32_t)pw) % (uint32_t)ord);
                const int i = n - 1 - pw;
                const uint32_t v = (uint32_t)gf.E(gf.L(a) + ord - e) << (8 * (i & 3));
#pragma unroll
                for (int j = 0; j < N4; ++j) r[j] ^= (i >> 2) == j ? v : 0u;
            };
            fix(p1, a1);
            if (L == 2) fix(p2, a2);
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
                    for (int i = tid; i < bytes >> 2; i += 256) ((uint32_t *)dst)[i] = ((const uint32_t *)from)[i];
                    if (tid < (bytes & 3)) dst[(bytes & ~3) + tid] = from[(bytes & ~3) + tid];
                } else {
                    for (int i = tid; i < bytes; i += 256) dst[i] = from[i];
                }
            };
            if (cw) copy_out(cw + w0 * n, s_word, cnt * n);
            copy_out(msg + w0 * k, s_msg, cnt * k);
            __syncthreads();
        }
        if (mine) {
            nerr[w] = (int8_t)(ok ? L : -1);
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
//   Syndromes   each lane evaluates its own symbols by Horner's rule in alpha^(G (fcr + j)): a step is one look-up in
//               that constant's table (256 bytes: one dword per LDS bank, so no bank conflicts) and one XOR for
//               each j; the lane's own power is multiplied on at the end and the terms are added up over the lanes.
//   Recursion   Berlekamp-Massey without inversions in its systolic form (the "RiBM" of Sarwate and Shanbhag): lane i
//               holds coefficient i of the 3t + 1 of one polynomial, an iteration is two products per lane and a
//               shift by one lane, and at the end lanes t .. 2t hold the locator Lambda and lanes 0 .. t-1 the
//               high part Omega_h of Lambda S = Omega + x^(2t) Omega_h.  It replaces a recursion that every lane
//               repeated over all coefficients: 2t (3t + 2) products per lane are now 4t.
//   Chien       every lane steps through its positions; the terms Lambda_j x^j and Omega_h,j x^j are carried along,
//               each multiplied by alpha^(G j) per step.
//   Forney      error value X^(-fcr-2t) Omega_h(1/X) / (sum of the odd terms of Lambda at 1/X); Omega(1/X) equals
//               X^(-2t) Omega_h(1/X) because Lambda(1/X) = 0.
// A wavefront whose words are all error free stops after the syndromes.
// Bound by vector instructions and LDS look-ups; 20000 words of RS(255,239): 37 us a pass (the recursion
// repeated on all 64 lanes of a word: 388 us).
// ------------------------------------------------------------------------------------------------
template <int G>
__device__ __forceinline__ uint32_t group_xor(uint32_t v)
{
#pragma unroll
    for (int off = G / 2; off >= 1; off >>= 1) v ^= (uint32_t)__shfl_xor((int)v, off, G);
    return v;
}

template <int G>
__device__ __forceinline__ uint32_t group_mask(bool pred, int lane) // lanes of this lane's group where pred holds
{
    const unsigned long long mask = __ballot(pred);
    return (uint32_t)(mask >> (lane / G * G)) & (uint32_t)((1ull << G) - 1ull);
}

// The value of the lane above within the group; the top lane gets `fill`.
template <int G>
__device__ __forceinline__ int from_above(int v, int fill, int lane_g)
{
    if (G == 16) return __builtin_amdgcn_update_dpp(fill, v, 0x101, 0xf, 0xf, false); // row_shl:1
    const int up = __shfl_down(v, 1);
    return lane_g == G - 1 ? fill : up;
}

// The value of the group's lane 0.
template <int G>
__device__ __forceinline__ int from_first(int v, int lane)
{
    if (G == 16) return __builtin_amdgcn_update_dpp(0, v, 0x150, 0xf, 0xf, false); // row_newbcast:0
    const int a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 32);
    return lane < 32 ? a : b;
}

template <int G, int TMAX, int SPL>
__global__ __launch_bounds__(256) void rs_decode_group_kernel(RsParams p, const uint8_t *__restrict__ sym, int64_t N,
                                                              uint8_t *__restrict__ msg, uint8_t *__restrict__ cw,
                                                              int8_t *__restrict__ nerr, KeyArgs key)
{
    static_assert(3 * TMAX + 1 <= G, "one lane per coefficient");
    __shared__ __attribute__((aligned(16))) uint8_t s_tab[kCodeAt + kMaxGroupTables];
    __shared__ uint8_t s_key[256];
    const int tid = threadIdx.x, lane = tid & 63, l = tid % G;
    const int n = p.n, k = p.k, ord = p.q - 1, q = p.q, two_t = p.two_t, t = p.two_t / 2;
    const bool with_key = key.matches != nullptr;
    load_tables(s_tab, p);
    s_key[tid] = (with_key && tid < k) ? key.key[tid] : 0;
    __syncthreads();
    const Gf gf{s_tab, (const uint16_t *)(s_tab + kLogAt)};
    const uint8_t *mul_syn = s_tab + kCodeAt, *mul_chien = mul_syn + two_t * q - q; // + j q: times alpha^(G j)

    // this lane's fixed exponents: its last symbol's power (as an exponent of alpha) and where Chien starts
    const int last_pw = ((n - 1 - l - G * (SPL - 1)) % ord + ord) % ord;
    const int first_x = ((l - (n - 1)) % ord + ord) % ord; // exponent of x = alpha^(-power) at symbol l
    const int last_e0 = (int)((uint32_t)(p.fcr * last_pw) % (uint32_t)ord);
    const int lift = (p.fcr + two_t) % ord;                // X^(-fcr-2t) = x^(fcr+2t)
    const int lift0 = (int)((uint32_t)(lift * first_x) % (uint32_t)ord), lift_step = (int)((uint32_t)(lift * G) % (uint32_t)ord);

    constexpr int GPB = 256 / G; // words per workgroup and iteration
    const int64_t stride = (int64_t)gridDim.x * GPB;
    const int64_t iters = (N + stride - 1) / stride; // the same for every lane: cross-lane operations see full wavefronts
    for (int64_t it = 0; it < iters; ++it) {
        const int64_t w = it * stride + (int64_t)blockIdx.x * GPB + tid / G;
        const bool valid = w < N;
        int r[SPL];
#pragma unroll
        for (int s = 0; s < SPL; ++s) {
            const int i = l + s * G;
            r[s] = (valid && i < n) ? sym[w * n + i] & (q - 1) : 0;
        }
        // ---- syndromes
        constexpr int ND = (2 * TMAX + 3) / 4;
        uint32_t Spk[ND];
#pragma unroll
        for (int d = 0; d < ND; ++d) Spk[d] = 0;
        {
            int e = last_e0;
#pragma unroll
            for (int j = 0; j < 2 * TMAX; ++j)
                if (j < two_t) {
                    int v = r[0];
#pragma unroll
                    for (int s = 1; s < SPL; ++s) v = mul_syn[j * q + v] ^ r[s];
                    Spk[j / 4] |= (uint32_t)gf.E(gf.L(v) + e) << (8 * (j % 4));
                    e = mod_once(e + last_pw, ord);
                }
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
            int delta = 0;
#pragma unroll
            for (int d = 0; d < ND; ++d)
                if ((l >> 2) == d) delta = (int)((Spk[d] >> (8 * (l & 3))) & 0xffu);
            delta = l < two_t ? delta : (l == 3 * t ? 1 : 0);
            int ldelta = gf.L(delta), ltheta = ldelta, lgamma = 0, kk = 0;
            for (int rr = 0; rr < two_t; ++rr) {
                const int up = from_above<G>(ldelta, kZeroLog, l), d0 = from_first<G>(ldelta, lane);
                delta = gf.E(lgamma + up) ^ gf.E(d0 + ltheta);
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

            // ---- Chien: terms at this lane's first position, then stepped
            int lam[TMAX + 1], om[TMAX];
            {
                int e = 0;
#pragma unroll
                for (int j = 0; j <= TMAX; ++j) {
                    lam[j] = 0;
                    if (j < TMAX) om[j] = 0;
                    if (j <= t) {
                        lam[j] = gf.E(__shfl(ldelta, t + j, G) + e);
                        if (j < TMAX) if (j < t) om[j] = gf.E(__shfl(ldelta, j, G) + e);
                        e = mod_once(e + first_x, ord);
                    }
                }
            }
            int nroots = 0;
            bool bad = false;
            int lx = lift0;
            uint32_t ev[(SPL + 3) / 4]; // error values, a byte each
#pragma unroll
            for (int s = 0; s < SPL; ++s) {
                if (s % 4 == 0) ev[s / 4] = 0;
                int odd = 0, even = lam[0], num = om[0];
#pragma unroll
                for (int j = 1; j <= TMAX; ++j) {
                    if (j & 1) odd ^= lam[j];
                    else even ^= lam[j];
                    if (j < TMAX) num ^= om[j];
                }
                const bool root = odd == even && l + s * G < n && !fail && L > 0;
                if (__ballot(root)) {
                    nroots += __popc(group_mask<G>(root, lane));
                    if (root) {
                        bad = bad || odd == 0 || num == 0;
                        const int quot = gf.E(gf.L(num) + (odd ? ord - gf.L(odd) : 0));
                        ev[s / 4] |= (uint32_t)gf.E(gf.L(quot) + lx) << (8 * (s % 4));
                    }
                }
                if (s + 1 < SPL) {
#pragma unroll
                    for (int j = 1; j <= TMAX; ++j)
                        if (j <= t) {
                            lam[j] = mul_chien[j * q + lam[j]];
                            if (j < TMAX) om[j] = mul_chien[j * q + om[j]];
                        }
                    lx = mod_once(lx + lift_step, ord);
                }
            }
            if (nroots != L || group_mask<G>(bad, lane) != 0) fail = true;
            if (!fail) {
#pragma unroll
                for (int s = 0; s < SPL; ++s) r[s] ^= (int)((ev[s / 4] >> (8 * (s % 4))) & 0xffu);
            }
        }

        // ---- write back
        int agree = 0;
#pragma unroll
        for (int s = 0; s < SPL; ++s) {
            const int i = l + s * G;
            if (valid && i < n) {
                if (cw) cw[w * n + i] = (uint8_t)r[s];
                if (i < k) {
                    msg[w * k + i] = (uint8_t)r[s];
                    if (with_key) agree += p.m - __popc((unsigned)(r[s] ^ s_key[i]) & (unsigned)ord);
                }
            }
        }
        if (valid && l == 0) nerr[w] = (int8_t)(fail ? -1 : L);
        if (with_key) {
#pragma unroll
            for (int off = G / 2; off >= 1; off >>= 1) agree += __shfl_xor(agree, off, G);
            if (valid && l == 0) {
                key.matches[w] = agree;
                if (key.detected) key.detected[w] = (uint8_t)(agree >= key.tau);
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
    constexpr int GPB = 256 / G;
    int64_t blocks = (N + GPB - 1) / GPB;
    const int64_t rounds = (blocks + kGroupBlocks - 1) / kGroupBlocks;
    if (rounds > 1) blocks = (blocks + rounds - 1) / rounds;
    hipLaunchKernelGGL((rs_decode_group_kernel<G, TMAX, SPL>), dim3((unsigned)blocks), dim3(256), 0, s, p, sym, N, msg,
                       cw, nerr, key);
    return hipGetLastError();
}

template <int N4>
hipError_t launch_lane(const RsParams &p, const uint8_t *sym, int64_t N, uint8_t *msg, uint8_t *cw, int8_t *nerr,
                       const KeyArgs &key, hipStream_t s)
{
    int64_t blocks = (N + 255) / 256;
    if (blocks > kDecodeBlocks) blocks = kDecodeBlocks;
    const bool words = p.n % 4 == 0 && p.k % 4 == 0 && (((uintptr_t)sym | (uintptr_t)msg | (uintptr_t)cw) & 3) == 0;
    if (words)
        hipLaunchKernelGGL((rs_decode_lane_kernel<N4, true>), dim3((unsigned)blocks), dim3(256), (unsigned)p.tab_bytes, s, p, sym,
                           N, msg, cw, nerr, key);
    else
        hipLaunchKernelGGL((rs_decode_lane_kernel<N4, false>), dim3((unsigned)blocks), dim3(256), (unsigned)p.tab_bytes, s, p, sym,
                           N, msg, cw, nerr, key);
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
        for (int j = 0; j < p.two_t; ++j)
            for (int v = 0; v < q; ++v) img.push_back(mul_pow(v, G * (p.fcr + j)));
        for (int j = 1; j <= p.two_t / 2; ++j)
            for (int v = 0; v < q; ++v) img.push_back(mul_pow(v, G * j));
        img.resize((img.size() + 15) / 16 * 16, 0);
    };
    add_group(group_lanes(p.two_t));
    p.tab_bytes = (int)img.size();
    if (second_split(p.n, p.two_t)) { // a second image behind the first
        img.insert(img.end(), common.begin(), common.end());
        add_group(32);
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
        return launch_group<32, 4, 8>(second, sym, N, msg, cw, nerr, key, s);
    }
    if (group_lanes(p.two_t) == 16) {
        if (p.n <= 16) return launch_group<16, 4, 1>(p, sym, N, msg, cw, nerr, key, s);
        if (p.n <= 32) return launch_group<16, 4, 2>(p, sym, N, msg, cw, nerr, key, s);
        if (p.n <= 64) return launch_group<16, 4, 4>(p, sym, N, msg, cw, nerr, key, s);
        if (p.n <= 128) return launch_group<16, 4, 8>(p, sym, N, msg, cw, nerr, key, s);
        return launch_group<16, 4, 16>(p, sym, N, msg, cw, nerr, key, s);
    }
    if (p.n <= 32) return launch_group<32, 8, 1>(p, sym, N, msg, cw, nerr, key, s);
    if (p.n <= 64) return launch_group<32, 8, 2>(p, sym, N, msg, cw, nerr, key, s);
    if (p.n <= 128) return launch_group<32, 8, 4>(p, sym, N, msg, cw, nerr, key, s);
    return launch_group<32, 8, 8>(p, sym, N, msg, cw, nerr, key, s);
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
