// Reed-Solomon words of up to 16 symbols with t <= 2: what the kernel that decodes a batch of them (rs_decode.hip) and the head of
// the extractor, which decodes the word of its own image (extractor.hip), have in common.
#pragma once

#include "qrm_internal.h"

namespace qrm {

// ---- the table image of a code, in global memory and (the same bytes) in LDS
constexpr int kZeroLog = 512;                 // log of zero: any sum with it indexes the zeros of the antilog table
constexpr int kExpBytes = 1056;               // antilogs of 0 .. 2 ord - 1, then zeros up to 2 kZeroLog
constexpr int kLogAt = kExpBytes;             // u16 [256]
constexpr int kQuadAt = kLogAt + 512;         // u8 [256]: a y with y^2 + y = index, 0 when there is none
constexpr int kCodeAt = kQuadAt + 256;        // what follows depends on the code; for these ones:
//   u32 [4 ceil(n/4)][q], the (up to four) syndrome terms of symbol value v at position i, a byte each

inline bool lane_code(int n, int two_t) { return n <= 16 && two_t <= 4; }

struct Gf {
    const uint8_t *exp; // LDS
    const uint16_t *lg; // LDS
    __device__ __forceinline__ int E(int i) const { return exp[i]; }
    __device__ __forceinline__ int L(int a) const { return lg[a]; }
};

__device__ __forceinline__ int mod_once(int e, int ord) { return (int)min((uint32_t)e, (uint32_t)(e - ord)); } // 0 <= e < 2 ord

// The errors of a word from its syndromes S0 .. S3 (bytes of S; 0 from 2t on):
//   all zero                              no error
//   D = S1^2 + S0 S2 = 0                  one error, X = S1 / S0, if S1 S2 = S0 S3 (and S0, S1 are not zero)
//   D != 0                                two errors: sigma1 = (S1 S2 + S0 S3) / D, sigma2 = (S2^2 + S1 S3) / D,
//                                         X = sigma1 y with y^2 + y = sigma2 / sigma1^2 from a table
// and a locator outside the word, a double root or a vanishing sigma is an uncorrectable word: the same words, as
// these are exactly the cases in which the shortest recursion for S has length 1 or 2 and distinct roots.  t = 1
// is the one-error branch with S0, S1 alone.
struct LaneErrors {
    bool ok;
    int count;
    int p1, p2; // locators as powers: the symbol is n - 1 - p
    int a1, a2; // alpha^(fcr p) weighted error values (lane_error_value)
};

__device__ __forceinline__ LaneErrors lane_errors(const Gf &gf, const uint8_t *quad, uint32_t S, int n, int ord, int two_t)
{
    const int S0 = S & 0xff, S1 = (S >> 8) & 0xff;
    const int l0 = gf.L(S0), l1 = gf.L(S1);
    int D = 0, lA = kZeroLog, lB = kZeroLog;
    bool one_ok = S0 && S1;
    if (two_t == 4) {
        const int l2 = gf.L((S >> 16) & 0xff), l3 = gf.L(S >> 24);
        D = gf.E(l1 + l1) ^ gf.E(l0 + l2);
        const int A = gf.E(l1 + l2) ^ gf.E(l0 + l3), B = gf.E(l2 + l2) ^ gf.E(l1 + l3);
        one_ok = one_ok && A == 0;
        lA = gf.L(A);
        lB = gf.L(B);
    }
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
    return LaneErrors{ok, L, p1, p2, a1, a2};
}

// error value = a * alpha^(- fcr pw)
__device__ __forceinline__ int lane_error_value(const Gf &gf, int pw, int a, int fcr, int ord)
{
    int e = pw;
    if (fcr != 1) e = (int)(__umul24((uint32_t)fcr, (uint32_t)pw) % (uint32_t)ord);
    return gf.E(gf.L(a) + ord - e);
}

} // namespace qrm
