// hb_issue.hpp -- the three compressions ordered for a SIMD that several waves share.
//
// What bounds them: a gfx950 SIMD has two places to run a wave64 VALU instruction.  The
// plain 32-bit ones (v_bitop3_b32, VOP2 v_add_u32 / v_xor_b32: "plain" below) go to
// either, the others this path uses (v_alignbit_b32, v_add3_u32, v_xad_u32, v_perm_b32:
// "wide") to one of them only; each instruction holds its place for four cycles.  Two
// waves can therefore run two instructions at a time, one of them plain, and the least a
// block can take is max(4 wide, 2 (plain + wide)) cycles.  Left to itself the oldest wave
// issues whenever it can, with its plain instructions too, and every other wave ends up
// stopped at its next wide instruction: three plain to one wide, four waves, take 3.3
// cycles an instruction where 2.0 are possible, and the compiler's order of MD5 / SHA-1 /
// SM3 1,319 / 2,403 / 5,294 cycles per wave and block (hb_probe_valu, from registers).
//
// So each round is written as one run of plain instructions and one of wide ones, and a
// wave raises its priority for the wide run: a wave waiting for the wide place then goes
// before the waves that could use the other.  The three-to-one pattern so takes 2.44
// cycles an instruction, and the compressions, from registers at four waves per SIMD,
// 804 (MD5), 1,712 (SHA-1) and 3,704 (SM3) cycles -- 1.64, 1.40 and 1.43 times as fast; at
// eight waves 764, 1,603 and 3,523 (the least possible: 648, about 1,350 and 2,950).  Two
// places working also draw more power: over milliseconds the engine clock falls from 2.37
// to 2.05-2.15 GHz, so kernels gain less than the cycles say.
//
// The choice of instructions follows from the same two bounds: of the sums that could be
// one wide v_add3_u32 / v_xad_u32 or two plain instructions, each round takes as many wide
// ones as keep 4 wide <= 2 (plain + wide): MD5 one (3 plain + 2 wide a step), SHA-1 one of
// two (5 + 4 a round), SM3 two of four (12 + 12 a round with its expansion).  Written the
// other way they were slower by, MD5 without v_add3_u32 24 %, SHA-1 without 12, SM3 without
// v_xad_u32 9.
//
// What a kernel does between two blocks -- loads, realignment and byte reversal, v_perm_b32
// being wide -- runs at the raised priority too, so that a wave gets its next loads out: each
// function starts with a plain run and ends at the raised priority (2^22 SM3 messages of 0 to
// 4,096 bytes: 4,849 us when it ended at the plain one, 4,688 so).
//
// A wave alone on its SIMD issues one instruction per four cycles or slower whatever its
// kind, so there the two priority changes a round only cost (MD5 1,896 against 1,385
// cycles): launches of at most one wave per SIMD take compress<A> instead.
//
// Each function is one asm block: the order is the point, and the compiler neither keeps
// an order it is given nor knows these rules.  No memory is touched and nothing waits.
#pragma once

#include "hb_device.hpp"

namespace hb {

#define HB_TT_XOR3 "0x96"  // x ^ y ^ z
#define HB_TT_MAJ "0xe8"   // majority
#define HB_TT_CH "0xca"    // x ? y : z
#define HB_TT_G "0xe4"     // z ? x : y
#define HB_TT_I "0x39"     // y ^ (x | ~z)
static_assert(TT_XOR3 == 0x96 && TT_MAJ == 0xe8 && TT_CH == 0xca && TT_MD5_G == 0xe4 && TT_MD5_I == 0x39,
              "bitop3 tables as spelled in the asm below");

#define HB_WIDE "s_setprio 1\n\t"   // a run of wide instructions follows
#define HB_PLAIN "s_setprio 0\n\t"  // a run of plain instructions follows

// ---------------------------------------------------------------------------------------
// MD5 (RFC 1321 Sec. 3.4): a = b + ((a + F(b, c, d) + X[k] + T) <<< s), s given as 32 - s
// ---------------------------------------------------------------------------------------

#define HB_MD5_I(a, b, c, d, w, s, T, F)                                                      \
    "v_add_u32 %[" #a "], " #T ", %[" #a "]\n\t"                                              \
    "v_bitop3_b32 %[t], %[" #b "], %[" #c "], %[" #d "] bitop3:" F "\n\t"                     \
    HB_WIDE                                                                                   \
    "v_add3_u32 %[" #a "], %[" #a "], %[t], %[" #w "]\n\t"                                    \
    "v_alignbit_b32 %[" #a "], %[" #a "], %[" #a "], " #s "\n\t"                              \
    HB_PLAIN                                                                                  \
    "v_add_u32 %[" #a "], %[" #a "], %[" #b "]\n\t"

__device__ __forceinline__ void md5_compress_many(uint32_t s[8], const uint32_t X[16])
{
    uint32_t a = s[0], b = s[1], c = s[2], d = s[3], t;
    asm volatile(HB_PLAIN
        HB_MD5_I(a, b, c, d, w0, 25, 0xd76aa478, HB_TT_CH)
        HB_MD5_I(d, a, b, c, w1, 20, 0xe8c7b756, HB_TT_CH)
        HB_MD5_I(c, d, a, b, w2, 15, 0x242070db, HB_TT_CH)
        HB_MD5_I(b, c, d, a, w3, 10, 0xc1bdceee, HB_TT_CH)
        HB_MD5_I(a, b, c, d, w4, 25, 0xf57c0faf, HB_TT_CH)
        HB_MD5_I(d, a, b, c, w5, 20, 0x4787c62a, HB_TT_CH)
        HB_MD5_I(c, d, a, b, w6, 15, 0xa8304613, HB_TT_CH)
        HB_MD5_I(b, c, d, a, w7, 10, 0xfd469501, HB_TT_CH)
        HB_MD5_I(a, b, c, d, w8, 25, 0x698098d8, HB_TT_CH)
        HB_MD5_I(d, a, b, c, w9, 20, 0x8b44f7af, HB_TT_CH)
        HB_MD5_I(c, d, a, b, w10, 15, 0xffff5bb1, HB_TT_CH)
        HB_MD5_I(b, c, d, a, w11, 10, 0x895cd7be, HB_TT_CH)
        HB_MD5_I(a, b, c, d, w12, 25, 0x6b901122, HB_TT_CH)
        HB_MD5_I(d, a, b, c, w13, 20, 0xfd987193, HB_TT_CH)
        HB_MD5_I(c, d, a, b, w14, 15, 0xa679438e, HB_TT_CH)
        HB_MD5_I(b, c, d, a, w15, 10, 0x49b40821, HB_TT_CH)
        HB_MD5_I(a, b, c, d, w1, 27, 0xf61e2562, HB_TT_G)
        HB_MD5_I(d, a, b, c, w6, 23, 0xc040b340, HB_TT_G)
        HB_MD5_I(c, d, a, b, w11, 18, 0x265e5a51, HB_TT_G)
        HB_MD5_I(b, c, d, a, w0, 12, 0xe9b6c7aa, HB_TT_G)
        HB_MD5_I(a, b, c, d, w5, 27, 0xd62f105d, HB_TT_G)
        HB_MD5_I(d, a, b, c, w10, 23, 0x02441453, HB_TT_G)
        HB_MD5_I(c, d, a, b, w15, 18, 0xd8a1e681, HB_TT_G)
        HB_MD5_I(b, c, d, a, w4, 12, 0xe7d3fbc8, HB_TT_G)
        HB_MD5_I(a, b, c, d, w9, 27, 0x21e1cde6, HB_TT_G)
        HB_MD5_I(d, a, b, c, w14, 23, 0xc33707d6, HB_TT_G)
        HB_MD5_I(c, d, a, b, w3, 18, 0xf4d50d87, HB_TT_G)
        HB_MD5_I(b, c, d, a, w8, 12, 0x455a14ed, HB_TT_G)
        HB_MD5_I(a, b, c, d, w13, 27, 0xa9e3e905, HB_TT_G)
        HB_MD5_I(d, a, b, c, w2, 23, 0xfcefa3f8, HB_TT_G)
        HB_MD5_I(c, d, a, b, w7, 18, 0x676f02d9, HB_TT_G)
        HB_MD5_I(b, c, d, a, w12, 12, 0x8d2a4c8a, HB_TT_G)
        HB_MD5_I(a, b, c, d, w5, 28, 0xfffa3942, HB_TT_XOR3)
        HB_MD5_I(d, a, b, c, w8, 21, 0x8771f681, HB_TT_XOR3)
        HB_MD5_I(c, d, a, b, w11, 16, 0x6d9d6122, HB_TT_XOR3)
        HB_MD5_I(b, c, d, a, w14, 9, 0xfde5380c, HB_TT_XOR3)
        HB_MD5_I(a, b, c, d, w1, 28, 0xa4beea44, HB_TT_XOR3)
        HB_MD5_I(d, a, b, c, w4, 21, 0x4bdecfa9, HB_TT_XOR3)
        HB_MD5_I(c, d, a, b, w7, 16, 0xf6bb4b60, HB_TT_XOR3)
        HB_MD5_I(b, c, d, a, w10, 9, 0xbebfbc70, HB_TT_XOR3)
        HB_MD5_I(a, b, c, d, w13, 28, 0x289b7ec6, HB_TT_XOR3)
        HB_MD5_I(d, a, b, c, w0, 21, 0xeaa127fa, HB_TT_XOR3)
        HB_MD5_I(c, d, a, b, w3, 16, 0xd4ef3085, HB_TT_XOR3)
        HB_MD5_I(b, c, d, a, w6, 9, 0x04881d05, HB_TT_XOR3)
        HB_MD5_I(a, b, c, d, w9, 28, 0xd9d4d039, HB_TT_XOR3)
        HB_MD5_I(d, a, b, c, w12, 21, 0xe6db99e5, HB_TT_XOR3)
        HB_MD5_I(c, d, a, b, w15, 16, 0x1fa27cf8, HB_TT_XOR3)
        HB_MD5_I(b, c, d, a, w2, 9, 0xc4ac5665, HB_TT_XOR3)
        HB_MD5_I(a, b, c, d, w0, 26, 0xf4292244, HB_TT_I)
        HB_MD5_I(d, a, b, c, w7, 22, 0x432aff97, HB_TT_I)
        HB_MD5_I(c, d, a, b, w14, 17, 0xab9423a7, HB_TT_I)
        HB_MD5_I(b, c, d, a, w5, 11, 0xfc93a039, HB_TT_I)
        HB_MD5_I(a, b, c, d, w12, 26, 0x655b59c3, HB_TT_I)
        HB_MD5_I(d, a, b, c, w3, 22, 0x8f0ccc92, HB_TT_I)
        HB_MD5_I(c, d, a, b, w10, 17, 0xffeff47d, HB_TT_I)
        HB_MD5_I(b, c, d, a, w1, 11, 0x85845dd1, HB_TT_I)
        HB_MD5_I(a, b, c, d, w8, 26, 0x6fa87e4f, HB_TT_I)
        HB_MD5_I(d, a, b, c, w15, 22, 0xfe2ce6e0, HB_TT_I)
        HB_MD5_I(c, d, a, b, w6, 17, 0xa3014314, HB_TT_I)
        HB_MD5_I(b, c, d, a, w13, 11, 0x4e0811a1, HB_TT_I)
        HB_MD5_I(a, b, c, d, w4, 26, 0xf7537e82, HB_TT_I)
        HB_MD5_I(d, a, b, c, w11, 22, 0xbd3af235, HB_TT_I)
        HB_MD5_I(c, d, a, b, w2, 17, 0x2ad7d2bb, HB_TT_I)
        HB_MD5_I(b, c, d, a, w9, 11, 0xeb86d391, HB_TT_I)
        HB_WIDE
        : [a] "+v"(a), [b] "+v"(b), [c] "+v"(c), [d] "+v"(d), [t] "=&v"(t)
        : [w0] "v"(X[0]), [w1] "v"(X[1]), [w2] "v"(X[2]), [w3] "v"(X[3]), [w4] "v"(X[4]), [w5] "v"(X[5]),
          [w6] "v"(X[6]), [w7] "v"(X[7]), [w8] "v"(X[8]), [w9] "v"(X[9]), [w10] "v"(X[10]), [w11] "v"(X[11]),
          [w12] "v"(X[12]), [w13] "v"(X[13]), [w14] "v"(X[14]), [w15] "v"(X[15]));
    s[0] += a; s[1] += b; s[2] += c; s[3] += d;
}

// ---------------------------------------------------------------------------------------
// SHA-1 (FIPS 180-4 Sec. 6.1.2): e += (a <<< 5) + f(b, c, d) + K + W, b <<<= 30; the
// schedule word is formed in its slot of the 16-word window in the round that uses it
// ---------------------------------------------------------------------------------------

#define HB_SHA1_PLAIN(b, c, d, e, k, F)                                                       \
    "v_add_u32 %[" #e "], %[" #k "], %[" #e "]\n\t"                                           \
    "v_bitop3_b32 %[f], %[" #b "], %[" #c "], %[" #d "] bitop3:" F "\n\t"                     \
    "v_add_u32 %[" #e "], %[" #e "], %[f]\n\t"
#define HB_SHA1_WIDE(a, b, e, w)                                                              \
    "v_alignbit_b32 %[u], %[" #a "], %[" #a "], 27\n\t"                                       \
    "v_alignbit_b32 %[" #b "], %[" #b "], %[" #b "], 2\n\t"                                   \
    "v_add3_u32 %[" #e "], %[" #e "], %[u], %[" #w "]\n\t"                                    \
    HB_PLAIN
#define HB_SHA1_I(a, b, c, d, e, w, k, F) HB_SHA1_PLAIN(b, c, d, e, k, F) HB_WIDE HB_SHA1_WIDE(a, b, e, w)
#define HB_SHA1_X(a, b, c, d, e, w, w3, w8, w14, k, F)                                        \
    "v_bitop3_b32 %[" #w "], %[" #w "], %[" #w3 "], %[" #w8 "] bitop3:" HB_TT_XOR3 "\n\t"     \
    "v_xor_b32 %[" #w "], %[" #w "], %[" #w14 "]\n\t"                                         \
    HB_SHA1_PLAIN(b, c, d, e, k, F) HB_WIDE                                                   \
    "v_alignbit_b32 %[" #w "], %[" #w "], %[" #w "], 31\n\t"                                  \
    HB_SHA1_WIDE(a, b, e, w)

__device__ __forceinline__ void sha1_compress_many(uint32_t s[8], const uint32_t M[16])
{
    uint32_t W[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) W[t] = M[t];
    uint32_t a = s[0], b = s[1], c = s[2], d = s[3], e = s[4], f, u;
    asm volatile(HB_PLAIN
        HB_SHA1_I(a, b, c, d, e, w0, k0, HB_TT_CH)
        HB_SHA1_I(e, a, b, c, d, w1, k0, HB_TT_CH)
        HB_SHA1_I(d, e, a, b, c, w2, k0, HB_TT_CH)
        HB_SHA1_I(c, d, e, a, b, w3, k0, HB_TT_CH)
        HB_SHA1_I(b, c, d, e, a, w4, k0, HB_TT_CH)
        HB_SHA1_I(a, b, c, d, e, w5, k0, HB_TT_CH)
        HB_SHA1_I(e, a, b, c, d, w6, k0, HB_TT_CH)
        HB_SHA1_I(d, e, a, b, c, w7, k0, HB_TT_CH)
        HB_SHA1_I(c, d, e, a, b, w8, k0, HB_TT_CH)
        HB_SHA1_I(b, c, d, e, a, w9, k0, HB_TT_CH)
        HB_SHA1_I(a, b, c, d, e, w10, k0, HB_TT_CH)
        HB_SHA1_I(e, a, b, c, d, w11, k0, HB_TT_CH)
        HB_SHA1_I(d, e, a, b, c, w12, k0, HB_TT_CH)
        HB_SHA1_I(c, d, e, a, b, w13, k0, HB_TT_CH)
        HB_SHA1_I(b, c, d, e, a, w14, k0, HB_TT_CH)
        HB_SHA1_I(a, b, c, d, e, w15, k0, HB_TT_CH)
        HB_SHA1_X(e, a, b, c, d, w0, w13, w8, w2, k0, HB_TT_CH)
        HB_SHA1_X(d, e, a, b, c, w1, w14, w9, w3, k0, HB_TT_CH)
        HB_SHA1_X(c, d, e, a, b, w2, w15, w10, w4, k0, HB_TT_CH)
        HB_SHA1_X(b, c, d, e, a, w3, w0, w11, w5, k0, HB_TT_CH)
        HB_SHA1_X(a, b, c, d, e, w4, w1, w12, w6, k1, HB_TT_XOR3)
        HB_SHA1_X(e, a, b, c, d, w5, w2, w13, w7, k1, HB_TT_XOR3)
        HB_SHA1_X(d, e, a, b, c, w6, w3, w14, w8, k1, HB_TT_XOR3)
        HB_SHA1_X(c, d, e, a, b, w7, w4, w15, w9, k1, HB_TT_XOR3)
        HB_SHA1_X(b, c, d, e, a, w8, w5, w0, w10, k1, HB_TT_XOR3)
        HB_SHA1_X(a, b, c, d, e, w9, w6, w1, w11, k1, HB_TT_XOR3)
        HB_SHA1_X(e, a, b, c, d, w10, w7, w2, w12, k1, HB_TT_XOR3)
        HB_SHA1_X(d, e, a, b, c, w11, w8, w3, w13, k1, HB_TT_XOR3)
        HB_SHA1_X(c, d, e, a, b, w12, w9, w4, w14, k1, HB_TT_XOR3)
        HB_SHA1_X(b, c, d, e, a, w13, w10, w5, w15, k1, HB_TT_XOR3)
        HB_SHA1_X(a, b, c, d, e, w14, w11, w6, w0, k1, HB_TT_XOR3)
        HB_SHA1_X(e, a, b, c, d, w15, w12, w7, w1, k1, HB_TT_XOR3)
        HB_SHA1_X(d, e, a, b, c, w0, w13, w8, w2, k1, HB_TT_XOR3)
        HB_SHA1_X(c, d, e, a, b, w1, w14, w9, w3, k1, HB_TT_XOR3)
        HB_SHA1_X(b, c, d, e, a, w2, w15, w10, w4, k1, HB_TT_XOR3)
        HB_SHA1_X(a, b, c, d, e, w3, w0, w11, w5, k1, HB_TT_XOR3)
        HB_SHA1_X(e, a, b, c, d, w4, w1, w12, w6, k1, HB_TT_XOR3)
        HB_SHA1_X(d, e, a, b, c, w5, w2, w13, w7, k1, HB_TT_XOR3)
        HB_SHA1_X(c, d, e, a, b, w6, w3, w14, w8, k1, HB_TT_XOR3)
        HB_SHA1_X(b, c, d, e, a, w7, w4, w15, w9, k1, HB_TT_XOR3)
        HB_SHA1_X(a, b, c, d, e, w8, w5, w0, w10, k2, HB_TT_MAJ)
        HB_SHA1_X(e, a, b, c, d, w9, w6, w1, w11, k2, HB_TT_MAJ)
        HB_SHA1_X(d, e, a, b, c, w10, w7, w2, w12, k2, HB_TT_MAJ)
        HB_SHA1_X(c, d, e, a, b, w11, w8, w3, w13, k2, HB_TT_MAJ)
        HB_SHA1_X(b, c, d, e, a, w12, w9, w4, w14, k2, HB_TT_MAJ)
        HB_SHA1_X(a, b, c, d, e, w13, w10, w5, w15, k2, HB_TT_MAJ)
        HB_SHA1_X(e, a, b, c, d, w14, w11, w6, w0, k2, HB_TT_MAJ)
        HB_SHA1_X(d, e, a, b, c, w15, w12, w7, w1, k2, HB_TT_MAJ)
        HB_SHA1_X(c, d, e, a, b, w0, w13, w8, w2, k2, HB_TT_MAJ)
        HB_SHA1_X(b, c, d, e, a, w1, w14, w9, w3, k2, HB_TT_MAJ)
        HB_SHA1_X(a, b, c, d, e, w2, w15, w10, w4, k2, HB_TT_MAJ)
        HB_SHA1_X(e, a, b, c, d, w3, w0, w11, w5, k2, HB_TT_MAJ)
        HB_SHA1_X(d, e, a, b, c, w4, w1, w12, w6, k2, HB_TT_MAJ)
        HB_SHA1_X(c, d, e, a, b, w5, w2, w13, w7, k2, HB_TT_MAJ)
        HB_SHA1_X(b, c, d, e, a, w6, w3, w14, w8, k2, HB_TT_MAJ)
        HB_SHA1_X(a, b, c, d, e, w7, w4, w15, w9, k2, HB_TT_MAJ)
        HB_SHA1_X(e, a, b, c, d, w8, w5, w0, w10, k2, HB_TT_MAJ)
        HB_SHA1_X(d, e, a, b, c, w9, w6, w1, w11, k2, HB_TT_MAJ)
        HB_SHA1_X(c, d, e, a, b, w10, w7, w2, w12, k2, HB_TT_MAJ)
        HB_SHA1_X(b, c, d, e, a, w11, w8, w3, w13, k2, HB_TT_MAJ)
        HB_SHA1_X(a, b, c, d, e, w12, w9, w4, w14, k3, HB_TT_XOR3)
        HB_SHA1_X(e, a, b, c, d, w13, w10, w5, w15, k3, HB_TT_XOR3)
        HB_SHA1_X(d, e, a, b, c, w14, w11, w6, w0, k3, HB_TT_XOR3)
        HB_SHA1_X(c, d, e, a, b, w15, w12, w7, w1, k3, HB_TT_XOR3)
        HB_SHA1_X(b, c, d, e, a, w0, w13, w8, w2, k3, HB_TT_XOR3)
        HB_SHA1_X(a, b, c, d, e, w1, w14, w9, w3, k3, HB_TT_XOR3)
        HB_SHA1_X(e, a, b, c, d, w2, w15, w10, w4, k3, HB_TT_XOR3)
        HB_SHA1_X(d, e, a, b, c, w3, w0, w11, w5, k3, HB_TT_XOR3)
        HB_SHA1_X(c, d, e, a, b, w4, w1, w12, w6, k3, HB_TT_XOR3)
        HB_SHA1_X(b, c, d, e, a, w5, w2, w13, w7, k3, HB_TT_XOR3)
        HB_SHA1_X(a, b, c, d, e, w6, w3, w14, w8, k3, HB_TT_XOR3)
        HB_SHA1_X(e, a, b, c, d, w7, w4, w15, w9, k3, HB_TT_XOR3)
        HB_SHA1_X(d, e, a, b, c, w8, w5, w0, w10, k3, HB_TT_XOR3)
        HB_SHA1_X(c, d, e, a, b, w9, w6, w1, w11, k3, HB_TT_XOR3)
        HB_SHA1_X(b, c, d, e, a, w10, w7, w2, w12, k3, HB_TT_XOR3)
        HB_SHA1_X(a, b, c, d, e, w11, w8, w3, w13, k3, HB_TT_XOR3)
        HB_SHA1_X(e, a, b, c, d, w12, w9, w4, w14, k3, HB_TT_XOR3)
        HB_SHA1_X(d, e, a, b, c, w13, w10, w5, w15, k3, HB_TT_XOR3)
        HB_SHA1_X(c, d, e, a, b, w14, w11, w6, w0, k3, HB_TT_XOR3)
        HB_SHA1_X(b, c, d, e, a, w15, w12, w7, w1, k3, HB_TT_XOR3)
        HB_WIDE
        : [a] "+v"(a), [b] "+v"(b), [c] "+v"(c), [d] "+v"(d), [e] "+v"(e), [f] "=&v"(f), [u] "=&v"(u),
          [w0] "+v"(W[0]), [w1] "+v"(W[1]), [w2] "+v"(W[2]), [w3] "+v"(W[3]), [w4] "+v"(W[4]), [w5] "+v"(W[5]),
          [w6] "+v"(W[6]), [w7] "+v"(W[7]), [w8] "+v"(W[8]), [w9] "+v"(W[9]), [w10] "+v"(W[10]),
          [w11] "+v"(W[11]), [w12] "+v"(W[12]), [w13] "+v"(W[13]), [w14] "+v"(W[14]), [w15] "+v"(W[15])
        : [k0] "s"(0x5a827999u), [k1] "s"(0x6ed9eba1u), [k2] "s"(0x8f1bbcdcu), [k3] "s"(0xca62c1d6u));
    s[0] += a; s[1] += b; s[2] += c; s[3] += d; s[4] += e;
}

// ---------------------------------------------------------------------------------------
// SM3 (GB/T 32905 Sec. 5.3.2-5.3.3).  Round j: the plain run forms A<<<12 + E + T, FF, GG,
// D + FF + W'_j (W'_j = W_j ^ W_{j+4}) and H + W_j; the wide run SS1, TT2 (in H's
// register), TT1 (in D's), the rotations of B, F and TT2 and the next round's A<<<12; the
// last plain instruction P0(TT2).  Woven in, one word a round: W_{j+5} from the window
// (x = W_{j-11} ^ W_{j-4} ^ (W_{j+2} <<< 15), y = (W_{j-8} <<< 7) ^ x ^ W_{j-1}, then
// W_{j+5} = y ^ (x <<< 15) ^ (x <<< 23)), its two rotated words taken a round earlier.
// ---------------------------------------------------------------------------------------

#define HB_SM3_F(a, b, c, d, e, f, g, h, w, w4, k, FF, GG)                                    \
    "v_add_u32 %[s], %[" #k "], %[" #e "]\n\t"                                                \
    "v_bitop3_b32 %[p], %[" #a "], %[" #b "], %[" #c "] bitop3:" FF "\n\t"                    \
    "v_bitop3_b32 %[q], %[" #e "], %[" #f "], %[" #g "] bitop3:" GG "\n\t"                    \
    "v_add_u32 %[s], %[s], %[r]\n\t"                                                          \
    "v_add_u32 %[" #h "], %[" #h "], %[" #w "]\n\t"                                           \
    "v_add_u32 %[" #d "], %[" #d "], %[p]\n\t"                                                \
    "v_xor_b32 %[p], %[" #w "], %[" #w4 "]\n\t"                                               \
    "v_add_u32 %[" #d "], %[" #d "], %[p]\n\t"
#define HB_SM3_F_X(x, y, w16, w9, w6)                                                         \
    "v_bitop3_b32 %[" #x "], %[" #x "], %[" #w16 "], %[" #w9 "] bitop3:" HB_TT_XOR3 "\n\t"    \
    "v_bitop3_b32 %[" #y "], %[" #y "], %[" #x "], %[" #w6 "] bitop3:" HB_TT_XOR3 "\n\t"
#define HB_SM3_H0                                                                             \
    HB_WIDE                                                                                   \
    "v_alignbit_b32 %[s], %[s], %[s], 25\n\t"
#define HB_SM3_H_X(x, w16)                                                                    \
    "v_alignbit_b32 %[" #w16 "], %[" #x "], %[" #x "], 17\n\t"                                \
    "v_alignbit_b32 %[" #x "], %[" #x "], %[" #x "], 9\n\t"
#define HB_SM3_H1(b, d, f, h)                                                                 \
    "v_add3_u32 %[" #h "], %[" #h "], %[q], %[s]\n\t"                                         \
    "v_alignbit_b32 %[" #b "], %[" #b "], %[" #b "], 23\n\t"                                  \
    "v_alignbit_b32 %[" #f "], %[" #f "], %[" #f "], 13\n\t"                                  \
    "v_xad_u32 %[" #d "], %[s], %[r], %[" #d "]\n\t"                                          \
    "v_alignbit_b32 %[q], %[" #h "], %[" #h "], 23\n\t"                                       \
    "v_alignbit_b32 %[s], %[" #h "], %[" #h "], 15\n\t"
#define HB_SM3_H_N(x, y, w3, w13)                                                             \
    "v_alignbit_b32 %[" #x "], %[" #w3 "], %[" #w3 "], 17\n\t"                                \
    "v_alignbit_b32 %[" #y "], %[" #w13 "], %[" #w13 "], 25\n\t"
#define HB_SM3_H2(a) "v_alignbit_b32 %[r], %[" #a "], %[" #a "], 20\n\t"
#define HB_SM3_E(h)                                                                           \
    HB_PLAIN                                                                                  \
    "v_bitop3_b32 %[" #h "], %[" #h "], %[q], %[s] bitop3:" HB_TT_XOR3 "\n\t"
#define HB_SM3_E_X(x, y, w)                                                                   \
    "v_bitop3_b32 %[" #w "], %[" #w "], %[" #x "], %[" #y "] bitop3:" HB_TT_XOR3 "\n\t"

__device__ __forceinline__ void sm3_compress_many(uint32_t s8[8], const uint32_t M[16])
{
    uint32_t W[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) W[t] = M[t];
    uint32_t a = s8[0], b = s8[1], c = s8[2], d = s8[3], e = s8[4], f = s8[5], g = s8[6], h = s8[7];
    uint32_t p, q, r, s, x0, x1, y0, y1;
    // the 48 distinct round constants as scalar operands: 4-byte adds (8-byte literals took 2 %
    // longer)
    asm volatile(
        HB_SM3_H2(a) HB_PLAIN
        HB_SM3_F(a, b, c, d, e, f, g, h, w0, w4, k0, HB_TT_XOR3, HB_TT_XOR3) HB_SM3_H0 HB_SM3_H1(b, d, f, h) HB_SM3_H2(d) HB_SM3_E(h)
        HB_SM3_F(d, a, b, c, h, e, f, g, w1, w5, k1, HB_TT_XOR3, HB_TT_XOR3) HB_SM3_H0 HB_SM3_H1(a, c, e, g) HB_SM3_H2(c) HB_SM3_E(g)
        HB_SM3_F(c, d, a, b, g, h, e, f, w2, w6, k2, HB_TT_XOR3, HB_TT_XOR3) HB_SM3_H0 HB_SM3_H1(d, b, h, f) HB_SM3_H2(b) HB_SM3_E(f)
        HB_SM3_F(b, c, d, a, f, g, h, e, w3, w7, k3, HB_TT_XOR3, HB_TT_XOR3) HB_SM3_H0 HB_SM3_H1(c, a, g, e) HB_SM3_H2(a) HB_SM3_E(e)
        HB_SM3_F(a, b, c, d, e, f, g, h, w4, w8, k4, HB_TT_XOR3, HB_TT_XOR3) HB_SM3_H0 HB_SM3_H1(b, d, f, h) HB_SM3_H2(d) HB_SM3_E(h)
        HB_SM3_F(d, a, b, c, h, e, f, g, w5, w9, k5, HB_TT_XOR3, HB_TT_XOR3) HB_SM3_H0 HB_SM3_H1(a, c, e, g) HB_SM3_H2(c) HB_SM3_E(g)
        HB_SM3_F(c, d, a, b, g, h, e, f, w6, w10, k6, HB_TT_XOR3, HB_TT_XOR3) HB_SM3_H0 HB_SM3_H1(d, b, h, f) HB_SM3_H2(b) HB_SM3_E(f)
        HB_SM3_F(b, c, d, a, f, g, h, e, w7, w11, k7, HB_TT_XOR3, HB_TT_XOR3) HB_SM3_H0 HB_SM3_H1(c, a, g, e) HB_SM3_H2(a) HB_SM3_E(e)
        HB_SM3_F(a, b, c, d, e, f, g, h, w8, w12, k8, HB_TT_XOR3, HB_TT_XOR3) HB_SM3_H0 HB_SM3_H1(b, d, f, h) HB_SM3_H2(d) HB_SM3_E(h)
        HB_SM3_F(d, a, b, c, h, e, f, g, w9, w13, k9, HB_TT_XOR3, HB_TT_XOR3) HB_SM3_H0 HB_SM3_H1(a, c, e, g) HB_SM3_H2(c) HB_SM3_E(g)
        HB_SM3_F(c, d, a, b, g, h, e, f, w10, w14, k10, HB_TT_XOR3, HB_TT_XOR3) HB_SM3_H0 HB_SM3_H1(d, b, h, f) HB_SM3_H_N(x1, y1, w13, w3) HB_SM3_H2(b) HB_SM3_E(f)
        HB_SM3_F(b, c, d, a, f, g, h, e, w11, w15, k11, HB_TT_XOR3, HB_TT_XOR3) HB_SM3_F_X(x1, y1, w0, w7, w10) HB_SM3_H0 HB_SM3_H_X(x1, w0) HB_SM3_H1(c, a, g, e) HB_SM3_H_N(x0, y0, w14, w4) HB_SM3_H2(a) HB_SM3_E(e) HB_SM3_E_X(x1, y1, w0)
        HB_SM3_F(a, b, c, d, e, f, g, h, w12, w0, k12, HB_TT_XOR3, HB_TT_XOR3) HB_SM3_F_X(x0, y0, w1, w8, w11) HB_SM3_H0 HB_SM3_H_X(x0, w1) HB_SM3_H1(b, d, f, h) HB_SM3_H_N(x1, y1, w15, w5) HB_SM3_H2(d) HB_SM3_E(h) HB_SM3_E_X(x0, y0, w1)
        HB_SM3_F(d, a, b, c, h, e, f, g, w13, w1, k13, HB_TT_XOR3, HB_TT_XOR3) HB_SM3_F_X(x1, y1, w2, w9, w12) HB_SM3_H0 HB_SM3_H_X(x1, w2) HB_SM3_H1(a, c, e, g) HB_SM3_H_N(x0, y0, w0, w6) HB_SM3_H2(c) HB_SM3_E(g) HB_SM3_E_X(x1, y1, w2)
        HB_SM3_F(c, d, a, b, g, h, e, f, w14, w2, k14, HB_TT_XOR3, HB_TT_XOR3) HB_SM3_F_X(x0, y0, w3, w10, w13) HB_SM3_H0 HB_SM3_H_X(x0, w3) HB_SM3_H1(d, b, h, f) HB_SM3_H_N(x1, y1, w1, w7) HB_SM3_H2(b) HB_SM3_E(f) HB_SM3_E_X(x0, y0, w3)
        HB_SM3_F(b, c, d, a, f, g, h, e, w15, w3, k15, HB_TT_XOR3, HB_TT_XOR3) HB_SM3_F_X(x1, y1, w4, w11, w14) HB_SM3_H0 HB_SM3_H_X(x1, w4) HB_SM3_H1(c, a, g, e) HB_SM3_H_N(x0, y0, w2, w8) HB_SM3_H2(a) HB_SM3_E(e) HB_SM3_E_X(x1, y1, w4)
        HB_SM3_F(a, b, c, d, e, f, g, h, w0, w4, k32, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w5, w12, w15) HB_SM3_H0 HB_SM3_H_X(x0, w5) HB_SM3_H1(b, d, f, h) HB_SM3_H_N(x1, y1, w3, w9) HB_SM3_H2(d) HB_SM3_E(h) HB_SM3_E_X(x0, y0, w5)
        HB_SM3_F(d, a, b, c, h, e, f, g, w1, w5, k33, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w6, w13, w0) HB_SM3_H0 HB_SM3_H_X(x1, w6) HB_SM3_H1(a, c, e, g) HB_SM3_H_N(x0, y0, w4, w10) HB_SM3_H2(c) HB_SM3_E(g) HB_SM3_E_X(x1, y1, w6)
        HB_SM3_F(c, d, a, b, g, h, e, f, w2, w6, k34, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w7, w14, w1) HB_SM3_H0 HB_SM3_H_X(x0, w7) HB_SM3_H1(d, b, h, f) HB_SM3_H_N(x1, y1, w5, w11) HB_SM3_H2(b) HB_SM3_E(f) HB_SM3_E_X(x0, y0, w7)
        HB_SM3_F(b, c, d, a, f, g, h, e, w3, w7, k35, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w8, w15, w2) HB_SM3_H0 HB_SM3_H_X(x1, w8) HB_SM3_H1(c, a, g, e) HB_SM3_H_N(x0, y0, w6, w12) HB_SM3_H2(a) HB_SM3_E(e) HB_SM3_E_X(x1, y1, w8)
        HB_SM3_F(a, b, c, d, e, f, g, h, w4, w8, k36, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w9, w0, w3) HB_SM3_H0 HB_SM3_H_X(x0, w9) HB_SM3_H1(b, d, f, h) HB_SM3_H_N(x1, y1, w7, w13) HB_SM3_H2(d) HB_SM3_E(h) HB_SM3_E_X(x0, y0, w9)
        HB_SM3_F(d, a, b, c, h, e, f, g, w5, w9, k37, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w10, w1, w4) HB_SM3_H0 HB_SM3_H_X(x1, w10) HB_SM3_H1(a, c, e, g) HB_SM3_H_N(x0, y0, w8, w14) HB_SM3_H2(c) HB_SM3_E(g) HB_SM3_E_X(x1, y1, w10)
        HB_SM3_F(c, d, a, b, g, h, e, f, w6, w10, k38, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w11, w2, w5) HB_SM3_H0 HB_SM3_H_X(x0, w11) HB_SM3_H1(d, b, h, f) HB_SM3_H_N(x1, y1, w9, w15) HB_SM3_H2(b) HB_SM3_E(f) HB_SM3_E_X(x0, y0, w11)
        HB_SM3_F(b, c, d, a, f, g, h, e, w7, w11, k39, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w12, w3, w6) HB_SM3_H0 HB_SM3_H_X(x1, w12) HB_SM3_H1(c, a, g, e) HB_SM3_H_N(x0, y0, w10, w0) HB_SM3_H2(a) HB_SM3_E(e) HB_SM3_E_X(x1, y1, w12)
        HB_SM3_F(a, b, c, d, e, f, g, h, w8, w12, k40, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w13, w4, w7) HB_SM3_H0 HB_SM3_H_X(x0, w13) HB_SM3_H1(b, d, f, h) HB_SM3_H_N(x1, y1, w11, w1) HB_SM3_H2(d) HB_SM3_E(h) HB_SM3_E_X(x0, y0, w13)
        HB_SM3_F(d, a, b, c, h, e, f, g, w9, w13, k41, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w14, w5, w8) HB_SM3_H0 HB_SM3_H_X(x1, w14) HB_SM3_H1(a, c, e, g) HB_SM3_H_N(x0, y0, w12, w2) HB_SM3_H2(c) HB_SM3_E(g) HB_SM3_E_X(x1, y1, w14)
        HB_SM3_F(c, d, a, b, g, h, e, f, w10, w14, k42, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w15, w6, w9) HB_SM3_H0 HB_SM3_H_X(x0, w15) HB_SM3_H1(d, b, h, f) HB_SM3_H_N(x1, y1, w13, w3) HB_SM3_H2(b) HB_SM3_E(f) HB_SM3_E_X(x0, y0, w15)
        HB_SM3_F(b, c, d, a, f, g, h, e, w11, w15, k43, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w0, w7, w10) HB_SM3_H0 HB_SM3_H_X(x1, w0) HB_SM3_H1(c, a, g, e) HB_SM3_H_N(x0, y0, w14, w4) HB_SM3_H2(a) HB_SM3_E(e) HB_SM3_E_X(x1, y1, w0)
        HB_SM3_F(a, b, c, d, e, f, g, h, w12, w0, k44, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w1, w8, w11) HB_SM3_H0 HB_SM3_H_X(x0, w1) HB_SM3_H1(b, d, f, h) HB_SM3_H_N(x1, y1, w15, w5) HB_SM3_H2(d) HB_SM3_E(h) HB_SM3_E_X(x0, y0, w1)
        HB_SM3_F(d, a, b, c, h, e, f, g, w13, w1, k45, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w2, w9, w12) HB_SM3_H0 HB_SM3_H_X(x1, w2) HB_SM3_H1(a, c, e, g) HB_SM3_H_N(x0, y0, w0, w6) HB_SM3_H2(c) HB_SM3_E(g) HB_SM3_E_X(x1, y1, w2)
        HB_SM3_F(c, d, a, b, g, h, e, f, w14, w2, k46, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w3, w10, w13) HB_SM3_H0 HB_SM3_H_X(x0, w3) HB_SM3_H1(d, b, h, f) HB_SM3_H_N(x1, y1, w1, w7) HB_SM3_H2(b) HB_SM3_E(f) HB_SM3_E_X(x0, y0, w3)
        HB_SM3_F(b, c, d, a, f, g, h, e, w15, w3, k47, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w4, w11, w14) HB_SM3_H0 HB_SM3_H_X(x1, w4) HB_SM3_H1(c, a, g, e) HB_SM3_H_N(x0, y0, w2, w8) HB_SM3_H2(a) HB_SM3_E(e) HB_SM3_E_X(x1, y1, w4)
        HB_SM3_F(a, b, c, d, e, f, g, h, w0, w4, k16, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w5, w12, w15) HB_SM3_H0 HB_SM3_H_X(x0, w5) HB_SM3_H1(b, d, f, h) HB_SM3_H_N(x1, y1, w3, w9) HB_SM3_H2(d) HB_SM3_E(h) HB_SM3_E_X(x0, y0, w5)
        HB_SM3_F(d, a, b, c, h, e, f, g, w1, w5, k17, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w6, w13, w0) HB_SM3_H0 HB_SM3_H_X(x1, w6) HB_SM3_H1(a, c, e, g) HB_SM3_H_N(x0, y0, w4, w10) HB_SM3_H2(c) HB_SM3_E(g) HB_SM3_E_X(x1, y1, w6)
        HB_SM3_F(c, d, a, b, g, h, e, f, w2, w6, k18, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w7, w14, w1) HB_SM3_H0 HB_SM3_H_X(x0, w7) HB_SM3_H1(d, b, h, f) HB_SM3_H_N(x1, y1, w5, w11) HB_SM3_H2(b) HB_SM3_E(f) HB_SM3_E_X(x0, y0, w7)
        HB_SM3_F(b, c, d, a, f, g, h, e, w3, w7, k19, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w8, w15, w2) HB_SM3_H0 HB_SM3_H_X(x1, w8) HB_SM3_H1(c, a, g, e) HB_SM3_H_N(x0, y0, w6, w12) HB_SM3_H2(a) HB_SM3_E(e) HB_SM3_E_X(x1, y1, w8)
        HB_SM3_F(a, b, c, d, e, f, g, h, w4, w8, k20, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w9, w0, w3) HB_SM3_H0 HB_SM3_H_X(x0, w9) HB_SM3_H1(b, d, f, h) HB_SM3_H_N(x1, y1, w7, w13) HB_SM3_H2(d) HB_SM3_E(h) HB_SM3_E_X(x0, y0, w9)
        HB_SM3_F(d, a, b, c, h, e, f, g, w5, w9, k21, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w10, w1, w4) HB_SM3_H0 HB_SM3_H_X(x1, w10) HB_SM3_H1(a, c, e, g) HB_SM3_H_N(x0, y0, w8, w14) HB_SM3_H2(c) HB_SM3_E(g) HB_SM3_E_X(x1, y1, w10)
        HB_SM3_F(c, d, a, b, g, h, e, f, w6, w10, k22, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w11, w2, w5) HB_SM3_H0 HB_SM3_H_X(x0, w11) HB_SM3_H1(d, b, h, f) HB_SM3_H_N(x1, y1, w9, w15) HB_SM3_H2(b) HB_SM3_E(f) HB_SM3_E_X(x0, y0, w11)
        HB_SM3_F(b, c, d, a, f, g, h, e, w7, w11, k23, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w12, w3, w6) HB_SM3_H0 HB_SM3_H_X(x1, w12) HB_SM3_H1(c, a, g, e) HB_SM3_H_N(x0, y0, w10, w0) HB_SM3_H2(a) HB_SM3_E(e) HB_SM3_E_X(x1, y1, w12)
        HB_SM3_F(a, b, c, d, e, f, g, h, w8, w12, k24, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w13, w4, w7) HB_SM3_H0 HB_SM3_H_X(x0, w13) HB_SM3_H1(b, d, f, h) HB_SM3_H_N(x1, y1, w11, w1) HB_SM3_H2(d) HB_SM3_E(h) HB_SM3_E_X(x0, y0, w13)
        HB_SM3_F(d, a, b, c, h, e, f, g, w9, w13, k25, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w14, w5, w8) HB_SM3_H0 HB_SM3_H_X(x1, w14) HB_SM3_H1(a, c, e, g) HB_SM3_H_N(x0, y0, w12, w2) HB_SM3_H2(c) HB_SM3_E(g) HB_SM3_E_X(x1, y1, w14)
        HB_SM3_F(c, d, a, b, g, h, e, f, w10, w14, k26, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w15, w6, w9) HB_SM3_H0 HB_SM3_H_X(x0, w15) HB_SM3_H1(d, b, h, f) HB_SM3_H_N(x1, y1, w13, w3) HB_SM3_H2(b) HB_SM3_E(f) HB_SM3_E_X(x0, y0, w15)
        HB_SM3_F(b, c, d, a, f, g, h, e, w11, w15, k27, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w0, w7, w10) HB_SM3_H0 HB_SM3_H_X(x1, w0) HB_SM3_H1(c, a, g, e) HB_SM3_H_N(x0, y0, w14, w4) HB_SM3_H2(a) HB_SM3_E(e) HB_SM3_E_X(x1, y1, w0)
        HB_SM3_F(a, b, c, d, e, f, g, h, w12, w0, k28, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w1, w8, w11) HB_SM3_H0 HB_SM3_H_X(x0, w1) HB_SM3_H1(b, d, f, h) HB_SM3_H_N(x1, y1, w15, w5) HB_SM3_H2(d) HB_SM3_E(h) HB_SM3_E_X(x0, y0, w1)
        HB_SM3_F(d, a, b, c, h, e, f, g, w13, w1, k29, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w2, w9, w12) HB_SM3_H0 HB_SM3_H_X(x1, w2) HB_SM3_H1(a, c, e, g) HB_SM3_H_N(x0, y0, w0, w6) HB_SM3_H2(c) HB_SM3_E(g) HB_SM3_E_X(x1, y1, w2)
        HB_SM3_F(c, d, a, b, g, h, e, f, w14, w2, k30, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w3, w10, w13) HB_SM3_H0 HB_SM3_H_X(x0, w3) HB_SM3_H1(d, b, h, f) HB_SM3_H_N(x1, y1, w1, w7) HB_SM3_H2(b) HB_SM3_E(f) HB_SM3_E_X(x0, y0, w3)
        HB_SM3_F(b, c, d, a, f, g, h, e, w15, w3, k31, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w4, w11, w14) HB_SM3_H0 HB_SM3_H_X(x1, w4) HB_SM3_H1(c, a, g, e) HB_SM3_H_N(x0, y0, w2, w8) HB_SM3_H2(a) HB_SM3_E(e) HB_SM3_E_X(x1, y1, w4)
        HB_SM3_F(a, b, c, d, e, f, g, h, w0, w4, k32, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w5, w12, w15) HB_SM3_H0 HB_SM3_H_X(x0, w5) HB_SM3_H1(b, d, f, h) HB_SM3_H_N(x1, y1, w3, w9) HB_SM3_H2(d) HB_SM3_E(h) HB_SM3_E_X(x0, y0, w5)
        HB_SM3_F(d, a, b, c, h, e, f, g, w1, w5, k33, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w6, w13, w0) HB_SM3_H0 HB_SM3_H_X(x1, w6) HB_SM3_H1(a, c, e, g) HB_SM3_H_N(x0, y0, w4, w10) HB_SM3_H2(c) HB_SM3_E(g) HB_SM3_E_X(x1, y1, w6)
        HB_SM3_F(c, d, a, b, g, h, e, f, w2, w6, k34, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w7, w14, w1) HB_SM3_H0 HB_SM3_H_X(x0, w7) HB_SM3_H1(d, b, h, f) HB_SM3_H_N(x1, y1, w5, w11) HB_SM3_H2(b) HB_SM3_E(f) HB_SM3_E_X(x0, y0, w7)
        HB_SM3_F(b, c, d, a, f, g, h, e, w3, w7, k35, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w8, w15, w2) HB_SM3_H0 HB_SM3_H_X(x1, w8) HB_SM3_H1(c, a, g, e) HB_SM3_H_N(x0, y0, w6, w12) HB_SM3_H2(a) HB_SM3_E(e) HB_SM3_E_X(x1, y1, w8)
        HB_SM3_F(a, b, c, d, e, f, g, h, w4, w8, k36, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w9, w0, w3) HB_SM3_H0 HB_SM3_H_X(x0, w9) HB_SM3_H1(b, d, f, h) HB_SM3_H_N(x1, y1, w7, w13) HB_SM3_H2(d) HB_SM3_E(h) HB_SM3_E_X(x0, y0, w9)
        HB_SM3_F(d, a, b, c, h, e, f, g, w5, w9, k37, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w10, w1, w4) HB_SM3_H0 HB_SM3_H_X(x1, w10) HB_SM3_H1(a, c, e, g) HB_SM3_H_N(x0, y0, w8, w14) HB_SM3_H2(c) HB_SM3_E(g) HB_SM3_E_X(x1, y1, w10)
        HB_SM3_F(c, d, a, b, g, h, e, f, w6, w10, k38, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w11, w2, w5) HB_SM3_H0 HB_SM3_H_X(x0, w11) HB_SM3_H1(d, b, h, f) HB_SM3_H_N(x1, y1, w9, w15) HB_SM3_H2(b) HB_SM3_E(f) HB_SM3_E_X(x0, y0, w11)
        HB_SM3_F(b, c, d, a, f, g, h, e, w7, w11, k39, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w12, w3, w6) HB_SM3_H0 HB_SM3_H_X(x1, w12) HB_SM3_H1(c, a, g, e) HB_SM3_H_N(x0, y0, w10, w0) HB_SM3_H2(a) HB_SM3_E(e) HB_SM3_E_X(x1, y1, w12)
        HB_SM3_F(a, b, c, d, e, f, g, h, w8, w12, k40, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w13, w4, w7) HB_SM3_H0 HB_SM3_H_X(x0, w13) HB_SM3_H1(b, d, f, h) HB_SM3_H_N(x1, y1, w11, w1) HB_SM3_H2(d) HB_SM3_E(h) HB_SM3_E_X(x0, y0, w13)
        HB_SM3_F(d, a, b, c, h, e, f, g, w9, w13, k41, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w14, w5, w8) HB_SM3_H0 HB_SM3_H_X(x1, w14) HB_SM3_H1(a, c, e, g) HB_SM3_H_N(x0, y0, w12, w2) HB_SM3_H2(c) HB_SM3_E(g) HB_SM3_E_X(x1, y1, w14)
        HB_SM3_F(c, d, a, b, g, h, e, f, w10, w14, k42, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w15, w6, w9) HB_SM3_H0 HB_SM3_H_X(x0, w15) HB_SM3_H1(d, b, h, f) HB_SM3_H_N(x1, y1, w13, w3) HB_SM3_H2(b) HB_SM3_E(f) HB_SM3_E_X(x0, y0, w15)
        HB_SM3_F(b, c, d, a, f, g, h, e, w11, w15, k43, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w0, w7, w10) HB_SM3_H0 HB_SM3_H_X(x1, w0) HB_SM3_H1(c, a, g, e) HB_SM3_H_N(x0, y0, w14, w4) HB_SM3_H2(a) HB_SM3_E(e) HB_SM3_E_X(x1, y1, w0)
        HB_SM3_F(a, b, c, d, e, f, g, h, w12, w0, k44, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w1, w8, w11) HB_SM3_H0 HB_SM3_H_X(x0, w1) HB_SM3_H1(b, d, f, h) HB_SM3_H_N(x1, y1, w15, w5) HB_SM3_H2(d) HB_SM3_E(h) HB_SM3_E_X(x0, y0, w1)
        HB_SM3_F(d, a, b, c, h, e, f, g, w13, w1, k45, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x1, y1, w2, w9, w12) HB_SM3_H0 HB_SM3_H_X(x1, w2) HB_SM3_H1(a, c, e, g) HB_SM3_H_N(x0, y0, w0, w6) HB_SM3_H2(c) HB_SM3_E(g) HB_SM3_E_X(x1, y1, w2)
        HB_SM3_F(c, d, a, b, g, h, e, f, w14, w2, k46, HB_TT_MAJ, HB_TT_CH) HB_SM3_F_X(x0, y0, w3, w10, w13) HB_SM3_H0 HB_SM3_H_X(x0, w3) HB_SM3_H1(d, b, h, f) HB_SM3_H2(b) HB_SM3_E(f) HB_SM3_E_X(x0, y0, w3)
        HB_SM3_F(b, c, d, a, f, g, h, e, w15, w3, k47, HB_TT_MAJ, HB_TT_CH) HB_SM3_H0 HB_SM3_H1(c, a, g, e) HB_SM3_E(e)
        HB_WIDE
        : [a] "+v"(a), [b] "+v"(b), [c] "+v"(c), [d] "+v"(d), [e] "+v"(e), [f] "+v"(f), [g] "+v"(g), [h] "+v"(h),
          [p] "=&v"(p), [q] "=&v"(q), [r] "=&v"(r), [s] "=&v"(s), [x0] "=&v"(x0), [x1] "=&v"(x1), [y0] "=&v"(y0),
          [y1] "=&v"(y1), [w0] "+v"(W[0]), [w1] "+v"(W[1]), [w2] "+v"(W[2]), [w3] "+v"(W[3]), [w4] "+v"(W[4]),
          [w5] "+v"(W[5]), [w6] "+v"(W[6]), [w7] "+v"(W[7]), [w8] "+v"(W[8]), [w9] "+v"(W[9]), [w10] "+v"(W[10]),
          [w11] "+v"(W[11]), [w12] "+v"(W[12]), [w13] "+v"(W[13]), [w14] "+v"(W[14]), [w15] "+v"(W[15])
        : [k0] "s"(sm3_tj(0)), [k1] "s"(sm3_tj(1)), [k2] "s"(sm3_tj(2)), [k3] "s"(sm3_tj(3)), [k4] "s"(sm3_tj(4)), [k5] "s"(sm3_tj(5)),
          [k6] "s"(sm3_tj(6)), [k7] "s"(sm3_tj(7)), [k8] "s"(sm3_tj(8)), [k9] "s"(sm3_tj(9)), [k10] "s"(sm3_tj(10)), [k11] "s"(sm3_tj(11)),
          [k12] "s"(sm3_tj(12)), [k13] "s"(sm3_tj(13)), [k14] "s"(sm3_tj(14)), [k15] "s"(sm3_tj(15)), [k16] "s"(sm3_tj(32)), [k17] "s"(sm3_tj(33)),
          [k18] "s"(sm3_tj(34)), [k19] "s"(sm3_tj(35)), [k20] "s"(sm3_tj(36)), [k21] "s"(sm3_tj(37)), [k22] "s"(sm3_tj(38)), [k23] "s"(sm3_tj(39)),
          [k24] "s"(sm3_tj(40)), [k25] "s"(sm3_tj(41)), [k26] "s"(sm3_tj(42)), [k27] "s"(sm3_tj(43)), [k28] "s"(sm3_tj(44)), [k29] "s"(sm3_tj(45)),
          [k30] "s"(sm3_tj(46)), [k31] "s"(sm3_tj(47)), [k32] "s"(sm3_tj(16)), [k33] "s"(sm3_tj(17)), [k34] "s"(sm3_tj(18)), [k35] "s"(sm3_tj(19)),
          [k36] "s"(sm3_tj(20)), [k37] "s"(sm3_tj(21)), [k38] "s"(sm3_tj(22)), [k39] "s"(sm3_tj(23)), [k40] "s"(sm3_tj(24)), [k41] "s"(sm3_tj(25)),
          [k42] "s"(sm3_tj(26)), [k43] "s"(sm3_tj(27)), [k44] "s"(sm3_tj(28)), [k45] "s"(sm3_tj(29)), [k46] "s"(sm3_tj(30)), [k47] "s"(sm3_tj(31)));
    s8[0] ^= a; s8[1] ^= b; s8[2] ^= c; s8[3] ^= d; s8[4] ^= e; s8[5] ^= f; s8[6] ^= g; s8[7] ^= h;
}

// The compression for a launch whose waves share their SIMDs.
template <int A> __device__ __forceinline__ void compress_many(uint32_t s[8], const uint32_t w[16])
{
    if constexpr (A == MD5) md5_compress_many(s, w);
    else if constexpr (A == SHA1) sha1_compress_many(s, w);
    else sm3_compress_many(s, w);
}

// ---------------------------------------------------------------------------------------
// A block whose words are the same for every lane -- the padding-only last block of a
// fixed-length batch -- from schedule words the host has formed: the rounds alone, a third
// fewer instructions (SM3 16 a round for 24).  Words: as md5_sched / sha1_sched / sm3_sched
// (hb_long.hpp) give them: X + T; W + K; W' and then W.
// ---------------------------------------------------------------------------------------

template <int A> struct UniformWords;
template <> struct UniformWords<MD5> { uint32_t w[64]; };
template <> struct UniformWords<SHA1> { uint32_t w[80]; };
template <> struct UniformWords<SM3> { uint32_t w[128]; };

#define HB_MD5_U(a, b, c, d, x, s, F)                                                         \
    "v_bitop3_b32 %[t], %[" #b "], %[" #c "], %[" #d "] bitop3:" F "\n\t"                     \
    HB_WIDE                                                                                   \
    "v_add3_u32 %[" #a "], %[" #a "], %[t], %[" #x "]\n\t"                                    \
    "v_alignbit_b32 %[" #a "], %[" #a "], %[" #a "], " #s "\n\t"                              \
    HB_PLAIN                                                                                  \
    "v_add_u32 %[" #a "], %[" #a "], %[" #b "]\n\t"
#define HB_MD5_U4(F, s0, s1, s2, s3)                                                          \
    asm volatile(HB_MD5_U(a, b, c, d, x0, s0, F) HB_MD5_U(d, a, b, c, x1, s1, F)              \
                 HB_MD5_U(c, d, a, b, x2, s2, F) HB_MD5_U(b, c, d, a, x3, s3, F)              \
                 : [a] "+v"(a), [b] "+v"(b), [c] "+v"(c), [d] "+v"(d), [t] "=&v"(t)           \
                 : [x0] "s"(x[0]), [x1] "s"(x[1]), [x2] "s"(x[2]), [x3] "s"(x[3]))

#define HB_SHA1_U(a, b, c, d, e, w, F)                                                        \
    "v_bitop3_b32 %[f], %[" #b "], %[" #c "], %[" #d "] bitop3:" F "\n\t"                     \
    "v_add_u32 %[" #e "], %[" #w "], %[" #e "]\n\t"                                           \
    HB_WIDE                                                                                   \
    "v_alignbit_b32 %[u], %[" #a "], %[" #a "], 27\n\t"                                       \
    "v_alignbit_b32 %[" #b "], %[" #b "], %[" #b "], 2\n\t"                                   \
    "v_add3_u32 %[" #e "], %[" #e "], %[f], %[u]\n\t"                                         \
    HB_PLAIN
#define HB_SHA1_U5(F)                                                                         \
    asm volatile(HB_SHA1_U(a, b, c, d, e, x0, F) HB_SHA1_U(e, a, b, c, d, x1, F)              \
                 HB_SHA1_U(d, e, a, b, c, x2, F) HB_SHA1_U(c, d, e, a, b, x3, F)              \
                 HB_SHA1_U(b, c, d, e, a, x4, F)                                              \
                 : [a] "+v"(a), [b] "+v"(b), [c] "+v"(c), [d] "+v"(d), [e] "+v"(e), [f] "=&v"(f), [u] "=&v"(u) \
                 : [x0] "s"(x[0]), [x1] "s"(x[1]), [x2] "s"(x[2]), [x3] "s"(x[3]), [x4] "s"(x[4]))

#define HB_SM3_U(a, b, c, d, e, f, g, h, w, x, k, FF, GG)                                     \
    "v_add_u32 %[s], %[" #k "], %[" #e "]\n\t"                                                \
    "v_bitop3_b32 %[p], %[" #a "], %[" #b "], %[" #c "] bitop3:" FF "\n\t"                    \
    "v_bitop3_b32 %[q], %[" #e "], %[" #f "], %[" #g "] bitop3:" GG "\n\t"                    \
    "v_add_u32 %[s], %[s], %[r]\n\t"                                                          \
    "v_add_u32 %[" #h "], %[" #w "], %[" #h "]\n\t"                                           \
    "v_add_u32 %[" #d "], %[" #d "], %[p]\n\t"                                                \
    "v_add_u32 %[" #d "], %[" #x "], %[" #d "]\n\t"                                           \
    HB_SM3_H0 HB_SM3_H1(b, d, f, h) HB_SM3_H2(d) HB_SM3_E(h)
#define HB_SM3_U4(FF, GG)                                                                     \
    asm volatile(HB_SM3_U(a, b, c, d, e, f, g, h, w0, x0, k0, FF, GG)                         \
                 HB_SM3_U(d, a, b, c, h, e, f, g, w1, x1, k1, FF, GG)                         \
                 HB_SM3_U(c, d, a, b, g, h, e, f, w2, x2, k2, FF, GG)                         \
                 HB_SM3_U(b, c, d, a, f, g, h, e, w3, x3, k3, FF, GG)                         \
                 : [a] "+v"(a), [b] "+v"(b), [c] "+v"(c), [d] "+v"(d), [e] "+v"(e), [f] "+v"(f), [g] "+v"(g), \
                   [h] "+v"(h), [r] "+v"(r), [p] "=&v"(p), [q] "=&v"(q), [s] "=&v"(s)         \
                 : [x0] "s"(x[0]), [x1] "s"(x[1]), [x2] "s"(x[2]), [x3] "s"(x[3]), \
                   [w0] "s"(x[64]), [w1] "s"(x[65]), [w2] "s"(x[66]), [w3] "s"(x[67]), \
                   [k0] "s"(sm3_tj(j)), [k1] "s"(sm3_tj(j + 1)), [k2] "s"(sm3_tj(j + 2)), [k3] "s"(sm3_tj(j + 3)))

#define HB_CONSTANT __attribute__((address_space(4)))

// The words are read a few rounds at a time, each read behind an opaque zero: all together
// would not fit the scalar registers, and the compiler would read them so.
template <int A> __device__ __forceinline__ void compress_uniform(uint32_t v[8], const HB_CONSTANT uint32_t *words)
{
    auto next = [&](int j) {
        uint32_t zero = 0;
        asm volatile("" : "+s"(zero));
        return words + zero + j;
    };
    if constexpr (A == MD5) {
        uint32_t a = v[0], b = v[1], c = v[2], d = v[3], t;
#pragma unroll
        for (int j = 0; j < 64; j += 4) {
            const HB_CONSTANT uint32_t *x = next(j);
            if (j < 16) HB_MD5_U4(HB_TT_CH, 25, 20, 15, 10);
            else if (j < 32) HB_MD5_U4(HB_TT_G, 27, 23, 18, 12);
            else if (j < 48) HB_MD5_U4(HB_TT_XOR3, 28, 21, 16, 9);
            else HB_MD5_U4(HB_TT_I, 26, 22, 17, 11);
        }
        v[0] += a; v[1] += b; v[2] += c; v[3] += d;
    } else if constexpr (A == SHA1) {
        uint32_t a = v[0], b = v[1], c = v[2], d = v[3], e = v[4], f, u;
#pragma unroll
        for (int j = 0; j < 80; j += 5) {
            const HB_CONSTANT uint32_t *x = next(j);
            if (j < 20) HB_SHA1_U5(HB_TT_CH);
            else if (j < 40 || j >= 60) HB_SHA1_U5(HB_TT_XOR3);
            else HB_SHA1_U5(HB_TT_MAJ);
        }
        v[0] += a; v[1] += b; v[2] += c; v[3] += d; v[4] += e;
    } else {
        uint32_t a = v[0], b = v[1], c = v[2], d = v[3], e = v[4], f = v[5], g = v[6], h = v[7], p, q, r = rotl<12>(a), s;
#pragma unroll
        for (int j = 0; j < 64; j += 4) {
            const HB_CONSTANT uint32_t *x = next(j);
            if (j < 16) HB_SM3_U4(HB_TT_XOR3, HB_TT_XOR3);
            else HB_SM3_U4(HB_TT_MAJ, HB_TT_CH);
        }
        v[0] ^= a; v[1] ^= b; v[2] ^= c; v[3] ^= d; v[4] ^= e; v[5] ^= f; v[6] ^= g; v[7] ^= h;
    }
}

#undef HB_MD5_U
#undef HB_MD5_U4
#undef HB_SHA1_U
#undef HB_SHA1_U5
#undef HB_SM3_U
#undef HB_SM3_U4
#undef HB_MD5_I
#undef HB_SHA1_PLAIN
#undef HB_SHA1_WIDE
#undef HB_SHA1_I
#undef HB_SHA1_X
#undef HB_SM3_F
#undef HB_SM3_F_X
#undef HB_SM3_H0
#undef HB_SM3_H_X
#undef HB_SM3_H1
#undef HB_SM3_H_N
#undef HB_SM3_H2
#undef HB_SM3_E
#undef HB_SM3_E_X
#undef HB_WIDE
#undef HB_PLAIN

}  // namespace hb
