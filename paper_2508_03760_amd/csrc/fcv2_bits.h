// fcv2_bits.h -- building blocks of the codec kernels: bf16 bit handling, order keys, a lane's part of the spike selection, and the
// shift/mask sequences that move code fields between "one code per byte" registers and the packed bit planes
// (Section 3.2 of arxiv 2508.03760: a b-bit code is split into 4/2/1-bit planes stored separately).
//
// Everything here works inside one lane, on 32-bit integers and fp32 numbers, and is usable from host and device, so the
// sequences can be unit-tested on the CPU.  The plane sequences work on 8 consecutive elements:
//   c0 = codes of elements 0..3, one per byte (element 0 in bits 0..7), c1 = elements 4..7.
#pragma once
#include <math.h>
#include <stddef.h>
#include <stdint.h>

#if defined(__HIPCC__)
#define FCV2_HD __host__ __device__ __forceinline__
#else
#define FCV2_HD inline
#endif

// Tables and the functions that index them: device-only inside the HIP translation unit, plain host code in
// the CPU test build.
#if defined(__HIPCC__)
#define FCV2_TABLE static __device__ const
#define FCV2_D __device__ __forceinline__
#else
#define FCV2_TABLE static const
#define FCV2_D inline
#endif

// Keeps the compiler from merging a chain of shift-or steps into one 32-bit multiply (quarter rate on CDNA).
#if defined(__HIP_DEVICE_COMPILE__)
#define FCV2_KEEP(v) asm volatile("" : "+v"(v))
#else
#define FCV2_KEEP(v) (void)(v)
#endif

namespace fcv2 {

// ---- single instructions whose form matters --------------------------------------------------------------------------
// Measured on the MI355X (8 waves per SIMD, independent chains): a wave-wide VALU instruction issues in about 2.4
// cycles when it is a two-operand instruction of a simple class -- and, or, xor, right shift, integer add, fp32
// add / subtract / multiply, move -- whose operands are vector registers, a literal or an inline constant; in about 3
// cycles for an fp32 FMA and for v_bitop3 on three vector registers; and in about 4.2 cycles otherwise: anything that
// reads a SCALAR register, left shifts, the three-operand integer forms, integer min/max/med3, conversions, packed
// 16-bit, DPP, SDWA, permutes, dot products (reciprocal: 8.3).  The compiler likes to park a constant that is used
// more than once in a scalar register, which turns the cheapest class into the dearest; the helpers below pin the
// cheap form.  On the host they are plain C.
#if defined(__HIP_DEVICE_COMPILE__)
template <uint32_t C> FCV2_D uint32_t and_lit(uint32_t x) {  // x & C as v_and_b32 with the literal in the instruction
    uint32_t r;
    asm("v_and_b32 %0, %1, %2" : "=v"(r) : "n"((int32_t)C), "v"(x));
    return r;
}
template <uint32_t C> FCV2_D uint32_t xor_lit(uint32_t x) {
    uint32_t r;
    asm("v_xor_b32 %0, %1, %2" : "=v"(r) : "n"((int32_t)C), "v"(x));
    return r;
}
// A constant held in a vector register the compiler cannot see through (so it cannot move it to a scalar one).
template <uint32_t C> FCV2_D uint32_t vreg_const() {
    uint32_t r;
    asm volatile("v_mov_b32 %0, %1" : "=v"(r) : "n"((int32_t)C));
    return r;
}
// (m & a) | (~m & b) in one v_bitop3 on three vector registers.
FCV2_D uint32_t bit_select(uint32_t m, uint32_t a, uint32_t b) { return __builtin_amdgcn_bitop3_b32(a, b, m, 0xE4); }
// (a | b) & m likewise.
FCV2_D uint32_t or_and(uint32_t a, uint32_t b, uint32_t m) { return __builtin_amdgcn_bitop3_b32(a, b, m, 0xA8); }
// sum of byte products: a.b0 * w.b0 + ... + a.b3 * w.b3 + c
FCV2_D uint32_t dot4_u8(uint32_t a, uint32_t w, uint32_t c) { return __builtin_amdgcn_udot4(a, w, c, false); }
FCV2_D uint32_t rotr32(uint32_t x, int r) { return __builtin_amdgcn_alignbit(x, x, r); }
FCV2_D uint32_t umed3(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
FCV2_D uint32_t umin3(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    asm("v_min3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
#define FCV2_F32_OP3(name, op)                                            \
    FCV2_D float name(float a, float b, float c) {                        \
        float r;                                                          \
        asm(op " %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));     \
        return r;                                                         \
    }
#define FCV2_F32_OP2(name, op)                                            \
    FCV2_D float name(float a, float b) {                                 \
        float r;                                                          \
        asm(op " %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));                 \
        return r;                                                         \
    }
FCV2_F32_OP3(f_med3, "v_med3_f32")
FCV2_F32_OP3(f_minimum3, "v_minimum3_f32")  // these two return NaN if any operand is one
FCV2_F32_OP3(f_maximum3, "v_maximum3_f32")
FCV2_F32_OP2(f_min, "v_min_f32")
FCV2_F32_OP2(f_max, "v_max_f32")
#undef FCV2_F32_OP3
#undef FCV2_F32_OP2
// (sign | flip) ^ w, sign = the sign bit of each 16-bit half spread over it: one three-register bitwise operation.
FCV2_D uint32_t keys_of_pair(uint32_t w, uint32_t key_flip) {
    typedef short short2v __attribute__((ext_vector_type(2)));
    const uint32_t sign = __builtin_bit_cast(uint32_t, __builtin_bit_cast(short2v, w) >> (short2v){15, 15});
    return __builtin_amdgcn_bitop3_b32(sign, w, key_flip, 0x36);
}
// The low (high) bf16 half of w with position p below it, as an fp32 number.  Single instructions, opaque to the compiler: it would
// keep the shifted and masked halves of all elements in registers from here to the quantizer, which takes the same halves (50
// registers more, two waves per SIMD fewer).
FCV2_D float composite_lo(uint32_t w, uint32_t p) {
    float x;
    asm("v_lshl_or_b32 %0, %1, 16, %2" : "=v"(x) : "v"(w), "i"(p));
    return x;
}
FCV2_D float composite_hi(uint32_t w, uint32_t hi_mask, uint32_t p) {
    float y;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(y) : "v"(w), "v"(hi_mask), "i"(p));
    return y;
}
#else  // the host pass of the HIP compiler, and the CPU test build
template <uint32_t C> FCV2_HD uint32_t and_lit(uint32_t x) { return x & C; }
template <uint32_t C> FCV2_HD uint32_t xor_lit(uint32_t x) { return x ^ C; }
template <uint32_t C> FCV2_HD uint32_t vreg_const() { return C; }
FCV2_HD uint32_t bit_select(uint32_t m, uint32_t a, uint32_t b) { return (m & a) | (~m & b); }
FCV2_HD uint32_t or_and(uint32_t a, uint32_t b, uint32_t m) { return (a | b) & m; }
FCV2_HD uint32_t dot4_u8(uint32_t a, uint32_t w, uint32_t c) {
    for (int i = 0; i < 4; ++i) c += ((a >> (8 * i)) & 0xFFu) * ((w >> (8 * i)) & 0xFFu);
    return c;
}
FCV2_HD uint32_t rotr32(uint32_t x, int r) { return (x >> r) | (x << ((32 - r) & 31)); }
FCV2_HD uint32_t umin3(uint32_t a, uint32_t b, uint32_t c) { return a < b ? (a < c ? a : c) : (b < c ? b : c); }
FCV2_HD uint32_t umed3(uint32_t a, uint32_t b, uint32_t c) {
    const uint32_t lo = a < b ? a : b, hi = a < b ? b : a;
    return c < lo ? lo : c > hi ? hi : c;
}
// -0 below +0, as the instructions have it; min and max of a number and a NaN are the number.
FCV2_HD bool f_below(float a, float b) { return a < b || (a == b && signbit(a) && !signbit(b)); }
FCV2_HD float f_min(float a, float b) { return a != a ? b : b != b ? a : f_below(b, a) ? b : a; }
FCV2_HD float f_max(float a, float b) { return a != a ? b : b != b ? a : f_below(a, b) ? b : a; }
FCV2_HD float f_minimum3(float a, float b, float c) { return (a != a || b != b || c != c) ? NAN : f_min(f_min(a, b), c); }
FCV2_HD float f_maximum3(float a, float b, float c) { return (a != a || b != b || c != c) ? NAN : f_max(f_max(a, b), c); }
FCV2_HD float f_med3(float a, float b, float c) { return f_max(f_min(a, b), f_min(f_max(a, b), c)); }
FCV2_HD uint32_t keys_of_pair(uint32_t w, uint32_t key_flip) {
    const uint32_t sign = ((w & 0x8000u) ? 0xFFFFu : 0u) | ((w & 0x80000000u) ? 0xFFFF0000u : 0u);
    return (sign | key_flip) ^ w;
}
FCV2_HD float composite_lo(uint32_t w, uint32_t p) { return __builtin_bit_cast(float, (w << 16) | p); }
FCV2_HD float composite_hi(uint32_t w, uint32_t hi_mask, uint32_t p) { return __builtin_bit_cast(float, (w & hi_mask) | p); }
#endif

// ---- plane structure of a b-bit code: widest plane first = most significant bits ---------------------------
template <int BITS> struct Planes;
template <> struct Planes<2> { static constexpr int w8 = 0, w4 = 0, w2 = 1, w1 = 0, sh4 = 0, sh2 = 0, sh1 = 0; };
template <> struct Planes<3> { static constexpr int w8 = 0, w4 = 0, w2 = 1, w1 = 1, sh4 = 0, sh2 = 1, sh1 = 0; };
template <> struct Planes<4> { static constexpr int w8 = 0, w4 = 1, w2 = 0, w1 = 0, sh4 = 0, sh2 = 0, sh1 = 0; };
template <> struct Planes<5> { static constexpr int w8 = 0, w4 = 1, w2 = 0, w1 = 1, sh4 = 1, sh2 = 0, sh1 = 0; };
template <> struct Planes<6> { static constexpr int w8 = 0, w4 = 1, w2 = 1, w1 = 0, sh4 = 2, sh2 = 0, sh1 = 0; };
template <> struct Planes<7> { static constexpr int w8 = 0, w4 = 1, w2 = 1, w1 = 1, sh4 = 3, sh2 = 1, sh1 = 0; };
template <> struct Planes<8> { static constexpr int w8 = 1, w4 = 0, w2 = 0, w1 = 0, sh4 = 0, sh2 = 0, sh1 = 0; };

// ---- bf16 ---------------------------------------------------------------------------------------------------
// Total order on bf16 bit patterns that equals numeric order on finite values, with -0 below +0.
FCV2_HD uint32_t key_of_bf16(uint32_t u) { return (u & 0x8000u) ? (~u & 0xFFFFu) : (u | 0x8000u); }
FCV2_HD uint32_t bf16_of_key(uint32_t k) { return (k & 0x8000u) ? (k ^ 0x8000u) : (~k & 0xFFFFu); }

// fp32 bits -> bf16 bits, round to nearest even; NaN stays a quiet NaN.
FCV2_HD uint32_t bf16_rne_bits(uint32_t u) {
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x0040u;
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// Smallest bf16-representable fp32 bit pattern that is >= the (positive, finite) input.
FCV2_HD uint32_t bf16_round_up_bits(uint32_t u) { return (u + 0xFFFFu) & 0xFFFF0000u; }

// ---- the spikes of a group: one lane's part (group_spikes puts the lanes together) -----------------------------------------
FCV2_D float u2f(uint32_t u) { return __builtin_bit_cast(float, u); }
FCV2_D uint32_t f2u(float f) { return __builtin_bit_cast(uint32_t, f); }

// Order-preserving map of fp32 bit patterns to unsigned integers (-0 below +0).
FCV2_D uint32_t key_of_f32(uint32_t x) { return x ^ ((uint32_t)((int32_t)x >> 31) | 0x80000000u); }

// Running two smallest values (m1 <= m2) of a stream, two new values at a time: the new second smallest is the smaller
// of the old one and the median of {m1, x, y} (m1 belongs to the three, so their median is the second smallest of the
// three; whatever is second smallest overall is either that or the old m2).  Three instructions for two values.
FCV2_D void push2_pair(uint32_t& m1, uint32_t& m2, uint32_t x, uint32_t y) {
    const uint32_t t = umed3(m1, x, y);
    m1 = umin3(m1, x, y);
    m2 = m2 < t ? m2 : t;
}

// Two smallest composites (key << 16 | position) of the lane and two smallest of (~key << 16 | position), for any bit
// patterns (NaN included).  Positions count inside the lane.
template <int EPL> FCV2_D void lane_extremes_any(const uint32_t (&w)[EPL / 2], uint32_t& a1, uint32_t& a2, uint32_t& b1, uint32_t& b2) {
    const uint32_t key_flip = vreg_const<0x80008000u>();
#pragma unroll
    for (int d = 0; d < EPL / 2; ++d) {
        const uint32_t k = keys_of_pair(w[d], key_flip);
        uint32_t e0 = (k << 16) | (uint32_t)(2 * d), e1 = (k & 0xFFFF0000u) | (uint32_t)(2 * d + 1);
        FCV2_KEEP(e0);  // keeps each composite one shift-or / and-or instruction (no regrouping with the xor below)
        FCV2_KEEP(e1);
        const uint32_t f0 = xor_lit<0xFFFF0000u>(e0), f1 = xor_lit<0xFFFF0000u>(e1);  // inverted key: min finds the largest value
        if (d == 0) {
            a1 = e0 < e1 ? e0 : e1;
            a2 = e0 < e1 ? e1 : e0;
            b1 = f0 < f1 ? f0 : f1;
            b2 = f0 < f1 ? f1 : f0;
        } else {
            push2_pair(a1, a2, e0, e1);
            push2_pair(b1, b2, f0, f1);
        }
    }
}

// A bf16 value with a position in the 16 bits below it is an fp32 number, so the two smallest and two largest come out of the
// fp32 median / minimum / maximum instructions: 8 instructions per pair of elements, where composites of integer order keys
// (lane_extremes_any) take 12, half of them to build the keys and to invert them for the maximum.  The position stands there
// inverted, so that of equal values the lowest index wins where the minimum is negative and the maximum is not; the other
// way round (a group of one sign) the position is looked for again (lane_spikes_upright).  hi_mask = 0xFFFF0000.
template <int EPL> FCV2_D void lane_spikes(const uint32_t (&w)[EPL / 2], uint32_t hi_mask, float& a1, float& a2, float& b1, float& b2) {
#pragma unroll
    for (int d = 0; d < EPL / 2; ++d) {
        const float x = composite_lo(w[d], (uint32_t)(EPL - 1 - 2 * d)), y = composite_hi(w[d], hi_mask, (uint32_t)(EPL - 2 - 2 * d));
        if (d == 0) {
            a1 = f_minimum3(x, y, y);
            a2 = f_max(x, y);
            b1 = f_maximum3(x, y, y);
            b2 = f_min(x, y);
        } else {
            const float ta = f_med3(a1, x, y), tb = f_med3(b1, x, y);
            a1 = f_minimum3(a1, x, y);
            b1 = f_maximum3(b1, x, y);
            a2 = f_min(a2, ta);
            b2 = f_max(b2, tb);
        }
    }
}

// The minimum and the two largest with the positions as they are.
template <int EPL> FCV2_D void lane_spikes_upright(const uint32_t (&w)[EPL / 2], uint32_t hi_mask, float& a1, float& b1, float& b2) {
#pragma unroll
    for (int d = 0; d < EPL / 2; ++d) {
        const float x = composite_lo(w[d], (uint32_t)(2 * d)), y = composite_hi(w[d], hi_mask, (uint32_t)(2 * d + 1));
        if (d == 0) {
            a1 = f_min(x, y);
            b1 = f_max(x, y);
            b2 = f_min(x, y);
        } else {
            const float t = f_med3(b1, x, y);
            a1 = f_minimum3(a1, x, y);
            b1 = f_maximum3(b1, x, y);
            b2 = f_max(b2, t);
        }
    }
}

// Whether lane_spikes and lane_spikes_upright hold for the lane: no value is an infinity or a NaN.  With a position below it both
// are NaNs, which minimum3 / maximum3 hand on to a1 and b1.  The one infinity that stays an infinity has position 0 below it,
// that is the lane's last element in lane_spikes and its first in lane_spikes_upright; it then is the extreme of its side, so
// looking for an infinity in a1 and b1 finds it too, before the second look makes it a NaN.
FCV2_D bool spikes_are_finite(float a1, float b1) { return a1 > -INFINITY && b1 < INFINITY; }

// What a lane found as integer composites (key << 16 | position in the group; the key inverted on the maximum's side).  The
// inverted position of a negative number (of a non-negative one on the maximum's side) turns back here.
template <int EPL> FCV2_D uint32_t spike_composite(float f, uint32_t lbase) {
    return (key_of_f32(f2u(f)) & (0xFFFF0000u | (uint32_t)(EPL - 1))) | lbase;
}
template <int EPL> FCV2_D uint32_t spike_composite_inv(float f, uint32_t lbase) {
    return (~key_of_f32(f2u(f)) & (0xFFFF0000u | (uint32_t)(EPL - 1))) | lbase;
}

// The group's minimum is +0 or above, or its maximum is negative: the positions of that side are still inverted.
FCV2_D bool spikes_of_one_sign(uint32_t a1, uint32_t b1) { return (int32_t)(a1 | b1) < 0; }

// ... and come from the second look (c1 the minimum, d1 and d2 the two largest) instead.
FCV2_D void take_upright(uint32_t c1, uint32_t d1, uint32_t d2, uint32_t& a1, uint32_t& b1, uint32_t& b2) {
    if ((int32_t)a1 < 0) a1 = c1;
    if ((int32_t)b1 < 0) {
        b1 = d1;
        b2 = d2;
    }
}

// d / QMAX with IEEE rounding for d >= 0, without the long division sequence: multiply by the rounded
// reciprocal, then one exact-residual correction (Markstein).  Checked against IEEE division for every fp32
// significand and every QMAX = 2^b - 1 by the host tests; +inf and NaN are passed through.
template <int QMAX> FCV2_HD float div_by_qmax(float d) {
    constexpr float y = 1.0f / (float)QMAX;
    const float q0 = d * y;
    const float r = fmaf(-(float)QMAX, q0, d);
    const float q1 = fmaf(r, y, q0);
    return (d < INFINITY) ? q1 : d;
}

// ---- integer metadata (Section 3.3, Eq. 1: scale_int = round(log2(scale) * 10), one signed byte) -------------
// kPow10th[j + 1] = 2^(j/10) rounded to fp32 for j = -1..10.  kThr10th[j] = 2^((j - 1/2)/10) rounded UP to fp32 for
// j = 0..10: a scale s has round(log2(s) * 10) >= 10e + j exactly when s >= 2^e * kThr10th[j] (the true thresholds
// are irrational, so rounding them up to the next fp32 changes no decision).
#define FCV2_POW10TH_VALUES                                                                                                    \
    {0x1.ddb680p-1f, 0x1.000000p+0f, 0x1.125fbep+0f, 0x1.261118p+0f, 0x1.3b2c48p+0f, 0x1.51cb46p+0f,                               \
     0x1.6a09e6p+0f, 0x1.840600p+0f, 0x1.9fdf8cp+0f, 0x1.bdb8cep+0f, 0x1.ddb680p+0f, 0x1.000000p+1f}
#define FCV2_THR10TH_VALUES                                                                                                    \
    {0x1.ee8f36p-1f, 0x1.090720p+0f, 0x1.1c0cc0p+0f, 0x1.306fe2p+0f, 0x1.46499cp+0f, 0x1.5db4d2p+0f,                               \
     0x1.76ce52p+0f, 0x1.91b502p+0f, 0x1.ae89fap+0f, 0x1.cd70b4p+0f, 0x1.ee8f36p+0f}
FCV2_TABLE float kPow10th[12] = FCV2_POW10TH_VALUES;
FCV2_TABLE float kThr10th[11] = FCV2_THR10TH_VALUES;

// k = 10e + j with 0 <= j <= 9, for -128 <= k <= 127.
FCV2_D void split_tenths(int k, int& e, int& j) {
    const uint32_t u = (uint32_t)(k + 130);
    const uint32_t q = (u * 205u) >> 11;  // u / 10 for u < 1029
    e = (int)q - 13;
    j = (int)(u - 10u * q);
}

// The scale a receiver reconstructs from the byte: 2^(k/10) as an fp32 value (the table entry scaled by an exact
// power of two).
FCV2_D float scale_of_int(int k) {
    int e, j;
    split_tenths(k, e, j);
    return ldexpf(kPow10th[j + 1], e);
}

// round(log2(s) * 10) to within 1 from the bit pattern alone: exponent + significand fraction is a piecewise-linear
// log2 that is low by at most 0.0861; centring that error leaves |10 * error| < 0.44, so the rounded estimate is
// at most one off.
FCV2_D int scale_int_estimate(float s) {
    uint32_t bits;
    __builtin_memcpy(&bits, &s, 4);
    const float t = (float)((int32_t)bits - 0x3F800000) * (10.0f / 8388608.0f) + 0.43f;
    return (int)rintf(fminf(fmaxf(t, -128.0f), 127.0f));
}

struct ScaleInt {
    int k;    // Eq. 1, clamped to a signed byte
    float s;  // 2^(k/10)
};

// Eq. 1 without a logarithm: the estimate is corrected by comparing s with the two thresholds around it.
// Zero, negative and NaN inputs give the lowest code.
FCV2_D ScaleInt scale_int_of(float s) {
    int k0 = (s > 0.0f) ? scale_int_estimate(s) : -128;
    int e, j;
    split_tenths(k0, e, j);
    const float below = ldexpf(kThr10th[j], e), above = ldexpf(kThr10th[j + 1], e);
    int d = 0;
    if (s >= above) d = 1;
    if (s < below) d = -1;
    if (k0 + d > 127 || k0 + d < -128) d = 0;
    ScaleInt r;
    r.k = k0 + d;
    r.s = ldexpf(kPow10th[j + 1 + d], e);
    return r;
}

// The same two functions from per-code tables (the kernels keep them in LDS): pow_tab[k + 129] = 2^(k/10) for
// k = -128..127 (entries 0 and 257 are never selected, they only keep the neighbour reads in bounds),
// thr_tab[k + 128] = smallest fp32 whose code is >= k, for k = -128..128.  Entry t of each:
FCV2_D float scale_table_pow(int t) { return (t >= 1 && t <= 256) ? scale_of_int(t - 129) : 0.0f; }
FCV2_D float scale_table_thr(int t) {
    int e, j;
    split_tenths(t - 128, e, j);  // the split also holds for k = 128
    return ldexpf(kThr10th[j], e);
}
constexpr int kScaleTablePow = 258, kScaleTableThr = 257;

// Both tables written out at compile time, the power table first: what a kernel copies into LDS.  An entry is one of the
// twelve (eleven) values above times an exact power of two between 2^-13 and 2^13, so the products are the values that
// scale_table_pow and scale_table_thr compute (the host tests compare all of them).
struct ScaleTables {
    float v[kScaleTablePow + kScaleTableThr];
};
constexpr float exact_pow2(int e) {
    float r = 1.0f;
    for (; e > 0; --e) r *= 2.0f;
    for (; e < 0; ++e) r *= 0.5f;
    return r;
}
constexpr ScaleTables make_scale_tables() {
    constexpr float pow10th[12] = FCV2_POW10TH_VALUES;
    constexpr float thr10th[11] = FCV2_THR10TH_VALUES;
    ScaleTables T{};
    for (int t = 0; t < kScaleTablePow + kScaleTableThr; ++t) {
        const bool is_pow = t < kScaleTablePow;
        const int k = is_pow ? t - 129 : t - kScaleTablePow - 128;  // the code the entry belongs to
        const int u = k + 130, q = (u * 205) >> 11, e = q - 13, j = u - 10 * q;  // split_tenths
        T.v[t] = is_pow ? ((t >= 1 && t <= 256) ? pow10th[j + 1] * exact_pow2(e) : 0.0f) : thr10th[j] * exact_pow2(e);
    }
    return T;
}
FCV2_TABLE ScaleTables kScaleTablesInit = make_scale_tables();

FCV2_D ScaleInt scale_int_from_tables(float s, const float* pow_tab, const float* thr_tab) {
    const int k0 = (s > 0.0f) ? scale_int_estimate(s) : -128;
    const float below = thr_tab[k0 + 128], above = thr_tab[k0 + 129];
    int d = 0;
    if (s >= above) d = 1;
    if (s < below) d = -1;
    if (k0 + d > 127 || k0 + d < -128) d = 0;
    ScaleInt r;
    r.k = k0 + d;
    r.s = pow_tab[k0 + 129 + d];
    return r;
}

// ---- launch plan of the row-staged dispatch kernel (host) ---------------------------------------------------------
// A block takes `rows` consecutive tokens of `lpr` lanes each (a lane = 32 elements) and has `threads` = their lanes
// rounded up to whole waves, at most 8 waves.  Its LDS holds a transpose scratch per wave, the packed records, the
// destination rows, the E expert starts (+ 8 words for the block scan) and, for integer metadata, the scale tables;
// 64 KiB at most.  Among the row counts 1..64 that fit, the one with the smallest share of idle lanes wins (the first
// such).  rows = 0: the shape does not fit the kernel.
constexpr uint32_t kWaveScratchBytes = 4096, kRowsPlanThreadsMax = 512;
struct RowsPlan {
    uint32_t rows, threads;
    size_t lds_bytes;
};
static inline RowsPlan rows_plan(uint32_t lpr, uint32_t K, uint32_t row_bytes, bool int_meta, uint32_t E) {
    // Candidates: R rows per block, as many whole waves as they need.  First choice: the count with the fewest idle lanes
    // (the smallest such count).  If that block is larger than four waves and a smaller count fills at least four waves
    // with at most an eighth of their lanes idle, the smallest such count is taken instead: smaller blocks finish their
    // load - quantize - copy sequence sooner (measured on 7168-element rows: one row in four waves, 32 lanes idle,
    // 62.3 us for the call, against two rows in seven full waves, 64.4 us).
    RowsPlan best = {0, 0, 0}, small = {0, 0, 0};
    uint32_t best_idle = ~0u;
    for (uint32_t R = 1; R <= 64 && R * lpr <= kRowsPlanThreadsMax; ++R) {
        const uint32_t waves = (R * lpr + 63) / 64;
        const size_t lds = (size_t)waves * kWaveScratchBytes + (size_t)R * row_bytes + (size_t)R * K * 4 + ((size_t)E + 8) * 4 +
                           (int_meta ? (size_t)(kScaleTablePow + kScaleTableThr) * 4 : 0);
        if (lds > 64 * 1024) break;
        const uint32_t idle = (waves * 64 - R * lpr) * 1024 / (waves * 64);  // idle lanes, in 1/1024 of the block
        if (idle < best_idle) {
            best_idle = idle;
            best = {R, waves * 64, lds};
        }
        if (small.rows == 0 && waves >= 4 && idle <= 128) small = {R, waves * 64, lds};
    }
    if (best.threads > 4 * 64 && small.rows != 0 && small.rows < best.rows) return small;
    return best;
}

// ---- codes (one per byte) -> planes ---------------------------------------------------------------------------
// Field (code >> SH) & (2^W - 1) of each byte, moved to the top W bits of that byte.
template <int W, int SH, int BITS> FCV2_HD uint32_t top_align(uint32_t c) {
    constexpr int lsh = 8 - W - SH;
    constexpr uint32_t m = (((0xFFu << (8 - W)) & 0xFFu) * 0x01010101u);
    uint32_t f = lsh > 0 ? (c << (lsh > 0 ? lsh : 0)) : c;
    // when the field reaches up to the top bit of the code nothing can spill into the next byte
    return (SH + W == BITS && SH == 0) ? f : (f & m);
}

// 8 nibbles: bits 4i..4i+3 = field of element i.
template <int SH, int BITS> FCV2_HD uint32_t pack_plane4(uint32_t c0, uint32_t c1) {
    uint32_t f0 = top_align<4, SH, BITS>(c0), f1 = top_align<4, SH, BITS>(c1);
    uint32_t a0 = (f0 << 4) | f0;  // bytes 1 and 3 hold (e0 | e1 << 4) and (e2 | e3 << 4)
    uint32_t a1 = (f1 << 4) | f1;
    return ((a0 >> 8) & 0xFFu) | ((a0 >> 16) & 0xFF00u) | ((a1 << 8) & 0xFF0000u) | (a1 & 0xFF000000u);
}

// 8 two-bit fields: bits 2i..2i+1 = field of element i (16 bits, nothing above them).  The four fields of a register
// are gathered by one byte dot product with the weights 1, 4, 16, 64 (the masked bytes are field << SH, so the sum is
// the packed byte << SH).
template <int SH, int BITS> FCV2_HD uint32_t pack_plane2(uint32_t c0, uint32_t c1) {
    constexpr uint32_t W = 0x40100401u;
    const uint32_t m0 = (BITS == 2) ? c0 : and_lit<(0x03030303u << SH)>(c0);
    const uint32_t m1 = (BITS == 2) ? c1 : and_lit<(0x03030303u << SH)>(c1);
    const uint32_t d0 = dot4_u8(m0, W, 0u), d1 = dot4_u8(m1, W, 0u);
    return ((d1 << 8) | d0) >> SH;
}

// 8 one-bit fields: bit i = field of element i (8 bits, nothing above them): two byte dot products with the weights 1, 2, 4, 8 and
// 16, 32, 64, 128, the second adding to the first.  The 1-bit plane always holds bit 0 of the code.
template <int SH, int BITS> FCV2_HD uint32_t pack_plane1(uint32_t c0, uint32_t c1) {
    static_assert(SH == 0, "the 1-bit plane is the least significant bit of the code");
    const uint32_t d = dot4_u8(and_lit<0x01010101u>(c0), 0x08040201u, 0u);
    return dot4_u8(and_lit<0x01010101u>(c1), 0x80402010u, d);
}

// ---- planes -> codes --------------------------------------------------------------------------------------------
// 8 one-bit fields (bit i) -> 8 nibbles (bit 4i).
FCV2_HD uint32_t spread1to4(uint32_t x) {
    x = (x | (x << 12)) & 0x000F000Fu;
    x = (x | (x << 6)) & 0x03030303u;
    x = (x | (x << 3)) & 0x11111111u;
    return x;
}
// 8 two-bit fields (bits 2i) -> 8 nibbles (bits 4i).
FCV2_HD uint32_t spread2to4(uint32_t x) {
    x = (x | (x << 8)) & 0x00FF00FFu;
    x = (x | (x << 4)) & 0x0F0F0F0Fu;
    x = (x | (x << 2)) & 0x33333333u;
    return x;
}

// Codes of the 8 elements as two "even/odd" registers: ev = elements 0,2,4,6 one per byte, od = 1,3,5,7.
// p4 / p2 / p1 are the lane's 32 / 16 / 8 bits of the planes; for BITS == 8 use the plane bytes directly.
template <int BITS> FCV2_HD void codes_even_odd(uint32_t p4, uint32_t p2, uint32_t p1, uint32_t& ev, uint32_t& od) {
    using P = Planes<BITS>;
    constexpr uint32_t M = 0x0F0F0F0Fu;
    uint32_t low = 0;  // nibble word of the planes below the 4-bit plane
    if (P::w2) low = spread2to4(p2) << P::sh2;
    if (P::w1) low |= spread1to4(p1);
    if (P::w4) {
        ev = ((p4 & M) << P::sh4) | (low & M);
        od = (((p4 >> 4) & M) << P::sh4) | ((low >> 4) & M);
    } else {
        ev = low & M;
        od = (low >> 4) & M;
    }
    FCV2_KEEP(ev);  // consumers convert byte k directly (v_cvt_f32_ubyte<k>); do not re-derive from the nibbles
    FCV2_KEEP(od);
}

// Codes of 8 elements as four "pair" registers: Q[k] holds element k in bits 0..15 and element k+4 in bits
// 16..31, each zero-extended.  Read as an fp16 denormal, a 16-bit integer q is exactly q * 2^-24, which lets a
// mixed-precision FMA consume the code without a separate integer-to-float conversion.
// 8 bits: p8lo / p8hi are the 8 bytes of the plane.  (2 to 7 bits: codes_pairs16.)
FCV2_HD void codes_pairs_b8(uint32_t p8lo, uint32_t p8hi, uint32_t (&Q)[4]) {
#if defined(__HIP_DEVICE_COMPILE__)
    Q[0] = __builtin_amdgcn_perm(p8hi, p8lo, 0x0C040C00u);
    Q[1] = __builtin_amdgcn_perm(p8hi, p8lo, 0x0C050C01u);
    Q[2] = __builtin_amdgcn_perm(p8hi, p8lo, 0x0C060C02u);
    Q[3] = __builtin_amdgcn_perm(p8hi, p8lo, 0x0C070C03u);
#else
    for (int k = 0; k < 4; ++k) Q[k] = ((p8lo >> (8 * k)) & 0xFFu) | (((p8hi >> (8 * k)) & 0xFFu) << 16);
#endif
}

// ---- 16 elements of a lane -> 8 registers of (element | element) 16-bit halves, for 2 to 7 bits ------------------
// As above, but the fields are only masked, never moved to bit 0: each half ends up holding code << pos with
// zeros around it, and the consumer folds 2^-pos into the scale it multiplies the half with (a half read as an
// fp16 denormal is an exact integer multiple of 2^-24 at any position below bit 10).  PairMap says which element
// sits where.  p2 = 32 bits (elements 0..15), p1 = 16 bits, p4a/p4b = elements 0..7 / 8..15.
template <int BITS> struct PairMap;
template <> struct PairMap<2> {  // 2-bit fields at offset 2e: direct for e = 0..4 (with e + 8), rotated by 10 for 5..7
    static constexpr int n_pos = 5;
    static constexpr int lo(int k) { return k; }
    static constexpr int hi(int k) { return k + 8; }
    static constexpr int pos(int k) { return k < 5 ? 2 * k : 2 * (k - 5); }
    static constexpr int k_of(int e) { return e & 7; }       // the register that holds element e ...
    static constexpr bool in_hi(int e) { return e >= 8; }    // ... and the half of it
};
template <> struct PairMap<3> {  // 2-bit field at offset o with the extra bit below it: o = 2, 4, 6, 8
    static constexpr int n_pos = 4;
    static constexpr int lo(int k) { return k + 1; }
    static constexpr int hi(int k) { return (k + 9) & 15; }
    static constexpr int pos(int k) { return 2 * (k & 3) + 1; }
    static constexpr int k_of(int e) { return (e + 7) & 7; }
    static constexpr bool in_hi(int e) { return e == 0 || e >= 9; }
};
template <> struct PairMap<4> {  // nibbles at offset 0 and 4 of each half, directly and after a rotation by 8
    static constexpr int n_pos = 2;
    static constexpr int lo(int k) { return (k & 3) + 8 * (k >> 2); }
    static constexpr int hi(int k) { return lo(k) + 4; }
    static constexpr int pos(int k) { return 4 * (k & 1); }
    static constexpr int k_of(int e) { return (e & 3) + 4 * (e >> 3); }
    static constexpr bool in_hi(int e) { return ((e >> 2) & 1) != 0; }
};
// 5, 6 and 7 bits: register k holds elements k and k + 8.  Element k of a half sits at bit 2k of the 2-bit plane word, at
// bit k of the 1-bit plane's half and at nibble k & 3 of a register that holds four nibbles per half; the plane shifts
// in codes_pairs16_wide bring its fields next to each other at `pos`.
struct PairMapWide {
    static constexpr int lo(int k) { return k; }
    static constexpr int hi(int k) { return k + 8; }
    static constexpr int k_of(int e) { return e & 7; }
    static constexpr bool in_hi(int e) { return e >= 8; }
};
template <> struct PairMap<5> : PairMapWide { static constexpr int pos(int k) { return k & 1; } };
template <> struct PairMap<6> : PairMapWide { static constexpr int pos(int k) { return k < 3 ? 2 * k : k < 6 ? 2 * (k - 3) : 2 * (k - 6); } };
template <> struct PairMap<7> : PairMapWide { static constexpr int pos(int k) { return k & 1; } };

template <int BITS> constexpr bool pair_map_consistent() {
    using M = PairMap<BITS>;
    for (int k = 0; k < 8; ++k)
        if (M::k_of(M::lo(k)) != k || M::in_hi(M::lo(k)) || M::k_of(M::hi(k)) != k || !M::in_hi(M::hi(k)) || M::pos(k) + BITS > 10) return false;
    return true;
}
static_assert(pair_map_consistent<2>() && pair_map_consistent<3>() && pair_map_consistent<4>() && pair_map_consistent<5>() &&
                  pair_map_consistent<6>() && pair_map_consistent<7>(),
              "PairMap: element <-> (register, half) maps disagree");

// Every mask below is a literal of a two-operand `and` (see the note on instruction forms at the top), shifts go to
// the right wherever a plain shift does, and the one wrap-around that is needed (element 0 of the 3-bit layout) is a
// rotate.
// The 16 bits of the 1-bit plane spread so that the bit of element e sits at 2e - 1, directly below the element's 2-bit
// field of the 2-bit plane at 2e, 2e + 1 (element 0's bit wraps to bit 31).
FCV2_HD uint32_t spread_extra_bits16(uint32_t p1) {
    uint32_t x = and_lit<0x00FF00FFu>((p1 << 8) | p1);  // bit e -> 2e ...
    x = and_lit<0x0F0F0F0Fu>((x << 4) | x);
    x = and_lit<0x33333333u>((x << 2) | x);
    x = and_lit<0x55555555u>((x << 1) | x);
    return rotr32(x, 1);  // ... then turned right by one
}

// 3 bits: the pair registers from the 2-bit plane word and the spread extra bits S.
FCV2_HD void codes_pairs16_b3(uint32_t p2, uint32_t S, uint32_t (&Q)[8]) {
    // even elements: field at 4j, 4j + 1 from the plane, bit at 4j - 1 from S; odd elements: bit at 4j + 1 from S, field
    // at 4j + 2, 4j + 3 from the plane.  One bit-select each, with the same mask.
    const uint32_t M = vreg_const<0x33333333u>();
    const uint32_t We = bit_select(M, p2, S), Wo = bit_select(M, S, p2);
    const uint32_t We8 = rotr32(We, 8), Wo8 = Wo >> 8;  // elements 6, 8 / 14, 0 and 5, 7 / 13, 15 at the same four positions
    Q[0] = and_lit<0x000E000Eu>(Wo);   // elements 1, 9    at bit 1
    Q[1] = and_lit<0x00380038u>(We);   // elements 2, 10   at bit 3
    Q[2] = and_lit<0x00E000E0u>(Wo);   // elements 3, 11   at bit 5
    Q[3] = and_lit<0x03800380u>(We);   // elements 4, 12   at bit 7
    Q[4] = and_lit<0x000E000Eu>(Wo8);  // elements 5, 13
    Q[5] = and_lit<0x00380038u>(We8);  // elements 6, 14
    Q[6] = and_lit<0x00E000E0u>(Wo8);  // elements 7, 15
    Q[7] = and_lit<0x03800380u>(We8);  // elements 8, 0
}

// 5, 6 and 7 bits.  The nibbles of elements k and k + 8 meet in one register (a byte permute each for k < 4 and k >= 4); then
// one shift per plane and register puts a nibble directly above its lower bits, a bit-select joins them and a literal mask
// keeps the element: 5.6, 5.3 and 8.3 VALU cycles per element by the costs above, against 6.9, 6.9 and 11.4 where every field
// was moved to bit 0 and the planes joined with and-or instructions that read scalar masks.
// reduce_requant of 16 M elements, 8 peers, groups of 128 / 256, us before -> after: 5 bits 31.8 -> 31.1 / 31.4 -> 30.7, 6 bits
// 32.3 -> 32.1 / 32.7 -> 31.8, 7 bits 37.6 -> 35.8 / 37.0 -> 34.9.
template <int BITS> FCV2_HD void codes_pairs16_wide(uint32_t p4a, uint32_t p4b, uint32_t p2, uint32_t p1, uint32_t (&Q)[8]) {
#if defined(__HIP_DEVICE_COMPILE__)
    const uint32_t na = __builtin_amdgcn_perm(p4b, p4a, 0x05040100u), nb = __builtin_amdgcn_perm(p4b, p4a, 0x07060302u);
#else
    const uint32_t na = (p4a & 0xFFFFu) | (p4b << 16), nb = (p4a >> 16) | (p4b & 0xFFFF0000u);
#endif
    const uint32_t x1 = (p1 << 8) | p1;  // bit k of each half: elements k and k + 8 (further bits above them)
    if (BITS == 5) {
        const uint32_t n0 = vreg_const<0x001E001Eu>(), n1 = vreg_const<0x003C003Cu>();
        const uint32_t x12 = x1 >> 2, x14 = x1 >> 4, x16 = x1 >> 6;
        Q[0] = and_lit<0x001F001Fu>(bit_select(n0, na << 1, x1));
        Q[1] = and_lit<0x003E003Eu>(bit_select(n1, na >> 2, x1));
        Q[2] = and_lit<0x001F001Fu>(bit_select(n0, na >> 7, x12));
        Q[3] = and_lit<0x003E003Eu>(bit_select(n1, na >> 10, x12));
        Q[4] = and_lit<0x001F001Fu>(bit_select(n0, nb << 1, x14));
        Q[5] = and_lit<0x003E003Eu>(bit_select(n1, nb >> 2, x14));
        Q[6] = and_lit<0x001F001Fu>(bit_select(n0, nb >> 7, x16));
        Q[7] = and_lit<0x003E003Eu>(bit_select(n1, nb >> 10, x16));
    } else if (BITS == 6) {
        const uint32_t n0 = vreg_const<0x003C003Cu>(), n2 = vreg_const<0x00F000F0u>(), n4 = vreg_const<0x03C003C0u>();
        const uint32_t x26 = p2 >> 6, x2c = p2 >> 12;
        Q[0] = and_lit<0x003F003Fu>(bit_select(n0, na << 2, p2));
        Q[1] = and_lit<0x00FC00FCu>(bit_select(n2, na, p2));
        Q[2] = and_lit<0x03F003F0u>(bit_select(n4, na >> 2, p2));
        Q[3] = and_lit<0x003F003Fu>(bit_select(n0, na >> 10, x26));
        Q[4] = and_lit<0x00FC00FCu>(bit_select(n2, nb << 4, x26));
        Q[5] = and_lit<0x03F003F0u>(bit_select(n4, nb << 2, x26));
        Q[6] = and_lit<0x003F003Fu>(bit_select(n0, nb >> 6, x2c));
        Q[7] = and_lit<0x00FC00FCu>(bit_select(n2, nb >> 8, x2c));
    } else {
        const uint32_t n0 = vreg_const<0x00780078u>(), n1 = vreg_const<0x00F000F0u>();   // the nibble ...
        const uint32_t e0 = vreg_const<0x00010001u>(), e1 = vreg_const<0x00020002u>();   // ... and the extra bit, at pos 0 and 1
        const uint32_t x12 = x1 >> 2, x14 = x1 >> 4, x16 = x1 >> 6;
        Q[0] = and_lit<0x007F007Fu>(bit_select(e0, x1, bit_select(n0, na << 3, p2 << 1)));
        Q[1] = and_lit<0x00FE00FEu>(bit_select(e1, x1, bit_select(n1, na, p2)));
        Q[2] = and_lit<0x007F007Fu>(bit_select(e0, x12, bit_select(n0, na >> 5, p2 >> 3)));
        Q[3] = and_lit<0x00FE00FEu>(bit_select(e1, x12, bit_select(n1, na >> 8, p2 >> 4)));
        Q[4] = and_lit<0x007F007Fu>(bit_select(e0, x14, bit_select(n0, nb << 3, p2 >> 7)));
        Q[5] = and_lit<0x00FE00FEu>(bit_select(e1, x14, bit_select(n1, nb, p2 >> 8)));
        Q[6] = and_lit<0x007F007Fu>(bit_select(e0, x16, bit_select(n0, nb >> 5, p2 >> 11)));
        Q[7] = and_lit<0x00FE00FEu>(bit_select(e1, x16, bit_select(n1, nb >> 8, p2 >> 12)));
    }
}

template <int BITS> FCV2_HD void codes_pairs16(uint32_t p4a, uint32_t p4b, uint32_t p2, uint32_t p1, uint32_t (&Q)[8]) {
    if (BITS == 2) {
        const uint32_t B = p2 >> 10;  // element 5 at bit 0, element 13 at bit 16
        Q[0] = and_lit<0x00030003u>(p2);
        Q[1] = and_lit<0x000C000Cu>(p2);
        Q[2] = and_lit<0x00300030u>(p2);
        Q[3] = and_lit<0x00C000C0u>(p2);
        Q[4] = and_lit<0x03000300u>(p2);
        Q[5] = and_lit<0x00030003u>(B);
        Q[6] = and_lit<0x000C000Cu>(B);
        Q[7] = and_lit<0x00300030u>(B);
    } else if (BITS == 3) {
        codes_pairs16_b3(p2, spread_extra_bits16(p1), Q);
    } else if (BITS > 4) {
        codes_pairs16_wide<BITS>(p4a, p4b, p2, p1, Q);
    } else {
        const uint32_t Ba = p4a >> 8, Bb = p4b >> 8;
        Q[0] = and_lit<0x000F000Fu>(p4a);
        Q[1] = and_lit<0x00F000F0u>(p4a);
        Q[2] = and_lit<0x000F000Fu>(Ba);
        Q[3] = and_lit<0x00F000F0u>(Ba);
        Q[4] = and_lit<0x000F000Fu>(p4b);
        Q[5] = and_lit<0x00F000F0u>(p4b);
        Q[6] = and_lit<0x000F000Fu>(Bb);
        Q[7] = and_lit<0x00F000F0u>(Bb);
    }
}

}  // namespace fcv2
