// gem_device.hpp -- device-side numerics of the GEM commit pipeline (gfx950).
//
// Counter-based noise and the elementwise GEM step, evaluated in IEEE binary32
// with round-to-nearest-even in a fixed operation order: explicit fma where
// written, correctly rounded division and square root (hipcc's IEEE lowering
// on gfx950, or its core steps where the operand range leaves the rest
// nothing to do), denormals kept, no contraction (built with
// -ffp-contract=off).
// Any IEEE implementation of the same steps -- in particular the host-side
// test oracle, written separately -- produces the same bits.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gemk {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror & Shaw, SC'11).  Each round multiplies
// words 0 and 2 by the two Philox multipliers and mixes the high halves with
// the odd words and the key; the key advances by the two Weyl increments
// after every round.
// ---------------------------------------------------------------------------
struct Words4 {
    uint32_t x0, x1, x2, x3;
};

// a ^ b ^ c.  On the device one V_BITOP3_B32 (gfx950's three-input bitwise
// operation; truth table 0x96 is the odd-parity function), which the compiler
// does not form from two XORs by itself.
__host__ __device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
#else
    return a ^ b ^ c;
#endif
}

__host__ __device__ __forceinline__ Words4 philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                          uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t pa = static_cast<uint64_t>(0xD2511F53u) * c0;
        const uint64_t pb = static_cast<uint64_t>(0xCD9E8D57u) * c2;
        const uint32_t y0 = xor3(static_cast<uint32_t>(pb >> 32), c1, k0);
        const uint32_t y2 = xor3(static_cast<uint32_t>(pa >> 32), c3, k1);
        c1 = static_cast<uint32_t>(pb);
        c3 = static_cast<uint32_t>(pa);
        c0 = y0;
        c2 = y2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return Words4{c0, c1, c2, c3};
}

// The same for the noise's counters (q_lo, q_hi, t, 0), whose q_hi and keys are
// uniform.  What a commit loop's compiler can keep or compute once is grouped
// so that it does: the first round's product with q_lo does not depend on t,
// nor does the second round's with word 2; with a uniform t (UNIFORM) the
// other two products of these rounds and their XORs are scalar.  The rest is
// two products and two XORs a round from the third on: 34 vector instructions
// a commit, 42 before they were grouped.
template <bool UNIFORM>
__device__ __forceinline__ Words4 philox10_noise(uint32_t q_lo, uint32_t q_hi, uint32_t t,
                                                 uint32_t k0, uint32_t k1)
{
    constexpr uint32_t kM0 = 0xD2511F53u, kM1 = 0xCD9E8D57u, kW0 = 0x9E3779B9u, kW1 = 0xBB67AE85u;
    uint64_t pa = static_cast<uint64_t>(kM0) * q_lo;
    uint64_t pb = static_cast<uint64_t>(kM1) * t;
    uint32_t c0 = static_cast<uint32_t>(pb >> 32) ^ (q_hi ^ k0);
    uint32_t c2 = static_cast<uint32_t>(pa >> 32) ^ k1;
    uint32_t c1 = static_cast<uint32_t>(pb), c3 = static_cast<uint32_t>(pa);
    k0 += kW0;
    k1 += kW1;
    pa = static_cast<uint64_t>(kM0) * c0;
    pb = static_cast<uint64_t>(kM1) * c2;
    c0 = c1 ^ (static_cast<uint32_t>(pb >> 32) ^ k0);
    c2 = static_cast<uint32_t>(pa >> 32) ^ (c3 ^ k1);
    c1 = static_cast<uint32_t>(pb);
    c3 = static_cast<uint32_t>(pa);
#pragma unroll
    for (int r = 2; r < 10; ++r) {
        k0 += kW0;
        k1 += kW1;
        pa = static_cast<uint64_t>(kM0) * c0;
        pb = static_cast<uint64_t>(kM1) * c2;
        c0 = xor3(static_cast<uint32_t>(pb >> 32), c1, k0);
        c2 = UNIFORM && r == 2 ? static_cast<uint32_t>(pa >> 32) ^ (c3 ^ k1)
                               : xor3(static_cast<uint32_t>(pa >> 32), c3, k1);
        c1 = static_cast<uint32_t>(pb);
        c3 = static_cast<uint32_t>(pa);
    }
    return Words4{c0, c1, c2, c3};
}

// ---------------------------------------------------------------------------
// Correctly rounded division and square root for operand ranges where the
// general IEEE sequences' range handling has nothing to do.  hipcc lowers a / b
// to scale operands near the ends of the exponent range, refine a hardware
// reciprocal by Newton steps with fma residual corrections, and fix up special
// values; sqrt(x) likewise scales and fixes up.  On operands with no scaling
// and no special value fewer steps give the same, correctly rounded, result --
// which the self-test library checks exhaustively over the domains used below
// and on a wide random sample for the guarded quotient.
// ---------------------------------------------------------------------------

// a / b, correctly rounded, for normal b and a quotient well inside the
// normal range (no scaling of either operand).  The reciprocal takes one Newton
// step, the quotient one residual correction: correctly rounded for all 2^46
// pairs of significands (the self-test library checks each on the device; the
// steps commute with scaling by powers of two in this range).  Correcting with
// the unrefined reciprocal fails on 26473 of those pairs.
__device__ __forceinline__ float div_rn_core(float a, float b)
{
    float r = __builtin_amdgcn_rcpf(b);
    const float e = __builtin_fmaf(-b, r, 1.0f);
    r = __builtin_fmaf(e, r, r);                    // refined reciprocal
    const float q = a * r;
    const float e2 = __builtin_fmaf(-b, q, a);
    return __builtin_fmaf(e2, r, q);
}

// The product by the rule that zero times anything is zero (V_MUL_LEGACY_F32;
// the compiler has the intrinsic but no builtin for it).
__device__ float mul_legacy(float a, float b) __asm("llvm.amdgcn.fmul.legacy");

// -sqrt(-x), the root correctly rounded, for the negated Box-Muller radicands
// x = 2 ln(k 2^-24), k in [1, 2^24] (+0 or in [-33.3, -1.1e-7]).  One Newton step
// from the hardware reciprocal root y of -x: n = x y, the negated root, then
// n + (n^2 + x) (y / 2).  The step is the correctly rounded root for every one of
// the 2^24 radicands (the self-test library checks all of them on the device).
// Four instructions and the root; stepping v_sqrt's result to the neighbour with
// the right residual sign takes eight.  y / 2 is an integer step of the exponent.
//
// The signs are turned for u = 1, whose radius is sqrt(-2 ln 1) = sqrt(-0) = -0.
// There x is +0 and y is -inf; the legacy product, whose zero times anything is
// +0, makes n = +0, and the step ends in (+0) (-2^127) + (+0) = +0: the radius
// negated, with its sign.  (With r = x y from a positive x it would be +0 as well.)
// They also spare the two multiply-adds their source modifiers, which take the
// longer encoding.
__device__ __forceinline__ float neg_radius(float x)
{
    const float y = __builtin_amdgcn_rsqf(-x);
    const float n = mul_legacy(x, y);
    const float half_y = __uint_as_float(__float_as_uint(y) - 0x00800000u);
    const float e = __builtin_fmaf(n, n, x);
    return __builtin_fmaf(e, half_y, n);
}

// num / den, correctly rounded for every input: the core steps when both
// magnitudes lie in [2^-60, 2^60] (quotient in [2^-120, 2^120]), the general
// division otherwise (zero, tiny, huge, infinite or NaN operands).
__device__ __forceinline__ float div_rn(float num, float den)
{
    const float an = __builtin_fabsf(num), ad = __builtin_fabsf(den);
    const bool core = an >= 0x1p-60f && an <= 0x1p60f && ad >= 0x1p-60f && ad <= 0x1p60f;
    float q;
    if (core) q = div_rn_core(num, den);
    else q = num / den;
    return q;
}

// (f - 1) / (f + 1), correctly rounded, for the binary32 f in (sqrt(1/2),
// sqrt(2)] the logarithm below reduces to (or that times a power of two): the
// hardware reciprocal r of f + 1 and one residual correction of the quotient
// (f - 1) r.  f - 1 is exact,
// f + 1 lies in (1.7, 2.5), and on these 2^23 operand pairs the two steps
// give the correctly rounded quotient every time (the self-test library
// checks all of them on the device against the IEEE division); the general
// core above takes four more steps.
__device__ __forceinline__ float ln_quotient(float a, float b)
{
    const float r = __builtin_amdgcn_rcpf(b);
    const float q = a * r;
    const float e = __builtin_fmaf(-b, q, a);
    return __builtin_fmaf(e, r, q);
}

// ---------------------------------------------------------------------------
// 2 ln u of u = k * 2^-24, k in [1, 2^24]: the Box-Muller radicand -2 ln u, negated.
// u = 2^e f with f in (sqrt(1/2), sqrt(2)]; ln f = 2 atanh((f-1)/(f+1)) by its
// series to the s^9 term (Abramowitz & Stegun 4.1.27); ln u = e ln2 + ln f
// with ln 2 split into a 15-bit head and a binary32 tail so that e * head is
// exact.
//
// The defined steps are p = ((s^2/9 + 1/7) s^2 + 1/5) s^2 + 1/3, p s^2, then
// ln f = fma(2s, p s^2, 2s), ln u = fma(e, head, fma(e, tail, ln f)) and the
// radicand -2 ln u.  Here every value carries the power-of-two factor that
// makes the doublings disappear: s' = 4 s (the quotient of 4 (f - 1), exact),
// s'^2 = 16 s^2 against coefficients divided by 16 per degree, and the tail and
// head times 2.  Scaling by a power of two commutes with rounding (nothing here
// is subnormal or overflows), so the bits are those of the defined steps, in 2
// instructions fewer.
//
// The reduction works on the integer: k as binary32 (exact) has u's
// significand and an exponent 24 larger; subtracting the bits of 2^24 * the
// least binary32 above sqrt(1/2) leaves e in the bits above the significand.
// Those bits alone, as an integer, are e 2^23 (the constants of e carry 2^-23),
// and k's bits less them are 2^24 f: the quotient of 2^24 (f - 1) and
// 2^24 (f + 1) is the same.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float neg_radicand_of_k24(uint32_t k)
{
    constexpr uint32_t kLeast = 0x3F3504F4u;   // least binary32 above sqrt(1/2)
    const uint32_t bits = __float_as_uint(static_cast<float>(k));
    const uint32_t eb = (bits - (kLeast + (24u << 23))) & 0xFF800000u;
    const float ef = static_cast<float>(static_cast<int32_t>(eb));          // 2^23 e
    const float f = __uint_as_float(bits - eb);                             // 2^24 f
    const float s = ln_quotient(__builtin_fmaf(f, 4.0f, -0x1p26f), f + 0x1p24f);   // 4 (f-1)/(f+1)
    const float z = s * s;
    float p = (1.0f / 9.0f) * 0x1p-16f;
    p = __builtin_fmaf(p, z, (1.0f / 7.0f) * 0x1p-12f);
    p = __builtin_fmaf(p, z, (1.0f / 5.0f) * 0x1p-8f);
    p = __builtin_fmaf(p, z, (1.0f / 3.0f) * 0x1p-4f);
    p = p * z;
    const float ln_f = __builtin_fmaf(s, p, s);   // 2 ln f
    const float ln2_tail = 0x1.7f7d1cp-20f;       // RN(ln 2 - ln2_head)
    const float ln2_head = 0x1.62e4p-1f;
    const float r = __builtin_fmaf(ef, 2.0f * ln2_tail * 0x1p-23f, ln_f);
    return __builtin_fmaf(ef, 2.0f * ln2_head * 0x1p-23f, r);
}

// r cos(phi) and r sin(phi) for phi = 2 pi (xb >> 8) / 2^24, from neg_r = -r.
// With k = xb >> 8, the angle is reduced to the nearest quarter turn on the
// integer, exactly; the rest, |x| <= pi/4, goes through the Taylor series of sin
// (to x^9) and cos (to x^10).  k minus its nearest multiple of 2^22 is k's low 22
// bits read as a signed number.
//
// Quadrant q (bits 30 and 31 of xb + 2^29): (sin, cos) = (sx, cx), (cx, -sx),
// (-sx, -cx), (-cx, sx): an odd quadrant takes (cx, -sx), and quadrants 2 and
// 3 negate both, which here goes into r's sign before the two products (a
// product's bits but for its sign do not depend on its factors' signs).  r may
// be of either sign, zeros included: the radius of u1 = 1 is -0.
__device__ __forceinline__ void turn_times(float neg_r, uint32_t xb, float& zc, float& zs)
{
    const int rem = static_cast<int>(xb << 2) >> 10;
    const float step = 6.28318530717958647692f * 0x1p-24f;   // RN(2 pi) 2^-24
    const float x = static_cast<float>(rem) * step;
    const float x2 = x * x;

    float ps = 1.0f / 362880.0f;
    ps = __builtin_fmaf(ps, x2, -1.0f / 5040.0f);
    ps = __builtin_fmaf(ps, x2, 1.0f / 120.0f);
    ps = __builtin_fmaf(ps, x2, -1.0f / 6.0f);
    ps = ps * x2;
    const float sx = __builtin_fmaf(x, ps, x);

    float pc = -1.0f / 3628800.0f;
    pc = __builtin_fmaf(pc, x2, 1.0f / 40320.0f);
    pc = __builtin_fmaf(pc, x2, -1.0f / 720.0f);
    pc = __builtin_fmaf(pc, x2, 1.0f / 24.0f);
    pc = __builtin_fmaf(pc, x2, -0.5f);
    const float cx = __builtin_fmaf(pc, x2, 1.0f);

    // bit 30 of y = xb + 2^29: |y| as a binary32 is at least 2 (or a NaN) with it
    const uint32_t y = xb + 0x20000000u;
    const bool odd = !(__builtin_fabsf(__uint_as_float(y)) < 2.0f);
    // neg_r ^ (~y & sign bit): one V_BITOP3_B32 (a ^ (~b & c), table 0xD2)
    const float rs = __uint_as_float(__builtin_amdgcn_bitop3_b32(
        __float_as_uint(neg_r), y, 0x80000000u, 0xD2));
    zs = rs * (odd ? cx : sx);
    zc = rs * (odd ? -sx : cx);
}

// Box-Muller (1958): from two words, u1 = ((xa >> 8) + 1) 2^-24 in (0, 1] and
// the angle index xb >> 8, the pair r cos(phi), r sin(phi), r = sqrt(-2 ln u1).
__device__ __forceinline__ void box_muller(uint32_t xa, uint32_t xb, float& zc, float& zs)
{
    turn_times(neg_radius(neg_radicand_of_k24((xa >> 8) + 1u)), xb, zc, zs);
}

// Four standard normals for elements 4q..4q+3 at clock t.  UNIFORM: t is the
// same for the whole wave.
template <bool UNIFORM = true>
__device__ __forceinline__ float4 normals4(uint64_t q, uint32_t t, uint32_t k0, uint32_t k1)
{
    const Words4 w = philox10_noise<UNIFORM>(static_cast<uint32_t>(q),
                                             static_cast<uint32_t>(q >> 32), t, k0, k1);
    float4 z;
    box_muller(w.x0, w.x1, z.x, z.y);
    box_muller(w.x2, w.x3, z.z, z.w);
    return z;
}

// Two binary32 values rounded to bfloat16, nearest-even (a NaN stays a quiet
// NaN), packed low half first: one V_CVT_PK_BF16_F32.  The integer steps of the
// rounding take 7 instructions for each value; the self-test library checks
// all 2^32 inputs against them.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

// Both values rounded to bfloat16, as binary32.
__device__ __forceinline__ void round_pair_to_bf16(float& a, float& b)
{
    const uint32_t p = pack_bf16(a, b);
    a = __uint_as_float(p << 16);
    b = __uint_as_float(p & 0xFFFF0000u);
}

}  // namespace gemk
