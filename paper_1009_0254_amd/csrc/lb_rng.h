// Device random numbers of the library (private): Philox4x32-10 and Box-Muller.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace lbf {

// ------------------------------------------------------------------ Philox4x32-10
// Salmon, Moraes, Dror & Shaw, SC'11: 10 rounds of two 32x32->64 products with the
// multipliers 0xD2511F53 / 0xCD9E8D57 and a Weyl key schedule 0x9E3779B9 / 0xBB67AE85.
// The three-way exclusive or of a round is one gfx950 v_bitop3_b32 (truth table 0x96).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
__device__ __forceinline__ uint4 philox10(uint4 c, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        const unsigned long long p0 = (unsigned long long)0xD2511F53u * c.x;
        const unsigned long long p1 = (unsigned long long)0xCD9E8D57u * c.z;
        const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
        const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
        // The callers vary only the first counter word across lanes, so some words stay uniform
        // for the first rounds: the first round's products of words 2 and 3 and its x, y; the
        // second round's hi0, lo0 (from that x).  There the exclusive ors pair the uniform
        // operands first (scalar instructions), as a three-way vector or may read only one scalar
        // operand and would need a move for the second; from the third round on one v_bitop3 each.
        if (r == 0)
            c = make_uint4(hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0);
        else if (r == 1)
            c = make_uint4(hi1 ^ (c.y ^ k0), lo1, c.w ^ (hi0 ^ k1), lo0);
        else if (r == 2)
            c = make_uint4(xor3(hi1, c.y, k0), lo1, hi0 ^ (c.w ^ k1), lo0);
        else
            c = make_uint4(xor3(hi1, c.y, k0), lo1, xor3(hi0, c.w, k1), lo0);
    }
    return c;
}

// the six 21-bit integers of one Philox block: the top 21 bits of each word, then the
// low 11 bits of words (0,1) and (2,3) joined (dropping one bit of words 1 and 3)
__device__ __forceinline__ void bits21(uint4 x, uint32_t b[6])
{
    b[0] = x.x >> 11;
    b[1] = x.y >> 11;
    b[2] = x.z >> 11;
    b[3] = x.w >> 11;
    b[4] = ((x.x & 0x7FFu) << 10) | ((x.y & 0x7FFu) >> 1);
    b[5] = ((x.z & 0x7FFu) << 10) | ((x.w & 0x7FFu) >> 1);
}

// ------------------------------------------------------------------ FP64 reciprocal and square root
// The compiler's FP64 division and square root guard every argument (scaling, special cases), 11 and
// about 17 instructions; the ranges here need less.  Both start from the hardware's ~2^-24 estimate:
// Newton's iteration doubles the correct bits, and the last residual, formed with fma, leaves one
// rounding of a value within ~2^-40 ulp of the exact one.  The host build takes the correctly rounded
// operations, which differ only beside a midpoint of two doubles (device against those, 2 million
// arguments each: no quotient, 12 reciprocals, 2 reciprocal roots, and the roots of 1 - k 2^-53 for odd k).

// 1 / v; zero, infinite and NaN arguments as the division has them
__host__ __device__ inline double rcp64(double v)
{
#if defined(__HIP_DEVICE_COMPILE__)
    double y = __builtin_amdgcn_rcp(v);
    y = fma(fma(-v, y, 1.0), y, y);
    y = fma(fma(-v, y, 1.0), y, y);
    return __builtin_amdgcn_div_fixup(y, v, 1.0);
#else
    return 1.0 / v;
#endif
}

// a / v for a = 0 or |a| of 2^-900 to 2^900 and normal v whose quotient is normal
__host__ __device__ inline double div64(double a, double v)
{
#if defined(__HIP_DEVICE_COMPILE__)
    double y = __builtin_amdgcn_rcp(v);
    y = fma(fma(-v, y, 1.0), y, y);
    const double q = a * y;
    return fma(fma(-v, q, a), y, q);
#else
    return a / v;
#endif
}

// sqrt(x) for finite x >= 0, NaN for a NaN and for +infinity (where the populations are not finite either).  The clamp, at the smallest positive double,
// keeps the estimate finite for x = 0 only; below the normal range the residual of the last line rounds
// away and what is left is Newton's step from the estimate, within 2^-44
__host__ __device__ inline double sqrt64(double x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const double y = __builtin_amdgcn_rsq(fmax(x, 0x1p-1074));
    double g = x * y;
    const double h = 0.5 * y;
    g = fma(fma(-h, g, 0.5), g, g);
    return fma(fma(-g, g, x), h, g);
#else
    return sqrt(x);
#endif
}

// the same with the reciprocal of the root: r = sqrt(x), ir = 1 / r for normal x > 0
__host__ __device__ inline void sqrt_rsqrt64(double x, double &r, double &ir)
{
#if defined(__HIP_DEVICE_COMPILE__)
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double e = fma(-h, g, 0.5);
    g = fma(e, g, g);
    h = fma(e, h, h);
    r = fma(fma(-g, g, x), h, g);
    const double i = h + h;
    ir = fma(fma(-r, i, 1.0), i, i);
#else
    r = sqrt(x);
    ir = 1.0 / r;
#endif
}

// ------------------------------------------------------------------ FP64 ln u, sin and cos of 2 pi u
// Box-Muller meets these only at u = (b + 1/2) 2^-21 with b a 21-bit integer, which admits exact
// argument reductions and short series instead of the general-argument library routines.  The
// series are least-maximum fits over the reduced ranges (Lawson's reweighted least squares in 80-bit
// arithmetic, coefficients rounded to double), their own error below 2e-17 of the result.  The
// operations are products, sums, explicit fma, one quotient and bit manipulation; a host build of these
// functions gives the same bits (both compared over every b with each other and with long double).

// ln u: u = (b + 1/2) 2^-21 = (2 b + 1) 2^-22 (exact) = m 2^e with m in [sqrt(1/2), sqrt(2)), m - 1 exact; ln m =
// 2 atanh(s), s = (m - 1) / (m + 1), |s| <= 0.1716: 2 s + 2 s^3 p(s^2) with p of degree 6; e ln 2
// with ln 2 = hi + lo, hi being ln 2 rounded to 40 significant bits (so that e hi is exact for
// |e| <= 22) and lo the rest rounded to double.
__host__ __device__ inline double u21_ln(uint32_t b)
{
    const double u = (double)(2u * b + 1u) * 0x1p-22;
    const unsigned long long bits = __builtin_bit_cast(unsigned long long, u);
    // exponent and mantissa from the high word, the mantissa's bound at sqrt(2) cut to that word
    const uint32_t hw = (uint32_t)(bits >> 32), up = (hw & 0xFFFFFu) > 0x6A09Eu ? 1u : 0u;
    const int e = (int)(hw >> 20) - 1023 + (int)up;
    const uint32_t mw = (hw & 0xFFFFFu) | (0x3FF00000u - (up << 20));
    const double m = __builtin_bit_cast(double, ((unsigned long long)mw << 32) | (bits & 0xFFFFFFFFull));
    const double f = m - 1.0;
    const double sv = div64(f, 2.0 + f);
    const double z = sv * sv;
    double p = 0x1.2f05742c2aeaep-4;
    p = fma(p, z, 0x1.39a1b9258881cp-4);
    p = fma(p, z, 0x1.74663ef8f8529p-4);
    p = fma(p, z, 0x1.c71c5208f4cd4p-4);
    p = fma(p, z, 0x1.24924941f1f1ap-3);
    p = fma(p, z, 0x1.999999997fd9cp-3);
    p = fma(p, z, 0x1.5555555555592p-2);
    const double s2 = 2.0 * sv;
    const double lnm = fma(s2 * z, p, s2);
    const double de = (double)e;
    return fma(de, 0x1.62e42fefa4000p-1, fma(de, -0x1.8432a1b0e2634p-43, lnm));
}

// sin and cos of 2 pi u: the angle is n pi 2^-21 with n = 2 b + 1; its quarter turn q = b >> 19 and
// the odd rest m = n mod 2^20 reduce it exactly to x = m' pi 2^-21 in (0, pi/4], m' = m or, past
// the eighth turn (bit 18 of b), 2^20 - m with sine and cosine exchanged; they are exchanged again in
// the odd quarters, sin is negative in the last two and cos in the middle two.
__host__ __device__ inline void u21_sincos_turn(uint32_t b, double &sn, double &cs)
{
    const uint32_t past = (uint32_t)((int32_t)(b << 13) >> 31);   // all ones when bit 18 is set
    const uint32_t m = (((2u * b + 1u) ^ past) & 0xFFFFFu) | 1u;
    const double x = (double)m * 0x1.921fb54442d18p-20;   // pi 2^-21
    const double z = x * x;
    double ps = 0x1.5d92fa85c3980p-33;
    ps = fma(ps, z, -0x1.ae5e660a2b2c3p-26);
    ps = fma(ps, z, 0x1.71de357755567p-19);
    ps = fma(ps, z, -0x1.a01a019c11080p-13);
    ps = fma(ps, z, 0x1.111111110f876p-7);
    ps = fma(ps, z, -0x1.5555555555549p-3);
    const double sx = fma(x * z, ps, x);
    double pc = -0x1.8fb15f588136cp-37;
    pc = fma(pc, z, 0x1.1ee9f120bd1d2p-29);
    pc = fma(pc, z, -0x1.27e4f81155b54p-22);
    pc = fma(pc, z, 0x1.a01a019cbb6dcp-16);
    pc = fma(pc, z, -0x1.6c16c16c151dbp-10);
    pc = fma(pc, z, 0x1.555555555554cp-5);
    pc = fma(pc, z, -0.5);
    const double cx = fma(z, pc, 1.0);
    const bool swap = ((b + (1u << 18)) & (1u << 19)) != 0;   // bit 18 xor bit 19
    const double s0 = swap ? cx : sx, c0 = swap ? sx : cx;
    const unsigned long long ss = (unsigned long long)((b << 11) & 0x80000000u) << 32;
    const unsigned long long sc = (unsigned long long)(((b + (1u << 19)) << 11) & 0x80000000u) << 32;
    sn = __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, s0) ^ ss);
    cs = __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, c0) ^ sc);
}

template <typename R> struct Gauss;

// the angle's revolutions plus one whole turn, 1 + (b + 1/2) 2^-21, assembled from the bits
// (exponent of 1, mantissa 4 b + 2): v_sin/v_cos take revolutions, so the added turn changes
// nothing and saves the conversion
__device__ __forceinline__ float turn21(uint32_t b) { return __builtin_bit_cast(float, 0x3F800002u | (b << 2)); }

template <> struct Gauss<float> {
    static __device__ __forceinline__ void pair(uint32_t be, uint32_t bo, float &a, float &b)
    {
#pragma clang fp contract(on)
        const float ue = __builtin_fmaf((float)be, 0x1p-21f, 0x1p-22f);   // (be + 1/2) 2^-21, exact
        const float uo = turn21(bo);
        // -2 ln u = -2 ln(2) log2(u); v_log_f32 is log2, v_sin/v_cos take revolutions
        const float r = __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(ue));
        a = r * __builtin_amdgcn_cosf(uo);
        b = r * __builtin_amdgcn_sinf(uo);
    }
};

template <> struct Gauss<double> {
    static __device__ __forceinline__ void pair(uint32_t be, uint32_t bo, double &a, double &b)
    {
#pragma clang fp contract(on)
        const double r = sqrt64(-2.0 * u21_ln(be));
        double s, c;
        u21_sincos_turn(bo, s, c);
        a = r * c;
        b = r * s;
    }
};

// Box-Muller with the radius scaled.  noise_scale(v, sqrt(v)) is what the pairs take for normals of
// variance v: the root in float; v itself in double, where it goes under the radius' root.
template <typename R> __device__ __forceinline__ R noise_scale(R var, R root) { return sizeof(R) == 8 ? var : root; }
template <typename R> __device__ __forceinline__ void gauss_pair_scaled(uint32_t be, uint32_t bo, R scale, R &a, R &b);
template <> __device__ __forceinline__ void gauss_pair_scaled<float>(uint32_t be, uint32_t bo, float scale, float &a, float &b)
{
#pragma clang fp contract(on)
    const float ue = __builtin_fmaf((float)be, 0x1p-21f, 0x1p-22f);
    const float uo = turn21(bo);
    const float r = __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(ue)) * scale;
    a = r * __builtin_amdgcn_cosf(uo);
    b = r * __builtin_amdgcn_sinf(uo);
}
template <> __device__ __forceinline__ void gauss_pair_scaled<double>(uint32_t be, uint32_t bo, double scale, double &a, double &b)
{
#pragma clang fp contract(on)
    const double r = sqrt64(-2.0 * u21_ln(be) * scale);
    double s, c;
    u21_sincos_turn(bo, s, c);
    a = r * c;
    b = r * s;
}

// the six normals of (node, rep, t) of the variance that `scale` (noise_scale) stands for
template <typename R>
__device__ __forceinline__ void normals6s(uint32_t node, uint32_t rep, unsigned long long t, uint32_t k0,
                                          uint32_t k1, R scale, R nu[6])
{
    const uint4 x = philox10(make_uint4(node, rep, (uint32_t)t, (uint32_t)(t >> 32)), k0, k1);
    uint32_t b[6];
    bits21(x, b);
    gauss_pair_scaled<R>(b[0], b[1], scale, nu[0], nu[1]);
    gauss_pair_scaled<R>(b[2], b[3], scale, nu[2], nu[3]);
    gauss_pair_scaled<R>(b[4], b[5], scale, nu[4], nu[5]);
}

template <typename R>
__device__ __forceinline__ void normals6(uint32_t node, uint32_t rep, unsigned long long t, uint32_t k0,
                                         uint32_t k1, R nu[6])
{
    const uint4 x = philox10(make_uint4(node, rep, (uint32_t)t, (uint32_t)(t >> 32)), k0, k1);
    uint32_t b[6];
    bits21(x, b);
    Gauss<R>::pair(b[0], b[1], nu[0], nu[1]);
    Gauss<R>::pair(b[2], b[3], nu[2], nu[3]);
    Gauss<R>::pair(b[4], b[5], nu[4], nu[5]);
}

// element at a 32-bit byte offset from a uniform base (lets the compiler address with an
// SGPR base and one 32-bit VGPR offset)
}  // namespace lbf
