// Device arithmetic of the per-row int4 quantizer, shared by the kernels that quantize a row they
// have just produced (quantize.hip, glue.hip).  Device code only.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

namespace sqap {

// Correctly rounded binary32 quotient v / s (IEEE division) for a half scale s and any binary32 v, with 1 / s in two parts formed
// once per row: hi = RN(1 / s), lo what that lacks.  hi + lo is within 2^-47 of 1 / s, and so is the sum that the multiply-add
// rounds, once; v / s is never that close to a midpoint of binary32: it is not one (25 odd bits times s would not fit v's
// 24), and v minus the midpoint times s is a whole number of units, which leaves at least 2^-12 ulp, 2^-36 of v / s.  Two instructions instead of the
// ~15 of a full IEEE division per element, or three with the remainder; every half / half pair is compared against the division operator by
// sqap_selftest_quotient.  (Quotients so small that v * lo underflows are code 0 either way.)
struct Reciprocal {
    float hi, lo;
};
__device__ __forceinline__ float quotient(float v, const Reciprocal &r) { return fmaf(v, r.hi, v * r.lo); }

// clamp(rint(q), -8, 7) as a 4-bit two's complement code, the low bits of the result.  Clamping first gives the same integer (both
// bounds are integers and rounding is monotone), and adding 1.5 * 2^23 rounds a value of that size to
// the nearest integer, ties to even like rint, and leaves it in the low mantissa bits: one addition
// instead of a rounding and a conversion.  A NaN quotient clamps to -8 either way.
__device__ __forceinline__ uint32_t code_bits(float q)       // the code in two's complement, added to kCodeBias
{
    return __float_as_uint(__builtin_amdgcn_fmed3f(q, -8.f, 7.f) + 12582912.0f);
}
constexpr uint32_t kCodeBias = 0x4b400000u;                   // the bits of 1.5 * 2^23

// Eight codes in a word, the first in the low bits.  Shifted and added as they come, one instruction each, they and their biases make one
// sum modulo 2^32; raised by 8 every code is a digit of 0 .. 15 and nothing carries, and the digit's top bit is the code's turned over.
__device__ __forceinline__ uint32_t pack_codes8(const float (&q)[8])
{
    uint32_t sum = code_bits(q[7]);
#pragma unroll
    for (int e = 6; e >= 0; --e) sum = (sum << 4) + code_bits(q[e]);
    return (sum + (0x88888888u - kCodeBias * 0x11111111u)) ^ 0x88888888u;
}

// scale = half(float(max|v| / 7)), the smallest subnormal when that rounds to zero (an all-zero row).  The division by the remainder of an estimate (7 is
// a half value): five instructions that wait for each other instead of a dozen.  An infinite maximum stays infinite: what the finite
// largest value lacks is infinite.  Two roundings, of which the first decides at ties between two halves: without the empty asm the last
// multiply-add and the conversion become one instruction that rounds once.  sqap_selftest_quotient compares all binary32 maxima with the division
// operator.
__device__ __forceinline__ __half row_scale(float amax)
{
    constexpr float seventh = 1.0f / 7.0f;
    const float q0 = fminf(amax * seventh, 3.402823466e+38f);
    float q = fmaf(fmaf(-q0, 7.0f, amax), seventh, q0);
    asm volatile("" : "+v"(q));
    __half sh = __float2half_rn(q);
    if (__half_as_ushort(sh) == 0) sh = __ushort_as_half((unsigned short)1);
    return sh;
}

// 1 / s of a finite half scale s: RN(1 / s) by one Newton step on the hardware's estimate (sqap_selftest_quotient compares all of them with the
// division operator), and the rest.  An infinite scale gives NaN, and quotients over it are NaN either way.
__device__ __forceinline__ Reciprocal scale_reciprocal(float s)
{
    const float y = __builtin_amdgcn_rcpf(s), hi = fmaf(fmaf(-s, y, 1.0f), y, y);
    return {hi, fmaf(-s, hi, 1.0f) * hi};
}

// Adds the squares of eight half values (held as floats), times 2^48, to the 128-bit integer hi:lo: exactly.
// A half is an integer m < 2^11 times 2^e, e >= -24, so x^2 * 2^48 is an integer below 2^80: m^2 shifted by 2 e + 48.
// (Asked for by the rare row that norm_factor_of leaves open: few registers, no more, next to a row that is held in them.)
__device__ __forceinline__ void add_squares8(const float (&v)[8], unsigned long long &hi, unsigned long long &lo)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        float x = v[e];
        asm volatile("" : "+v"(x), "+v"(lo));              // (one element after the other)
        const unsigned bits = __half_as_ushort(__float2half_rn(x));         // exact: v is a half value
        const unsigned exh = (bits >> 10) & 31u, man = bits & 1023u;
        const unsigned m = exh ? man + 1024u : man;
        const int sh = exh ? 2 * (int)exh - 2 : 0;                          // 2e + 48, at most 60
        const unsigned long long m2 = m * m;                                // below 2^22
        const unsigned long long add_lo = m2 << sh;
        const unsigned long long add_hi = sh > 42 ? m2 >> (64 - sh) : 0ull;
        lo += add_lo;
        hi += add_hi + (lo < add_lo ? 1ull : 0ull);
    }
}

// (float)(1 / sqrt(S / K + eps)) in binary64 of the exact sum: rounded to binary64 once (its top 64 bits with a sticky last bit, then the
// hardware's conversion, which rounds to nearest even).
__device__ __forceinline__ float exact_norm_factor(unsigned long long hi, unsigned long long lo, int K, float eps)
{
    double S;
    if (hi == 0) {
        S = (double)lo;
    } else {
        const int lz = __clzll((long long)hi);
        unsigned long long top = lz ? (hi << lz) | (lo >> (64 - lz)) : hi;
        const unsigned long long rest = lz ? lo << lz : lo;
        top |= rest != 0 ? 1ull : 0ull;
        S = ldexp((double)top, 64 - lz);
    }
    return (float)(1.0 / sqrt(ldexp(S, -48) / (double)K + (double)eps));
}

// r = (float)(1 / sqrt(S / K + eps)) of the RMSNorm from a sum of squares that is merely close: where everything within kNormReach of the
// estimate rounds to one binary32 value, that value is r, and true is returned.  `sum`: the squares (exact in binary64) added in binary64
// in any order.  With K <= 16384 and at least 256 threads a value goes through at most 64 + 7 + 16 additions, so the sum is off by
// less than 87 * 2^-53 of itself, its half power by half of that; mean, eps, the step below and the definition's own roundings add
// less than 12 * 2^-53: 55 * 2^-53 < 2^-47 in all.  The step is of third order: an error e of the hardware's estimate (tested: the squared
// one below 2^-18) leaves 5/16 e^3 < 2^-55.  About one row in 2^18 is open, and one that is not finite or has no norm: the exact sum decides.
constexpr double kNormReach = 0x1p-44;
__device__ __forceinline__ bool norm_factor_of(double sum, double inv_k, float eps, float &r)
{
    const double a = fma(sum, inv_k, (double)eps);
    double y = __builtin_amdgcn_rsq(a);
    const double e = fma(-a * y, y, 1.0);
    y = fma(y * e, fma(e, 0.375, 0.5), y);
    r = (float)(y * (1.0 - kNormReach));
    return r == (float)(y * (1.0 + kNormReach)) && fabs(e) < 0x1p-18;
}

// silu(g) = (float)(g / (1 + exp(-g))) as the definition evaluates it in binary64, for a half value g: the same binary32
// bits for every one of the 65536 halves (infinities and NaN among them).  exp(-g) = 2^k 2^f, |f| <= 1/2, with
// 2^f = 1 + f q(f) (q interpolated at Chebyshev nodes), which is exact where |g| is tiny and g / 2 + g^2 / 4 may end on
// a binary32 tie; the power of two enters the sum 1 + exp(-g) as a factor; the reciprocal by one Newton step on the
// hardware's estimate.  Some 25 instructions where the library's exponential and division took about 70.
// The binary64 value is off by up to 2e-12 relative (a polynomial of nine terms, an estimate's error squared), so that its
// rounding agrees everywhere is a matter of no half value ending that close to a tie, and near g = 0, where some do, of what
// v_rcp_f64 returns for arguments near 2: sqap_selftest_silu compares all of them on the device.
// The power's exponent stops at 2^1000, so a large negative g ends at -0; g = -inf makes f infinite and the result NaN,
// as -inf / inf is; g = +inf is held at 700 in the exponent only.
__device__ __forceinline__ float silu_of(float g)
{
    const float x = fmaxf(-g, -700.f);
    const float k = rintf(x * 1.442695040888963f);
    const double f = fma((double)x, 1.4426950408889634, -(double)k);
    double q = 0x1.63b2d79741c48p-20;
    q = fma(q, f, 0x1.00c0e4e154772p-16);
    q = fma(q, f, 0x1.4308c7183d394p-13);
    q = fma(q, f, 0x1.5d8775983509fp-10);
    q = fma(q, f, 0x1.3b2ab70ad2568p-7);
    q = fma(q, f, 0x1.c6b08da70cce3p-5);
    q = fma(q, f, 0x1.ebfbdff82a734p-3);
    q = fma(q, f, 0x1.62e42fef9cc69p-1);
    const int e = min((int)k, 1000);
    const double d = fma(fma(q, f, 1.0), __hiloint2double((e + 1023) << 20, 0), 1.0);
    double r = __builtin_amdgcn_rcp(d);
    r = fma(r, fma(-d, r, 1.0), r);
    return (float)((double)g * r);
}

// g := the half that silu_of(g) * u rounds to, for eight pairs.  Binary32 and the hardware's exponential and reciprocal give silu with an
// error of at most kSiluError where |g| <= kSiluMax, so that where both ends of r (1 +- kSiluReach) round to one half, that half is it:
// rounding is monotonic, and the reach covers the error, the product's rounding on both ways and the ends' own, 2^-24 each.  The exponent
// stops at kSiluMax: above it silu is g itself, and so is the estimate; below, the estimate is a negative number (zero for none) so small
// that its product with any finite u rounds to the zero that silu's does.  Two halves that differ in more than the sign (a low end
// of -0 comes out as +0) are open (0.2 % of the values, one wavefront in eight; an infinite r, whose low end is NaN), and silu_of decides; NaN is
// NaN by the definition too.  The estimates of all eight come first, so that none waits for another.
// None of this is taken from a manual: sqap_selftest_silu looks at all halves.
constexpr float kSiluMax = 80.f, kSiluError = 5.0e-7f, kSiluReach = 7.0e-7f;
static_assert(kSiluError + 3.0f / 16777216.0f < kSiluReach, "");

__device__ __forceinline__ float silu_estimate(float g)
{
    const float x = __builtin_amdgcn_fmed3f(g, -kSiluMax, kSiluMax), t = x * -1.442695040888963f, power = __builtin_amdgcn_exp2f(t);
    // what the rounding of t has taken from the exponent, with ln 2 in two parts
    const float lost = fmaf(t, 0x1.05c610p-29f, fmaf(t, -0x1.62e430p-1f, -x));
    return g * __builtin_amdgcn_rcpf(1.0f + fmaf(power, lost, power));
}

__device__ __forceinline__ void swiglu8(float (&g)[8], const float (&u)[8])
{
    typedef float v2f __attribute__((ext_vector_type(2)));
    typedef _Float16 v2h __attribute__((ext_vector_type(2)));
    union Pair { v2h h; uint32_t bits; } low[4], high[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const float a = silu_estimate(g[2 * p]) * u[2 * p], b = silu_estimate(g[2 * p + 1]) * u[2 * p + 1];
        low[p].h = __builtin_convertvector((v2f{fmaf(a, -kSiluReach, a), fmaf(b, -kSiluReach, b)}), v2h);
        high[p].h = __builtin_convertvector((v2f{fmaf(a, kSiluReach, a), fmaf(b, kSiluReach, b)}), v2h);
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        float a = (float)high[p].h[0], b = (float)high[p].h[1];
        const uint32_t open = low[p].bits ^ high[p].bits;
        if (open & 0x7fffu) {                              // (not the sign: that of a zero's low end is lost)
            float exact = silu_of(g[2 * p]) * u[2 * p];
            asm volatile("" : "+v"(exact));                // two roundings, not one mixed-precision instruction
            a = __half2float(__float2half_rn(exact));
        }
        if (open & 0x7fff0000u) {
            float exact = silu_of(g[2 * p + 1]) * u[2 * p + 1];
            asm volatile("" : "+v"(exact));
            b = __half2float(__float2half_rn(exact));
        }
        g[2 * p] = a;
        g[2 * p + 1] = b;
    }
}

}  // namespace sqap
