// Counter-based random numbers for the particle filter: Philox4x32-10
// (Salmon, Moraes, Dror, Shaw, SC'11) and the Box-Muller transform.
//
// The paper draws its normals in double and converts them to the working
// precision (Sec. 4, after Eq. (2)); the same seed is used by every precision
// (Sec. 5).  Here every particle k at step t owns the counter
// (k, t, stream_id, 0) and the step's resampling offset owns
// (0, t, stream_id, 1), so each draw is a pure function of its counter and
// no generator state is stored.  The double mode builds two 53-bit uniforms
// from the four words; the reduced modes take the top 24 bits of the same
// words, so every precision sees the same random stream.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "exp64.hpp"

namespace pf {

struct u32x4 {
    uint32_t v0, v1, v2, v3;
};

// Three-way exclusive or in one gfx950 instruction (v_bitop3_b32 with the
// truth table 0x96).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// Ten rounds; each multiplies two counter words by the Philox constants,
// swaps the halves and mixes in the round key, which advances by the Weyl
// increments (0x9E3779B9, 0xBB67AE85) between rounds.  The key words are
// uniform across the wave, so their updates stay scalar; per round and lane
// the work is two 32x32->64 multiplies and two three-way exclusive ors.
__device__ __forceinline__ u32x4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                               uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0);
        const uint32_t n1 = (uint32_t)p1;
        const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, k1);
        const uint32_t n3 = (uint32_t)p0;
        c0 = n0; c1 = n1; c2 = n2; c3 = n3;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return u32x4{c0, c1, c2, c3};
}

// 53-bit uniform in [0, 1) from (hi, lo): hi's 32 bits then lo's top 21.
__device__ __forceinline__ double uniform53(uint32_t hi, uint32_t lo)
{
    const uint64_t bits = ((uint64_t)hi << 21) | (uint64_t)(lo >> 11);
    return (double)bits * 0x1.0p-53;
}

// The same value times 2^32, exact (53 bits): two conversions of 32 bits and
// one fused multiply-add.
__device__ __forceinline__ double uniform53_times_2_32(uint32_t hi, uint32_t lo)
{
    return __builtin_fma((double)(lo >> 11), 0x1.0p-21, (double)hi);
}

// The three functions of the double Box-Muller, for its own arguments only.
// The library's log, sqrt and sincos take any argument; as inlined they were
// 98, 22 and 157 vector instructions a particle and most of the double pass A,
// which is bound by vector issue (87 % busy at 2^23 particles).  These are about
// 30, 11 and 36, and pass A needs 62 registers instead of 92 (8 waves per
// SIMD, not 5): a step of 2^23 + 1 particles (r = 8) 182 -> 161 us, of 2^20
// 31.8 -> 29.6 us.  Largest error of a normal over 2^21 draws 1.5e-15 (the
// library's 4.2e-15: it rounds 2 pi u before it reduces it).
// Polynomial coefficients: the functions' own Taylor series economised at
// Chebyshev nodes in 60 digits; what they leave out is below 2e-17 of the
// result.

// -2 ln(a) for a in [2^-53, 1].  a = 2^e m with m in [sqrt(1/2), sqrt(2)), f =
// m - 1, s = f / (2 + f): ln m = 2 atanh(s) = f - h + s (h + R) with h = f^2 / 2
// and R the series past 2 s, over s.  (The split at sqrt(1/2), this arrangement of
// the sum and ln 2 in two parts are those of the published fdlibm logarithm, Sun
// Microsystems 1993; the series' coefficients are our own.)
__device__ __forceinline__ double minus_2_ln(double a)
{
    const uint32_t hx = (uint32_t)__double2hiint(a);
    const int e = (int)(hx - 0x3fe6a09fu) >> 20;  // <= 0: floor
    const double m = __hiloint2double((int)(hx - ((uint32_t)e << 20)), __double2loint(a));
    const double f = m - 1.0;
    const double d = f + 2.0;
    double y = __builtin_amdgcn_rcp(d);
    y = __builtin_fma(__builtin_fma(-d, y, 1.0), y, y);
    y = __builtin_fma(__builtin_fma(-d, y, 1.0), y, y);
    double s = f * y;
    s = __builtin_fma(__builtin_fma(-d, s, f), y, s);
    const double z = s * s;
    double p = coef(0x1.2b584dae87b55p-3);
    p = __builtin_fma(p, z, coef(0x1.39fe60271f67fp-3));
    p = __builtin_fma(p, z, coef(0x1.7462b4ad0d879p-3));
    p = __builtin_fma(p, z, coef(0x1.c71c62e579789p-3));
    p = __builtin_fma(p, z, coef(0x1.2492492df14dfp-2));
    p = __builtin_fma(p, z, coef(0x1.99999999952e2p-2));
    p = __builtin_fma(p, z, coef(0x1.5555555555558p-1));
    const double h = 0.5 * f * f;
    const double ed = (double)e;
    // e ln 2 in two parts, the first exact (ln 2's leading 32 bits)
    const double t = __builtin_fma(s, __builtin_fma(z, p, h), ed * coef(0x1.a39ef35793c76p-33));
    const double l = __builtin_fma(ed, coef(0x1.62e42feep-1), -((h - t) - f));
    return -2.0 * l;
}

// sqrt(x) for x = 0 or x in [2^-53, 128]: reciprocal square root and three
// Goldschmidt corrections (no scaling: the argument is far from the range's
// ends; zero becomes 1e-150, so a particle that has drawn radius 0 moves by up
// to 1e-150 deviations instead of 0).
__device__ __forceinline__ double sqrt_near(double x)
{
    x = __builtin_fmax(x, 1e-300);
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, r, g);
    h = __builtin_fma(h, r, h);
    g = __builtin_fma(__builtin_fma(-g, g, x), h, g);
    g = __builtin_fma(__builtin_fma(-g, g, x), h, g);
    return g;
}

// cos and sin of 2 pi u 2^-32 for u in [0, 2^32): the quadrant and the rest of
// u are exact, so the angle is reduced before it is rounded.  (The cosine's last
// sum, with what 1 - z / 2 leaves out, is arranged as in fdlibm's cosine.)
__device__ __forceinline__ void cos_sin_turn(double u, double& c, double& s)
{
    const double k = __builtin_rint(u * 0x1.0p-30);  // quarter turns
    const double t = __builtin_fma(k, -0x1.0p30, u) * coef(0x1.921fb54442d18p+2 * 0x1.0p-32);
    const int q = (int)k;
    const double z = t * t;
    double p = coef(0x1.5e0b19f699a14p-33);
    p = __builtin_fma(p, z, coef(-0x1.ae600b02b0573p-26));
    p = __builtin_fma(p, z, coef(0x1.71de37968a0a7p-19));
    p = __builtin_fma(p, z, coef(-0x1.a01a019e83aaep-13));
    p = __builtin_fma(p, z, coef(0x1.1111111110bb2p-7));
    p = __builtin_fma(p, z, coef(-0x1.5555555555555p-3));
    const double sn = __builtin_fma(t * z, p, t);
    double w = coef(-0x1.907da3658b573p-37);
    w = __builtin_fma(w, z, coef(0x1.1eeb68e9387c9p-29));
    w = __builtin_fma(w, z, coef(-0x1.27e4fa17da071p-22));
    w = __builtin_fma(w, z, coef(0x1.a01a019f4eb01p-16));
    w = __builtin_fma(w, z, coef(-0x1.6c16c16c16967p-10));
    w = __builtin_fma(w, z, coef(0x1.5555555555555p-5));
    const double hz = 0.5 * z, one = 1.0 - hz;
    const double cs = one + __builtin_fma(z * z, w, (1.0 - one) - hz);
    const bool swap = (q & 1) != 0;
    const double a = swap ? sn : cs, b = swap ? cs : sn;
    // signs: cos is negative in quadrants 1 and 2, sin in 2 and 3
    const int sc = ((q + 1) & 2) << 30, ss = (q & 2) << 30;
    c = __hiloint2double(__double2hiint(a) ^ sc, __double2loint(a));
    s = __hiloint2double(__double2hiint(b) ^ ss, __double2loint(b));
}

// Box-Muller in double (Box & Muller 1958): rho = sqrt(-2 ln(1 - u_a)),
// (z_x, z_y) = rho (cos 2 pi u_b, sin 2 pi u_b).  Written operation by
// operation; the library is compiled without contraction so each product
// and sum rounds separately.
__device__ __forceinline__ void normal_pair_f64(const u32x4& w, double& zx, double& zy)
{
    // 1 - u_a is a multiple of 2^-53 in (0, 1]: exact
    const double rho = sqrt_near(minus_2_ln(__builtin_fma(uniform53_times_2_32(w.v0, w.v1), -0x1.0p-32, 1.0)));
    double s, c;
    cos_sin_turn(uniform53_times_2_32(w.v2, w.v3), c, s);
    zx = rho * c;
    zy = rho * s;
}

// Box-Muller in float from the top 24 bits of the same words.  Uses the
// hardware transcendental instructions: log2, square root, and sine/cosine
// whose argument is in revolutions (so sin(2 pi u) is sin_rev(u) with no
// multiply by 2 pi).  1 - u_a lies in [2^-24, 1], so the logarithm is finite.
__device__ __forceinline__ void normal_pair_f32(const u32x4& w, float& zx, float& zy)
{
    const float ua = (float)(w.v0 >> 8) * 0x1.0p-24f;
    const float ub = (float)(w.v2 >> 8) * 0x1.0p-24f;
    // -2 ln(1 - u) = -2 ln(2) log2(1 - u)
    const float l2 = __builtin_amdgcn_logf(1.0f - ua);
    const float rho = __builtin_amdgcn_sqrtf(-1.3862943611198906f * l2);
    zx = rho * __builtin_amdgcn_cosf(ub);
    zy = rho * __builtin_amdgcn_sinf(ub);
}

}  // namespace pf
