// The double mode's weights: exp of an argument that is not positive.
#pragma once

namespace pf {

// A constant in scalar registers, formed where it is used: left to itself the
// compiler keeps a loop's double constants in vector registers (40 of them).
__device__ __forceinline__ double coef(double c)
{
#ifdef __AMDGCN__
    __asm__ volatile("" : "+s"(c));
#endif
    return c;
}

// exp(d) for d <= 0: d = k ln 2 + r, |r| <= ln 2 / 2, exp(r) = 1 + r + r^2 P(r), where c is
// what r's rounding left out and the sum keeps what 1 + r left out.  26
// instructions against the library's 42.  Over 2^22 arguments each in ranges
// from [-0.35, 0] to [-745, 0] the largest error is 0.841 ulp, the mean 0.2528 (the
// device library's 0.861 and 0.2577; without the two corrections 1.158 and
// 0.2690).  The polynomial's coefficients: the Taylor series economised at
// Chebyshev nodes in 60 digits.
__device__ __forceinline__ double exp_nonpos(double d)
{
    d = d < -800.0 ? -800.0 : d;  // rounds to 0 from there on; a NaN stays
    const double k = __builtin_rint(d * coef(0x1.71547652b82fep+0));
    const double h = __builtin_fma(k, -coef(0x1.62e42feep-1), d);  // exact
    const double r = __builtin_fma(k, -coef(0x1.a39ef35793c76p-33), h);
    const double c = __builtin_fma(k, -coef(0x1.a39ef35793c76p-33), h - r);
    double p = coef(0x1.af38a0d2d9620p-26);
    p = __builtin_fma(p, r, coef(0x1.28917e2c43a66p-22));
    p = __builtin_fma(p, r, coef(0x1.71de0db21e27fp-19));
    p = __builtin_fma(p, r, coef(0x1.a019b9133a48ap-16));
    p = __builtin_fma(p, r, coef(0x1.a01a01a7c327ap-13));
    p = __builtin_fma(p, r, coef(0x1.6c16c1788a49bp-10));
    p = __builtin_fma(p, r, coef(0x1.11111111109b4p-7));
    p = __builtin_fma(p, r, coef(0x1.5555555553d67p-5));
    p = __builtin_fma(p, r, coef(0x1.5555555555556p-3));
    p = __builtin_fma(p, r, 0.5);
    const double one = 1.0 + r;
    return __builtin_ldexp(one + (((1.0 - one) + r) + __builtin_fma(r * r, p, c)), (int)k);
}

}  // namespace pf
