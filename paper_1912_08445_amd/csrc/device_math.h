// FP64 device arithmetic shared by the kernels (exponentials and a reciprocal without
// the library's special-case handling, for arguments these kernels produce).
#pragma once
#include <hip/hip_runtime.h>

namespace nlte {

// e^y for y <= 700 in FP64: y = n ln2 + r with |r| <= ln2/2 (two-part ln2), e^r by its
// degree-11 Taylor polynomial (truncation < 7e-15 relative), scaled by 2^n.  Results
// below the FP64 range come out as 0 through ldexp; no other special cases arise for
// the arguments used here (finite, at most 700).
__device__ __forceinline__ double exp_le700(double y)
{
    const double n = rint(y * 1.44269504088896338700);
    double r = fma(-n, 6.93147180369123816490e-01, y);
    r = fma(-n, 1.90821492927058770002e-10, r);
    double p = 2.50521083854417187751e-08;           // 1/11!
    p = fma(p, r, 2.75573192239858906526e-07);       // 1/10!
    p = fma(p, r, 2.75573192239858906526e-06);       // 1/9!
    p = fma(p, r, 2.48015873015873015873e-05);       // 1/8!
    p = fma(p, r, 1.98412698412698412698e-04);       // 1/7!
    p = fma(p, r, 1.38888888888888888889e-03);       // 1/6!
    p = fma(p, r, 8.33333333333333333333e-03);       // 1/5!
    p = fma(p, r, 4.16666666666666666667e-02);       // 1/4!
    p = fma(p, r, 1.66666666666666666667e-01);       // 1/3!
    p = fma(p, r, 0.5);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    const int ni = (int)fmax(n, -2200.0);
    return ldexp(p, ni);
}

// 2^{j/64}, j = 0..63, correctly rounded: the table of exp_tab64 (copied into LDS by the
// kernels that use it).
constexpr double kExp2SixtyFourths[64] = {
    0x1.0000000000000p+0, 0x1.02c9a3e778061p+0, 0x1.059b0d3158574p+0, 0x1.0874518759bc8p+0,
    0x1.0b5586cf9890fp+0, 0x1.0e3ec32d3d1a2p+0, 0x1.11301d0125b51p+0, 0x1.1429aaea92de0p+0,
    0x1.172b83c7d517bp+0, 0x1.1a35beb6fcb75p+0, 0x1.1d4873168b9aap+0, 0x1.2063b88628cd6p+0,
    0x1.2387a6e756238p+0, 0x1.26b4565e27cddp+0, 0x1.29e9df51fdee1p+0, 0x1.2d285a6e4030bp+0,
    0x1.306fe0a31b715p+0, 0x1.33c08b26416ffp+0, 0x1.371a7373aa9cbp+0, 0x1.3a7db34e59ff7p+0,
    0x1.3dea64c123422p+0, 0x1.4160a21f72e2ap+0, 0x1.44e086061892dp+0, 0x1.486a2b5c13cd0p+0,
    0x1.4bfdad5362a27p+0, 0x1.4f9b2769d2ca7p+0, 0x1.5342b569d4f82p+0, 0x1.56f4736b527dap+0,
    0x1.5ab07dd485429p+0, 0x1.5e76f15ad2148p+0, 0x1.6247eb03a5585p+0, 0x1.6623882552225p+0,
    0x1.6a09e667f3bcdp+0, 0x1.6dfb23c651a2fp+0, 0x1.71f75e8ec5f74p+0, 0x1.75feb564267c9p+0,
    0x1.7a11473eb0187p+0, 0x1.7e2f336cf4e62p+0, 0x1.82589994cce13p+0, 0x1.868d99b4492edp+0,
    0x1.8ace5422aa0dbp+0, 0x1.8f1ae99157736p+0, 0x1.93737b0cdc5e5p+0, 0x1.97d829fde4e50p+0,
    0x1.9c49182a3f090p+0, 0x1.a0c667b5de565p+0, 0x1.a5503b23e255dp+0, 0x1.a9e6b5579fdbfp+0,
    0x1.ae89f995ad3adp+0, 0x1.b33a2b84f15fbp+0, 0x1.b7f76f2fb5e47p+0, 0x1.bcc1e904bc1d2p+0,
    0x1.c199bdd85529cp+0, 0x1.c67f12e57d14bp+0, 0x1.cb720dcef9069p+0, 0x1.d072d4a07897cp+0,
    0x1.d5818dcfba487p+0, 0x1.da9e603db3285p+0, 0x1.dfc97337b9b5fp+0, 0x1.e502ee78b3ff6p+0,
    0x1.ea4afa2a490dap+0, 0x1.efa1bee615a27p+0, 0x1.f50765b6e4540p+0, 0x1.fa7c1819e90d8p+0,};

// e^y for y <= 700 in FP64, table-driven: y = (64 e + j) ln2/64 + r with |r| <= ln2/128
// (two-part ln2/64), e^y = 2^e 2^{j/64} e^r, e^r by its degree-5 Taylor polynomial (truncation
// < 4e-17 relative), tab = kExp2SixtyFourths.  The index comes from the low word of
// y 64/ln2 + 1.5 2^52 (rounded to the nearest integer by the addition).  Below -745.2 the result
// is 0 (y is first raised to -760, whose value is 0 after the scaling).  Within 2 ulp.  15
// instructions; 16 entries and degree 7 took 18 and two constants more, which matters in
// register-bound kernels.
__device__ __forceinline__ double exp_tab64(double y, const double *tab)
{
    constexpr double kRound = 0x1.8p52;
    y = fmax(y, -760.0);
    const double t = fma(y, 0x1.71547652b82fep+6, kRound);   // 64 / ln2
    const double n = t - kRound;
    double r = fma(-n, 0x1.62e42fe000000p-7, y);             // ln2/64, leading 29 bits
    r = fma(-n, 0x1.f473de6af278fp-36, r);                   // the rest of ln2/64
    double p = 0x1.1111111111111p-7;                         // 1/5!
    p = fma(p, r, 0x1.5555555555555p-5);                     // 1/4!
    p = fma(p, r, 0x1.5555555555555p-3);                     // 1/3!
    p = fma(p, r, 0.5);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    const int ni = __double2loint(t);
    return ldexp(tab[ni & 63] * p, ni >> 6);
}

// e^{-u} for 0 <= u <= 0.5 by its degree-13 Taylor polynomial (truncation < 1e-15).
__device__ __forceinline__ double exp_neg_small(double u)
{
    double p = -1.60590438368216145994e-10;          // -1/13!
    p = fma(p, u, 2.08767569878680989792e-09);       // 1/12!
    p = fma(p, u, -2.50521083854417187751e-08);
    p = fma(p, u, 2.75573192239858906526e-07);
    p = fma(p, u, -2.75573192239858906526e-06);
    p = fma(p, u, 2.48015873015873015873e-05);
    p = fma(p, u, -1.98412698412698412698e-04);
    p = fma(p, u, 1.38888888888888888889e-03);
    p = fma(p, u, -8.33333333333333333333e-03);
    p = fma(p, u, 4.16666666666666666667e-02);
    p = fma(p, u, -1.66666666666666666667e-01);
    p = fma(p, u, 0.5);
    p = fma(p, u, -1.0);
    return fma(p, u, 1.0);
}

// 1/x for a normal positive x: the hardware estimate refined by two Newton steps
// (relative error near 1 ulp; not correctly rounded).
__device__ __forceinline__ double rcp_refined(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}

}  // namespace nlte
