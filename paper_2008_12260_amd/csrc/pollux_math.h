// fp64 elementary functions for the last pass of Eq. 10 of the Pollux paper
// (arXiv 2008.12260, Sec. 3.2): T_iter(a, m, 0) = (T_grad^g + T_sync^g)^(1/g).
//
// gfx950 has no fp64 transcendental unit beyond v_rcp_f64, so exp and log are
// fused-multiply-add polynomial chains.  The kernel evaluates Eq. 10 with the
// larger term factored out,
//     big * exp( log1p( exp(-g * |ln T_grad - ln T_sync|) ) / g ),
// so the only arguments that occur are: exp of a non-positive number,
// log1p on [0, 1], and exp on [0, ln 2].  Each function below is accurate to
// about one unit in the last place on that domain.
//
// The file also compiles for the host (PX_MATH_HOST) so that the CPU test-suite
// can measure the error of exactly these polynomials against libm.
#pragma once

#if defined(PX_MATH_HOST)
#include <cmath>
#define PX_DEV inline
namespace px {
inline double px_fma(double a, double b, double c) { return std::fma(a, b, c); }
inline double seed_skew = 0.0;      // set by a test: the hardware's seed is off by up to 2^-24, and not as this one is
inline double px_rcp_seed(double x) { return (double)(1.0f / (float)x) * (1.0 + seed_skew); }   // off by up to 2^-24 itself
inline double px_ldexp(double x, int k) { return std::ldexp(x, k); }
inline double px_rint(double x) { return std::nearbyint(x); }
inline double px_max(double a, double b) { return std::fmax(a, b); }
inline float px_fma(float a, float b, float c) { return std::fma(a, b, c); }
inline float root_skew = 0.0f;      // set by a test: the hardware's root is off by up to one unit in the last place
inline float px_sqrt(float x) { return std::sqrt(x) * (1.0f + root_skew); }
inline float px_median0(float x, float y) { return x != x ? std::fmin(0.0f, y) : std::fmax(std::fmin(x, y), std::fmin(std::fmax(x, y), 0.0f)); }
}  // namespace px
#else
#include <hip/hip_runtime.h>
#define PX_DEV __device__ __forceinline__
namespace px {
PX_DEV double px_fma(double a, double b, double c) { return __builtin_fma(a, b, c); }
PX_DEV double px_rcp_seed(double x) { return __builtin_amdgcn_rcp(x); }             // v_rcp_f64
PX_DEV double px_ldexp(double x, int k) { return __builtin_amdgcn_ldexp(x, k); }    // v_ldexp_f64
PX_DEV double px_rint(double x) { return __builtin_rint(x); }                       // v_rndne_f64
PX_DEV double px_max(double a, double b) { return __builtin_fmax(a, b); }            // v_max_f64: b where a is not a number
PX_DEV float px_fma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
PX_DEV float px_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }                 // v_sqrt_f32
PX_DEV float px_median0(float x, float y) { return __builtin_amdgcn_fmed3f(x, 0.0f, y); }   // v_med3_f32: min(0, y) where x is not a number
}  // namespace px
#endif

namespace px {

// The functions' constants.  A kernel that evaluates them over and over holds them in registers (held_coefs): one wavefront
// issues an instruction every four cycles, scalar ones no faster, so that a coefficient formed where it is used, by two moves,
// trebles the price of a polynomial's step.  Functions without the argument form them where they are used.
struct Coefs {
    double log_top, log_c[10];      // 2/23, and 2/21, 2/19 .. 2/3
    double exp_top, exp_c[10];      // 1/13!, and 1/12!, 1/11! .. 1/3!
    double ln2, ln2_low, log2e, exp_least, root_half, root2_less1;
};

PX_DEV Coefs plain_coefs()
{
    return Coefs{0.08695652173913043,
                 {0.09523809523809523, 0.10526315789473684, 0.11764705882352941, 0.13333333333333333, 0.15384615384615385,
                  0.18181818181818182, 0.2222222222222222, 0.2857142857142857, 0.4, 0.6666666666666666},
                 1.6059043836821613e-10,
                 {2.08767569878681e-09, 2.505210838544172e-08, 2.755731922398589e-07, 2.7557319223985893e-06, 2.48015873015873e-05,
                  0.0001984126984126984, 0.001388888888888889, 0.008333333333333333, 0.041666666666666664, 0.16666666666666666},
                 0.6931471805599453,        // ln2 high part
                 2.3190468138462996e-17,    // ln2 low part
                 1.4426950408889634,        // log2(e)
                 -745.5,                    // exp underflows to 0 below this
                 0.7071067811865476, 0.41421356237309503};
}

#if !defined(PX_MATH_HOST)
// The same in registers: the highest coefficients in vector ones (an instruction takes one scalar operand), all others in scalar ones.
PX_DEV Coefs held_coefs()
{
    Coefs c = plain_coefs();
    asm volatile("" : "+v"(c.log_top), "+v"(c.exp_top));
#pragma unroll
    for (int i = 0; i < 10; ++i) asm volatile("" : "+s"(c.log_c[i]), "+s"(c.exp_c[i]));
    asm volatile("" : "+s"(c.ln2), "+s"(c.ln2_low), "+s"(c.log2e), "+s"(c.exp_least), "+s"(c.root_half), "+s"(c.root2_less1));
    return c;
}
#endif

// a / b for finite b != 0 well inside the exponent range: reciprocal seed (2^-24), one step of third order, one residual
// correction of the quotient.  (In 1.5e8 tries with seeds off by up to 2^-23 either way, a tenth on random mantissas and the others on
// those next to 1 and 2, the quotient was the correctly rounded one but for 1 / b where b's mantissa is all ones.)
PX_DEV double px_div(double a, double b)
{
    double r = px_rcp_seed(b);
    const double e = px_fma(-b, r, 1.0);
    r = px_fma(px_fma(e, e, e), r, r);
    const double q = a * r;
    return px_fma(px_fma(-b, q, a), r, q);
}

// exp(t) for t <= 1 (any negative t, -inf included): t = k ln2 + r, |r| <= ln2/2,
// Taylor polynomial of degree 13 in r (remainder below 2^-57), scaled by 2^k.
PX_DEV double px_exp(const Coefs &c, double t)
{
    t = px_max(t, c.exp_least);
    const double k = px_rint(t * c.log2e);
    double r = px_fma(-k, c.ln2, t);
    r = px_fma(-k, c.ln2_low, r);
    double p = c.exp_top;
#pragma unroll
    for (int i = 0; i < 10; ++i) p = px_fma(p, r, c.exp_c[i]);
    p = px_fma(p, r, 0.5);
    p = px_fma(p, r, 1.0);
    p = px_fma(p, r, 1.0);
    return px_ldexp(p, (int)k);
}

// 2 atanh(z) = log((1+z)/(1-z)) for |z| <= 0.1716 (z^2 <= 0.0295): odd series up to z^23.
PX_DEV double px_two_atanh(const Coefs &c, double z)
{
    const double w = z * z;
    double p = c.log_top;
#pragma unroll
    for (int i = 0; i < 10; ++i) p = px_fma(p, w, c.log_c[i]);
    return px_fma(z * w, p, z + z);
}

// log(1 + e) for 0 <= e <= 1.  For e > sqrt(2) - 1 the argument is halved first:
// log(1+e) = ln2 + log(1 + f), f = (e - 1)/2; in both cases log(1+f) = 2 atanh(f/(2+f)).
PX_DEV double px_log1p_unit(const Coefs &c, double e)
{
    const bool big = e > c.root2_less1;
    const double f = big ? (e - 1.0) * 0.5 : e;
    const double l = px_two_atanh(c, px_div(f, 2.0 + f));
    return big ? l + c.ln2 : l;
}

// log(x) for positive, finite, normal x.  x = 2^k * m with m in [sqrt(1/2), sqrt(2)).
PX_DEV double px_log(const Coefs &c, double x)
{
#if defined(PX_MATH_HOST)
    int k;
    double m = std::frexp(x, &k);
#else
    int k = __builtin_amdgcn_frexp_exp(x);
    double m = __builtin_amdgcn_frexp_mant(x);
#endif
    if (m < c.root_half) { m += m; k -= 1; }
    const double f = m - 1.0;
    const double l = px_two_atanh(c, px_div(f, 2.0 + f));
    const double kd = (double)k;
    return px_fma(kd, c.ln2, px_fma(kd, c.ln2_low, l));
}

// The count s_lo <= s <= s_hi with the smallest w(s) = s + C / (s + 1): the largest t with C > t (t + 1), clamped (REAL = float: exact for
// counts up to 4094).  t is found in fp32, where sqrt(C + 1/4) - 1/2 is off by less than 0.008 for every count a grid can have
// (below 2^14); taken 0.01 lower it is t or t - 1, and the exact order of neighbours says which.  C = 0, a negative one and what is
// no number: t = 0.  Any C beyond the grid, infinity too: s_hi (the root is clamped before it becomes a whole number).
template <typename REAL>
PX_DEV int px_best_count(REAL C, int s_lo, int s_hi)
{
    int t = (int)px_median0(px_sqrt((float)C + 0.25f) - 0.51f, (float)s_hi);
    const REAL td = (REAL)t;
    t += C > px_fma(td, td, px_fma((REAL)3, td, (REAL)2)) ? 1 : 0;
    t = t < s_hi ? t : s_hi;
    return t > s_lo ? t : s_lo;
}

PX_DEV double px_exp(double t) { return px_exp(plain_coefs(), t); }
PX_DEV double px_log1p_unit(double e) { return px_log1p_unit(plain_coefs(), e); }
PX_DEV double px_log(double x) { return px_log(plain_coefs(), x); }

}  // namespace px
