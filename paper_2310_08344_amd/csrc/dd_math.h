// Double-double arithmetic and the phi functions in double-double, shared
// by the host planner (plain C++) and the device planner (HIP).
//
// A value is hi + lo with |lo| <= ulp(hi)/2.  The error-free
// transformations are Knuth's TwoSum and Dekker's TwoProduct (with an FMA);
// addition, multiplication and division follow Hida, Li and Bailey,
// "Algorithms for quad-double precision floating point arithmetic" (2001).
// About 32 significant digits.
#pragma once

#include <math.h>

#if defined(__HIPCC__)
#define LX_HD __host__ __device__ inline
#else
#define LX_HD inline
#endif

// The error-free transformations need every product and sum rounded on its
// own: a multiply fused into a later add (which HIP device code allows by
// default, also across inlined calls) breaks them and leaves plain double
// precision.  Every function below switches contraction off for its body.
#if defined(__clang__)
#define LX_NO_CONTRACT _Pragma("clang fp contract(off)")
#else
#define LX_NO_CONTRACT
#endif

namespace lx {

struct dd {
    double hi, lo;
};

LX_HD dd two_sum(double a, double b) {
    LX_NO_CONTRACT
    const double s = a + b;
    const double bb = s - a;
    return {s, (a - (s - bb)) + (b - bb)};
}

LX_HD dd quick_two_sum(double a, double b) {
    LX_NO_CONTRACT
    const double s = a + b;
    return {s, b - (s - a)};
}

LX_HD dd two_prod(double a, double b) {
    LX_NO_CONTRACT
    const double p = a * b;
    return {p, fma(a, b, -p)};
}

LX_HD dd dd_add(dd x, dd y) {
    LX_NO_CONTRACT
    dd s = two_sum(x.hi, y.hi);
    const dd t = two_sum(x.lo, y.lo);
    s.lo += t.hi;
    s = quick_two_sum(s.hi, s.lo);
    s.lo += t.lo;
    return quick_two_sum(s.hi, s.lo);
}

LX_HD dd dd_neg(dd x) {
    LX_NO_CONTRACT
    return {-x.hi, -x.lo};
}
LX_HD dd dd_sub(dd x, dd y) {
    LX_NO_CONTRACT
    return dd_add(x, dd_neg(y));
}

LX_HD dd dd_mul(dd x, dd y) {
    LX_NO_CONTRACT
    dd p = two_prod(x.hi, y.hi);
    p.lo += x.hi * y.lo + x.lo * y.hi;
    return quick_two_sum(p.hi, p.lo);
}

LX_HD dd dd_mul_d(dd x, double b) {
    LX_NO_CONTRACT
    dd p = two_prod(x.hi, b);
    p.lo += x.lo * b;
    return quick_two_sum(p.hi, p.lo);
}

LX_HD dd dd_div(dd x, dd y) {
    LX_NO_CONTRACT
    const double q1 = x.hi / y.hi;
    dd r = dd_sub(x, dd_mul_d(y, q1));
    const double q2 = r.hi / y.hi;
    r = dd_sub(r, dd_mul_d(y, q2));
    const double q3 = r.hi / y.hi;
    const dd q = quick_two_sum(q1, q2);
    return dd_add(q, dd{q3, 0.0});
}

LX_HD dd dd_div_d(dd x, double b) {
    LX_NO_CONTRACT
    return dd_div(x, dd{b, 0.0});
}
LX_HD dd dd_ldexp(dd x, int e) {
    LX_NO_CONTRACT
    return {ldexp(x.hi, e), ldexp(x.lo, e)};
}

// e^r - 1 for a = k ln2 + r, |r| <= ln2/2: r is scaled by 2^-10, the Taylor
// series to order 12 is summed, then ten doublings
// e^{2x} - 1 = 2(e^x - 1) + (e^x - 1)^2 undo the scaling.  Returns k too.
LX_HD dd expm1_reduced(dd a, int* k_out) {
    LX_NO_CONTRACT
    const double ln2_hi = 6.931471805599452862e-01;   // ln 2 = hi + lo
    const double ln2_lo = 2.319046813846299558e-17;
    const double k = rint(a.hi / ln2_hi);
    dd r = dd_sub(a, dd_add(two_prod(k, ln2_hi), two_prod(k, ln2_lo)));
    r = dd_ldexp(r, -10);
    dd term = r, s = r;
    for (int n = 2; n <= 12; ++n) {
        term = dd_div_d(dd_mul(term, r), static_cast<double>(n));
        s = dd_add(s, term);
    }
    for (int i = 0; i < 10; ++i) s = dd_add(dd_mul_d(s, 2.0), dd_mul(s, s));
    *k_out = static_cast<int>(k);
    return s;
}

LX_HD dd dd_exp(dd a) {
    LX_NO_CONTRACT
    if (a.hi < -1000.0) return {0.0, 0.0};
    int k = 0;
    const dd s = expm1_reduced(a, &k);
    return dd_ldexp(dd_add(s, dd{1.0, 0.0}), k);
}

LX_HD dd dd_expm1(dd a) {
    LX_NO_CONTRACT
    if (a.hi < -1000.0) return {-1.0, 0.0};
    int k = 0;
    const dd s = expm1_reduced(a, &k);
    if (k == 0) return s;
    return dd_sub(dd_ldexp(dd_add(s, dd{1.0, 0.0}), k), dd{1.0, 0.0});
}

// phi_l(z) in double-double (Sec. 1 of the paper): the Taylor series
// sum_k z^k/(k+l)! while its terms decrease monotonically (|z| < max(1.5, l),
// 60 terms), otherwise phi_1 = expm1(z)/z and the recursion
// phi_{k+1} = (phi_k - 1/k!)/z.
LX_HD dd dd_phi(int l, dd z) {
    LX_NO_CONTRACT
    dd inv_fact_l{1.0, 0.0};
    for (int k = 2; k <= l; ++k) inv_fact_l = dd_div_d(inv_fact_l, static_cast<double>(k));
    if (z.hi == 0.0) return inv_fact_l;
    const double lim = (static_cast<double>(l) > 1.5) ? static_cast<double>(l) : 1.5;
    if (fabs(z.hi) < lim) {
        // Horner from the tail; coefficient k is 1/(k+l)!
        dd coef_top = inv_fact_l;
        for (int k = 1; k <= 60; ++k) coef_top = dd_div_d(coef_top, static_cast<double>(k + l));
        dd acc{0.0, 0.0};
        dd c = coef_top;
        for (int k = 60; k >= 0; --k) {
            acc = dd_add(dd_mul(acc, z), c);
            if (k > 0) c = dd_mul_d(c, static_cast<double>(k + l));   // 1/(k-1+l)!
        }
        return acc;
    }
    if (l == 0) return dd_exp(z);
    dd val = dd_div(dd_expm1(z), z);          // phi_1
    dd inv_fact{1.0, 0.0};                    // 1/k! for k = 1
    for (int k = 1; k < l; ++k) {
        val = dd_div(dd_sub(val, inv_fact), z);
        inv_fact = dd_div_d(inv_fact, static_cast<double>(k + 1));
    }
    return val;
}

// f(xi) = sigma * phi_l(alpha*h*(c + gamma*xi)) in double-double, from FP64
// inputs taken exactly
LX_HD dd dd_phi_at(int l, double alpha, double sigma, double h, double c, double gamma, double xi) {
    LX_NO_CONTRACT
    const dd ah = two_prod(alpha, h);
    const dd t = dd_add(dd{c, 0.0}, two_prod(gamma, xi));
    return dd_mul(dd{sigma, 0.0}, dd_phi(l, dd_mul(ah, t)));
}

// ---------------------------------------------------------------------------
// The same values by a shorter chain of operations, for the device planner:
// 1/k! from a table instead of a division per term, and divisions by a
// quantity whose reciprocal is at hand (rcp, any double within a few ulp of
// 1/y.hi: the second and third digits of the quotient correct the first).
// ---------------------------------------------------------------------------

// 1/k! rounded to double-double, k = 0..68
LX_HD dd dd_inv_fact(int k) {
    static constexpr double t[69][2] = {
        {0x1.0000000000000p+0, 0x0.0p+0},
        {0x1.0000000000000p+0, 0x0.0p+0},
        {0x1.0000000000000p-1, 0x0.0p+0},
        {0x1.5555555555555p-3, 0x1.5555555555555p-57},
        {0x1.5555555555555p-5, 0x1.5555555555555p-59},
        {0x1.1111111111111p-7, 0x1.1111111111111p-63},
        {0x1.6c16c16c16c17p-10, -0x1.f49f49f49f49fp-65},
        {0x1.a01a01a01a01ap-13, 0x1.a01a01a01a01ap-73},
        {0x1.a01a01a01a01ap-16, 0x1.a01a01a01a01ap-76},
        {0x1.71de3a556c734p-19, -0x1.c154f8ddc6c00p-73},
        {0x1.27e4fb7789f5cp-22, 0x1.cbbc05b4fa99ap-76},
        {0x1.ae64567f544e4p-26, -0x1.c062e06d1f209p-80},
        {0x1.1eed8eff8d898p-29, -0x1.2aec959e14c06p-83},
        {0x1.6124613a86d09p-33, 0x1.f28e0cc748ebep-87},
        {0x1.93974a8c07c9dp-37, 0x1.05d6f8a2efd1fp-92},
        {0x1.ae7f3e733b81fp-41, 0x1.1d8656b0ee8cbp-97},
        {0x1.ae7f3e733b81fp-45, 0x1.1d8656b0ee8cbp-101},
        {0x1.952c77030ad4ap-49, 0x1.ac981465ddc6cp-103},
        {0x1.6827863b97d97p-53, 0x1.eec01221a8b0bp-107},
        {0x1.2f49b46814157p-57, 0x1.2650f61dbdcb4p-112},
        {0x1.e542ba4020225p-62, 0x1.ea72b4afe3c2fp-120},
        {0x1.71b8ef6dcf572p-66, -0x1.d043ae40c4647p-120},
        {0x1.0ce396db7f853p-70, -0x1.aebcdbd20331cp-124},
        {0x1.761b41316381ap-75, -0x1.3423c7d91404fp-130},
        {0x1.f2cf01972f578p-80, -0x1.9ada5fcc1ab14p-135},
        {0x1.3f3ccdd165fa9p-84, -0x1.58ddadf344487p-139},
        {0x1.88e85fc6a4e5ap-89, -0x1.71c37ebd16540p-143},
        {0x1.d1ab1c2dccea3p-94, 0x1.054d0c78aea14p-149},
        {0x1.0a18a2635085dp-98, 0x1.b9e2e28e1aa54p-153},
        {0x1.259f98b4358adp-103, 0x1.eaf8c39dd9bc5p-157},
        {0x1.3932c5047d60ep-108, 0x1.832b7b530a627p-162},
        {0x1.434d2e783f5bcp-113, 0x1.0b87b91be9affp-167},
        {0x1.434d2e783f5bcp-118, 0x1.0b87b91be9affp-172},
        {0x1.3981254dd0d52p-123, -0x1.2b1f4c8015a2fp-177},
        {0x1.2710231c0fd7ap-128, 0x1.3f8a2b4af9d6bp-184},
        {0x1.0dc59c716d91fp-133, 0x1.419e3fad3f031p-188},
        {0x1.df983290c2ca9p-139, 0x1.5835c6895393bp-194},
        {0x1.9ec8d1c94e85bp-144, -0x1.670e9d4784ec6p-201},
        {0x1.5d4acb9c0c3abp-149, -0x1.6ec2c8f5b13b2p-205},
        {0x1.1e99449a4bacep-154, -0x1.fefbb89514b3cp-210},
        {0x1.ca8ed42a12ae3p-160, 0x1.a07244abad2abp-224},
        {0x1.65e61c39d0241p-165, -0x1.c0ed181727269p-220},
        {0x1.10af527530de8p-170, 0x1.b626c912ee5c8p-225},
        {0x1.95db45257e512p-176, 0x1.6e5d72b6f79b9p-231},
        {0x1.272b1b03fec6ap-181, 0x1.3f67cc9f9fdb8p-235},
        {0x1.a3cb872220648p-187, -0x1.c7f4e85b8e6cdp-241},
        {0x1.240804f659510p-192, 0x1.8b291b93c9718p-246},
        {0x1.8da8e0a127ebap-198, -0x1.21d2eac9d275cp-252},
        {0x1.091b406b6ff26p-203, 0x1.e973637973b18p-257},
        {0x1.5a42f0dfeb086p-209, -0x1.35ae015f78f6ep-264},
        {0x1.bb36f6e12cd78p-215, 0x1.02f85029a29b0p-270},
        {0x1.161872bf7b823p-220, 0x1.bb96c8e2e8897p-275},
        {0x1.56457989358c9p-226, -0x1.e3792533eafc8p-282},
        {0x1.9d4f1058674dfp-232, 0x1.03c81b6914d59p-286},
        {0x1.e9d8f6ed83eaap-238, -0x1.be25ac1066519p-293},
        {0x1.1d008faac5c50p-243, 0x1.50348ded2636fp-298},
        {0x1.45b77f9e98e12p-249, 0x1.e4b05119ccb1bp-303},
        {0x1.6db793c887b97p-255, -0x1.966963ad60539p-314},
        {0x1.938cc661b03f6p-261, 0x1.c4da1977e56d6p-318},
        {0x1.b5bfc17fa97d3p-267, -0x1.ff5794693c028p-321},
        {0x1.d2eeac43e7fcfp-273, 0x1.de9183d404419p-327},
        {0x1.e9e56d649f768p-279, 0x1.6fcf3a92e716ap-333},
        {0x1.f9b3059128bc7p-285, -0x1.be21d40d8511fp-339},
        {0x1.00dcf6a320e1cp-290, -0x1.239f67a557e8ap-344},
        {0x1.00dcf6a320e1cp-296, -0x1.239f67a557e8ap-350},
        {0x1.f9d2a2bb5471bp-303, 0x1.13d6bbbb1973ep-362},
        {0x1.ea7ead50ce01ap-309, 0x1.8514c58f37d88p-364},
        {0x1.d48849da8f4a3p-315, -0x1.b8cc0ca0d9dd6p-369},
        {0x1.b8f8bdfae136cp-321, -0x1.5bda721fb8375p-376}};
    return {t[k][0], t[k][1]};
}

// x / y: the remainder of the first digit is exact in its high part (an FMA),
// so one more digit completes the quotient
LX_HD dd dd_div_rcp(dd x, dd y, double rcp) {
    LX_NO_CONTRACT
    const double q1 = x.hi * rcp;
    const double r = fma(-q1, y.hi, x.hi) + fma(-q1, y.lo, x.lo);
    const double q2 = r * rcp;
    const dd q = quick_two_sum(q1, q2);
    const double r2 = fma(-q2, y.hi, r);
    return quick_two_sum(q.hi, q.lo + r2 * rcp);
}

// expm1_reduced with the Taylor series to order 12 by Horner
LX_HD dd expm1_reduced_fast(dd a, int* k_out) {
    LX_NO_CONTRACT
    const double ln2_hi = 6.931471805599452862e-01;   // ln 2 = hi + lo
    const double ln2_lo = 2.319046813846299558e-17;
    const double k = rint(a.hi * 1.442695040888963387);
    dd r = dd_sub(a, dd_add(two_prod(k, ln2_hi), two_prod(k, ln2_lo)));
    r = dd_ldexp(r, -10);
    dd s = dd_inv_fact(12);
#pragma unroll
    for (int n = 11; n >= 1; --n) s = dd_add(dd_mul(s, r), dd_inv_fact(n));
    s = dd_mul(s, r);
    for (int i = 0; i < 10; ++i) s = dd_add(dd_mul_d(s, 2.0), dd_mul(s, s));
    *k_out = static_cast<int>(k);
    return s;
}

// phi_l(z): the Taylor series while its terms decrease (36 + 3 l terms, the
// last below 1e-35 of the first for |z| < max(1.5, l), l <= 8), otherwise
// e^z, or the recursion from phi_1 = expm1(z)/z
LX_HD dd dd_phi_fast(int l, dd z) {
    LX_NO_CONTRACT
    if (z.hi == 0.0) return dd_inv_fact(l);
    const double lim = (static_cast<double>(l) > 1.5) ? static_cast<double>(l) : 1.5;
    if (fabs(z.hi) < lim) {
        const int top = 36 + 3 * l;
        dd acc = dd_inv_fact(top + l);
#pragma unroll 4
        for (int k = top - 1; k >= 0; --k) acc = dd_add(dd_mul(acc, z), dd_inv_fact(k + l));
        return acc;
    }
    if (z.hi < -1000.0 && l == 0) return {0.0, 0.0};
    dd val{-1.0, 0.0};   // expm1(z)
    if (z.hi >= -1000.0) {
        int k = 0;
        const dd s = expm1_reduced_fast(z, &k);
        const dd e = dd_ldexp(dd_add(s, dd{1.0, 0.0}), k);
        if (l == 0) return e;
        val = k == 0 ? s : dd_sub(e, dd{1.0, 0.0});
    }
    const double rcp = 1.0 / z.hi;
    val = dd_div_rcp(val, z, rcp);   // phi_1
    for (int k = 1; k < l; ++k) val = dd_div_rcp(dd_sub(val, dd_inv_fact(k)), z, rcp);
    return val;
}

LX_HD dd dd_phi_at_fast(int l, double alpha, double sigma, double h, double c, double gamma, double xi) {
    LX_NO_CONTRACT
    const dd ah = two_prod(alpha, h);
    const dd t = dd_add(dd{c, 0.0}, two_prod(gamma, xi));
    return dd_mul(dd{sigma, 0.0}, dd_phi_fast(l, dd_mul(ah, t)));
}

}  // namespace lx
