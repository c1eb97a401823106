// Node arithmetic of the rest-population schemes D1Q3Q2 (Sec. 2) and D2Q5Q4Q4
// (Sec. 3): equilibria and the moment-space relaxation with one rate per
// non-conserved moment (eq. 2-relaxation).  The formulas are stated in mrt.hip.
#pragma once

#include "internal.h"

namespace lbm {

// a / b rounded correctly: lbm_rcp(b) is the correctly rounded reciprocal, the
// product is within an ulp of the quotient, and one correction with its exact
// residual rounds to the quotient (Markstein's division).  3 operations more than
// the reciprocal, against 10 and a scaling test for the full division sequence,
// and one reciprocal serves every quotient by b.  The residual is exact for |a| >=
// 2^-1010; a smaller one counts for nothing in a state whose heights and g lie within
// kRestRange (its quotient is below 2^-510 there, squared or times a momentum zero).
// Beyond that range, the contexts run the WIDE collisions, with plain divisions.
__device__ __forceinline__ double div_by(double a, double b, double rb)
{
    const double q = a * rb;
    const double e = __builtin_fma(-b, q, a);
    return __builtin_fma(e, rb, q);
}

__device__ __forceinline__ void feq_rest1d(double h, double q, const Mrt &M, double *e)
{
    const double ih = 1.0 / h;
    const double u = q * ih;
    const double theta = M.g * h - 0.5 * (u * u);
    const double f0 = M.aK * theta;
    const double hr = h - f0;
    const double p = M.hg * (h * h);
    const double Fq = (q * q) * ih + p;
    e[0] = f0;
    e[1] = 0.5 * hr + q * M.c;
    e[2] = 0.5 * hr - q * M.c;
    e[3] = 0.5 * q + Fq * M.c;
    e[4] = 0.5 * q - Fq * M.c;
}

__device__ __forceinline__ void feq_rest2d(double h, double qx, double qy, const Mrt &M, double *e)
{
    const double ih = 1.0 / h;
    const double u = qx * ih, v = qy * ih;
    const double theta = M.g * h - 0.5 * (u * u + v * v);
    const double f0 = M.aK * theta;
    const double hr = h - f0;
    const double p = M.hg * (h * h);
    const double Fxx = (qx * qx) * ih + p, Fxy = (qx * qy) * ih, Fyy = (qy * qy) * ih + p;
    const double hq = 0.25 * hr, xq = 0.25 * qx, yq = 0.25 * qy;
    e[0] = f0;
    e[1] = hq + qx * M.c; e[2] = hq + qy * M.c; e[3] = hq - qx * M.c; e[4] = hq - qy * M.c;
    e[5] = xq + Fxx * M.c; e[6] = xq + Fxy * M.c; e[7] = xq - Fxx * M.c; e[8] = xq - Fxy * M.c;
    e[9] = yq + Fxy * M.c; e[10] = yq + Fyy * M.c; e[11] = yq - Fxy * M.c; e[12] = yq - Fyy * M.c;
}

template <bool WIDE = false>
__device__ __forceinline__ void collide_mrt1d(double *f, const Mrt &M)
{
    const double lam = M.lam, il = M.il;
    const double sp = f[1] + f[2];
    const double rho = f[0] + sp;
    double J = lam * (f[1] - f[2]);
    double eps = (lam * lam) * (sp - 2.0 * f[0]);
    const double q = f[3] + f[4];
    double Jq = lam * (f[3] - f[4]);
    const double u = WIDE ? q / rho : div_by(q, rho, lbm_rcp(rho));
    const double p = M.hg * (rho * rho);
    const double theta = M.g * rho - 0.5 * (u * u);
    J += M.rate[0] * (q - J);
    eps += M.rate[1] * ((lam * lam) * (rho - 3.0 * (M.aK * theta)) - eps);
    Jq += M.rate[2] * ((q * u + p) - Jq);
    const double r3 = rho - eps * (il * il);
    const double f0 = WIDE ? r3 / 3.0 : div_by(r3, 3.0, 1.0 / 3.0);
    const double S = rho - f0;
    f[0] = f0;
    f[1] = 0.5 * (S + J * il);
    f[2] = 0.5 * (S - J * il);
    f[3] = 0.5 * (q + Jq * il);
    f[4] = 0.5 * (q - Jq * il);
}

// Moments of one momentum family (g_1..g_4): total, x- and y-moments, XX.
__device__ __forceinline__ void fam_moments(const double *g, double lam, double &q, double &mx,
                                            double &my, double &xx)
{
    const double a = g[0] + g[2], b = g[1] + g[3];
    q = a + b;
    mx = lam * (g[0] - g[2]);
    my = lam * (g[1] - g[3]);
    xx = a - b;
}

__device__ __forceinline__ void fam_invert(double *g, double il, double q, double mx, double my,
                                           double xx)
{
    const double a = 0.5 * (q + xx), b = 0.5 * (q - xx);
    g[0] = 0.5 * (a + mx * il);
    g[2] = 0.5 * (a - mx * il);
    g[1] = 0.5 * (b + my * il);
    g[3] = 0.5 * (b - my * il);
}

template <bool WIDE = false>
__device__ __forceinline__ void collide_mrt2d(double *f, const Mrt &M)
{
    const double lam = M.lam, il = M.il;
    const double *r = M.rate;
    const double s13 = f[1] + f[3], s24 = f[2] + f[4];
    const double rho = f[0] + (s13 + s24);
    double Jx = lam * (f[1] - f[3]);
    double Jy = lam * (f[2] - f[4]);
    double eps = (s13 + s24) - 4.0 * f[0];
    double XX = s13 - s24;
    double qx, fxx, fxy, XXu, qy, fyx, fyy, XXv;
    fam_moments(f + 5, lam, qx, fxx, fxy, XXu);
    fam_moments(f + 9, lam, qy, fyx, fyy, XXv);
    const double ir = WIDE ? 1.0 / rho : lbm_rcp(rho);
    const double u = qx * ir, v = qy * ir;
    const double p = M.hg * (rho * rho);
    Jx += r[0] * (qx - Jx);
    Jy += r[1] * (qy - Jy);
    const double k2 = (1.25 * M.a) * (u * u + v * v);
    const double kg = WIDE ? k2 / M.g : div_by(k2, M.g, lbm_rcp(M.g));
    eps += r[2] * (((1.0 - 2.5 * M.a) * rho + kg) - eps);
    XX += r[3] * (0.0 - XX);
    fxx += r[4] * ((qx * u + p) - fxx);
    fxy += r[5] * (qx * v - fxy);
    XXu += r[6] * (0.0 - XXu);
    fyx += r[7] * (qy * u - fyx);
    fyy += r[8] * ((qy * v + p) - fyy);
    XXv += r[9] * (0.0 - XXv);
    const double f0 = 0.2 * (rho - eps);
    const double S = rho - f0;
    const double a = 0.5 * (S + XX), b = 0.5 * (S - XX);
    f[0] = f0;
    f[1] = 0.5 * (a + Jx * il);
    f[3] = 0.5 * (a - Jx * il);
    f[2] = 0.5 * (b + Jy * il);
    f[4] = 0.5 * (b - Jy * il);
    fam_invert(f + 5, il, qx, fxx, fxy, XXu);
    fam_invert(f + 9, il, qy, fyx, fyy, XXv);
}

} // namespace lbm
