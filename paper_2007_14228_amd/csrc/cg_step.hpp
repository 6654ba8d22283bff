// Arithmetic of one step of the inner CG (k_cg_step, k_cg_x, k_cg_scalars, k_cgb_iter): the
// element's recurrences and the column's coefficients.  Plain C++ apart from the
// annotations, so that the host tests replay it with g++.
//
// Between the blocks' values a step rounds nothing: z_j, J q_j, z_{j+1} and the
// pair of directions for x are formed in twice the block's digits (FP64: as
// unevaluated sums; FP32: in FP64), and only d_{j+1} and x are rounded, once
// each.  With J q stored and every operation rounded, the error of ten steps was
// 1.10 (FP64) and 1.09 (FP32) times that of the two-term form that keeps r; it is
// 0.92 and 0.88 times (mean of 128 systems a precision, graded meshes, shifts
// -0.05 to -50, replayed against 80-bit arithmetic).
#pragma once
#include <cmath>

#if defined(__HIPCC__)
#define OFKS_HD __host__ __device__ __forceinline__
#else
#define OFKS_HD inline
#endif

namespace ofks {

// z' (returned, for its sum), and d' = z' + be d into dn.  z = dm / dg where FIRST
// (dm holds g), else d - bm dm; z' = z - al q / dg.
template <bool FIRST>
OFKS_HD double cg_element(double q, double d, double dm, double dg, double al, double be, double bm, double &dn) {
#pragma clang fp contract(off)
    const double iv = 1.0 / dg;
    double zh, zl;   // z = zh + zl
    if (FIRST) {
        zh = dm * iv;
        zl = std::fma(-zh, dg, dm) * iv;
    } else {
        const double b = -(bm * dm), bl = std::fma(-bm, dm, -b);
        zh = d + b;
        const double t = zh - d;
        zl = ((d - (zh - t)) + (b - t)) + bl;
    }
    const double qj = q * iv, ql = std::fma(-qj, dg, q) * iv;   // q / dg = qj + ql
    const double u = -(al * qj), ul = std::fma(-al, qj, -u) - al * ql;
    const double sh = zh + u, t = sh - zh;
    const double sl = ((zh - (sh - t)) + (u - t)) + (zl + ul);   // z' = sh + sl
    const double v = be * d, vl = std::fma(be, d, -v);
    const double h = sh + v, t2 = h - sh;
    dn = h + (((sh - (h - t2)) + (v - t2)) + (sl + vl));
    return sh + sl;
}
template <bool FIRST>
OFKS_HD double cg_element(float q, float d, float dm, float dg, float al, float be, float bm, float &dn) {
    const double dgw = dg;
#if defined(__HIP_DEVICE_COMPILE__)
    double iv = __builtin_amdgcn_rcp(dgw);   // to 2^-23 at worst; 2^-45 after a Newton step
    iv = std::fma(std::fma(-dgw, iv, 1.0), iv, iv);
#else
    const double iv = 1.0 / dgw;
#endif
    const double qa = (double)al * (double)q;
    const double z = FIRST ? ((double)dm - qa) * iv : std::fma(-qa, iv, std::fma(-(double)bm, (double)dm, (double)d));
    dn = (float)std::fma((double)be, (double)d, z);
    return z;
}

// x + am dm + al d
OFKS_HD double cg_x2(double x, double am, double dm, double al, double d) {
#pragma clang fp contract(off)
    const double a = am * dm, ae = std::fma(am, dm, -a), b = al * d, bl = std::fma(al, d, -b);
    const double s = x + a, t = s - x, se = (x - (s - t)) + (a - t);
    const double h = s + b, t2 = h - s, he = (s - (h - t2)) + (b - t2);
    return h + ((se + he) + (ae + bl));
}
OFKS_HD float cg_x2(float x, float am, float dm, float al, float d) {
    return (float)std::fma((double)al, (double)d, std::fma((double)am, (double)dm, (double)x));
}

// x + al d for an x carried as x + lo: the new x, and lo for the next (last: x is all)
OFKS_HD double cg_carry(double x, double &lo, double al, double d, bool last) {
#pragma clang fp contract(off)
    const double a = al * d, ae = std::fma(al, d, -a);
    const double s = x + a, t = s - x, l = ((x - (s - t)) + (a - t)) + (lo + ae);
    const double h = s + l;
    lo = last ? 0.0 : l - (h - s);
    return h;
}

// A column's coefficients from its sums dq = <d, T d>, qw = <T d, J T d>, rz =
// <r, z>: alpha (0 where <d, T d> <= 0: nothing is left), and beta from the
// predicted <r', z'> = rz - 2 alpha dq + alpha^2 qw.
//
// The prediction's error is a few roundings of the block's type times rz, so
// beta's is that of a rounding of d, and in FP64 it serves until it is all
// rounding (1e-14 rz: a step that lowers the residual by seven digits or ends
// the solve), where the direction starts anew from z'.  FP32 comes there in
// real use, so below 1e-3 rz beta stays 0 here and old keeps rz (0 elsewhere): once
// the real <r', z'> is summed, d' gets its beta d after all.  An FP32 column whose
// rz has fallen by 24 digits since the start (rz0) stops, before its values
// leave the type's range.
template <typename T> struct CgCoef {
    T alpha, beta;
    double old;
};
template <typename T> OFKS_HD CgCoef<T> cg_coef(double dq, double qw, double rz, double rz0) {
    CgCoef<T> c{T(0), T(0), 0.0};
    if (!(dq > 0.0) || (sizeof(T) == 4 && rz <= 1e-24 * rz0)) return c;
    c.alpha = (T)(rz / dq);
    const double a = (double)c.alpha, next = std::fma(a, std::fma(a, qw, -2.0 * dq), rz);
    if (next > (sizeof(T) == 8 ? 1e-14 : 1e-3) * rz) c.beta = (T)(next / rz);
    else if (sizeof(T) == 4 && rz > 0.0) c.old = rz;
    return c;
}

}  // namespace ofks
