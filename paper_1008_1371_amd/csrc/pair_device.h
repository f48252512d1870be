// The rotation of one pair for the pairwise kernels that evaluate it in a
// latency-bound chain: the bits of rel_orthogonal and rotation_params in fewer
// instructions.
#pragma once
#include "internal.h"

namespace hsvd {

// Correctly rounded quotient and square root for operands whose exponents are
// moderate (|exponent| below 500, x > 2^-767): the quotient from the hardware's
// reciprocal estimate by two Newton-Raphson steps and a corrected product, the
// root from its reciprocal square root estimate by Goldschmidt's iteration and
// two corrections.  They give the bits of the operators / and sqrt, less the
// scaling steps, which do nothing in that range.
__device__ __forceinline__ double div_lean(double n, double d)
{
    double r = __builtin_amdgcn_rcp(d);
    double e = fma(-d, r, 1.0);
    r = fma(r, e, r);
    e = fma(-d, r, 1.0);
    r = fma(r, e, r);
    const double q = n * r;
    e = fma(-d, q, n);
    return fma(e, r, q);
}

__device__ __forceinline__ double sqrt_lean(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double s = x * y, h = y * 0.5;
    const double e = fma(-h, s, 0.5);
    s = fma(s, e, s);
    h = fma(h, e, h);
    double d = fma(-s, s, x);
    s = fma(d, h, s);
    d = fma(-s, s, x);
    return fma(d, h, s);
}

// The step's rotation of one slot: i and j sides as in rotation_params, the
// skip test (2.3); exact in every case.
struct SlotRotation {
    double t, c;
    bool skip, bad;
};

__device__ __forceinline__ SlotRotation slot_rotation(double aii, double ajj, double aij, bool trig, bool act,
                                                      bool any_hyp, double tol, double tol2, bool tol_ok)
{
    // Skip test: the squared form decides except within 2^-40 of the
    // threshold, where its own rounding could.
    const double lhs = aij * aij, rhs = tol2 * (aii * ajj);
    const bool below = lhs < rhs * (1.0 - 0x1p-40), above = lhs > rhs * (1.0 + 0x1p-40);
    SlotRotation o;
    o.skip = below;
    // rotation_params with the quotients and roots for moderate exponents
    const double two_aij = 2.0 * aij;
    const double num = trig ? (ajj - aii) : -(aii + ajj);
    const double zeta = div_lean(num, two_aij);
    const double az = fabs(zeta);
    const double sg = zeta < 0.0 ? -1.0 : 1.0;
    double root = sqrt_lean(trig ? 1.0 + zeta * zeta : az - 1.0);
    if (any_hyp) root = root * (trig ? 1.0 : sqrt_lean(az + 1.0));
    const double tt = div_lean(sg, az + root);
    const double cin = trig ? 1.0 + tt * tt : (1.0 - tt) * (1.0 + tt);
    o.t = tt;
    o.c = div_lean(1.0, sqrt_lean(cin));
    o.bad = !trig && !(az > 1.0);
    // entries in [2^-300, 2^300), |zeta| < 2^400, else the general routines
    const unsigned lo = (1023u - 300u) << 20, len = 600u << 20;
    const unsigned ei = (unsigned)__double2hiint(aii) - lo, ej = (unsigned)__double2hiint(ajj) - lo;
    const bool odd = act && (!tol_ok || max(ei, ej) >= len ||
                             (!below && (!above || (unsigned)__double2hiint(az) >= (1023u + 400u) << 20)));
    if (__builtin_expect(__ballot(odd) != 0ull, 0)) {
        if (odd) {
            o.skip = rel_orthogonal(aii, ajj, aij, tol);
            o.bad = rotation_params(aii, ajj, aij, trig ? -1 : 1, o.t, o.c) != 0;
        }
    }
    return o;
}

}  // namespace hsvd
