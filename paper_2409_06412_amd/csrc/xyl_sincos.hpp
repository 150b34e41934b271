// FP64 sine and cosine of lattice angles together.
#pragma once
#include <hip/hip_runtime.h>

namespace xyl {

// Cody-Waite reduction by pi/2 in two parts (the second exact to 2^-108, so
// that the reduced angle r + t is good to well below an ulp of itself for the
// multiples that arise here), then the Taylor series on [-pi/4, pi/4] to
// degrees 17 and 18 (the first terms left out are below 2^-63), with the
// reduction's tail t and the rounding of r^2 carried to first order.  Over
// 10^6 angles of up to 3 pi at most 0.74 ulp off, 0.290 root mean square (the
// general routine: 0.78 and 0.293), in about 45 operations against some 110
// instructions of FP64 arithmetic.  A caller takes the general routine for
// what is beyond 10 (a lattice's q theta is within 3 pi) or not finite.
__device__ __forceinline__ void sincos_reduced(double x, double& s_out, double& c_out) {
    const double k = __builtin_rint(x * 0.63661977236758134308);   // 2 / pi
    const double r0 = __builtin_fma(-k, 0x1.921fb54442d18p+0, x);
    const double r = __builtin_fma(-k, 0x1.1a62633145c07p-54, r0);
    const double t = __builtin_fma(-k, 0x1.1a62633145c07p-54, r0 - r);
    const double z = r * r, ez = __builtin_fma(r, r, -z);
    double p = 0x1.952c77030ad4ap-49;
    p = __builtin_fma(p, z, -0x1.ae7f3e733b81fp-41);
    p = __builtin_fma(p, z, 0x1.6124613a86d09p-33);
    p = __builtin_fma(p, z, -0x1.ae64567f544e4p-26);
    p = __builtin_fma(p, z, 0x1.71de3a556c734p-19);
    p = __builtin_fma(p, z, -0x1.a01a01a01a01ap-13);
    p = __builtin_fma(p, z, 0x1.1111111111111p-7);
    p = __builtin_fma(p, z, -0x1.5555555555555p-3);
    double q = -0x1.6827863b97d97p-53;
    q = __builtin_fma(q, z, 0x1.ae7f3e733b81fp-45);
    q = __builtin_fma(q, z, -0x1.93974a8c07c9dp-37);
    q = __builtin_fma(q, z, 0x1.1eed8eff8d898p-29);
    q = __builtin_fma(q, z, -0x1.27e4fb7789f5cp-22);
    q = __builtin_fma(q, z, 0x1.a01a01a01a01ap-16);
    q = __builtin_fma(q, z, -0x1.6c16c16c16c17p-10);
    q = __builtin_fma(q, z, 0x1.5555555555555p-5);
    const double h = 0.5 * z, w = 1.0 - h;
    const double sn = r + __builtin_fma(r * z, p, t * w);
    const double cs = w + (((1.0 - w) - h) + __builtin_fma(z * z, q, __builtin_fma(-0.5, ez, -(r * t))));
    const int n = (int)k;
    const double a = (n & 1) ? cs : sn, b = (n & 1) ? sn : cs;
    s_out = (n & 2) ? -a : a;
    c_out = ((n + 1) & 2) ? -b : b;
}

// The arguments that sincos_reduced is for, and the general routine for the
// others, out of line: its registers would otherwise cost every caller.
__device__ __forceinline__ bool sincos_reducible(double x) { return __builtin_fabs(x) <= 10.0; }
static __device__ __noinline__ double2 sincos_general(double x) {
    double s, c;
    ::sincos(x, &s, &c);
    return make_double2(c, s);
}
__device__ __forceinline__ void sincos_angle(double x, double& s, double& c) {
    sincos_reduced(x, s, c);
    if (__builtin_expect(!sincos_reducible(x), 0)) {
        const double2 z = sincos_general(x);
        c = z.x;
        s = z.y;
    }
}

}  // namespace xyl
