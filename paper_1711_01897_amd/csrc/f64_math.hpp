// FP64 building blocks of the entry kernels: the reciprocal square root and
// e^{ikr} without the library functions' special cases.
//
// The FP64 kernels are bound by FP64 instructions (full rate, no trans unit
// for the polynomials), so what a point pair costs is their count.  The
// library's sincos carries a reduction for arguments of any size and a
// quadrant swap; here the phase is taken in half turns, reduced exactly, and
// one sign serves sine and cosine: 27 instructions.  Helmholtz single layer
// P1, 501 x 1000 entries, 6-point rule: the entry kernel takes 472 us where it
// took 1,259 us with the library's functions and a dynamically indexed lane
// record (55 instructions per point pair, 0.82 of the FP64 issue rate).
#pragma once

#include <hip/hip_runtime.h>

namespace bem {

// 1 / sqrt(x): the hardware estimate y0 and one third-order step on the
// residual e = 1 - x y0^2 (y0 (1 - e)^{-1/2} = y0 (1 + e/2 + 3/8 e^2 + ...)).
// x = 0 gives infinity (coincident points of a mesh that is not welded): there
// e is not a number, which fmin replaces by 1 and leaves y0 = infinity.
__device__ __forceinline__ double rsqrt64(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fmin(fma(-x * y, y, 1.0), 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// The wavenumber as the phase needs it: k / pi (half turns per unit length) as
// a sum of two doubles, and the distance (double layer) or its square (else) that
// ends the phase: 2^50 half turns, past which a rounding of r turns the phase by as
// much as it likes.  Beyond it the phase must only stay what cis64 can reduce (the
// amplitude is still the true r's).  One minimum in 55 instructions.
struct Wave64 {
    double k, h, l, end;
};

// e^{ikr} up to a sign: returns cos and sin of pi f, f in [-1/2, 1/2] the
// phase in half turns past the nearest whole number n, and that number's
// parity in bit 31 of `flip` (set: both change sign).  r h is split exactly
// into n + f by the fused product, so the phase carries no rounding of k r.
// n comes from adding 1.5 x 2^52, which leaves its parity in the last bit of
// the sum (phases up to 2^51 half turns; Wave64::end keeps them there).
// Polynomials in f^2: minimax fits (Remez exchange in 60 digits) of
// sin(pi f) / f and (cos(pi f) - 1) / f^2 on f^2 in [0, 1/4], errors 6.5e-19
// relative and 1.6e-17 absolute.
__device__ __forceinline__ void cis64(double r, const Wave64 &w, double &cs, double &sn, unsigned &flip)
{
    const double p = r * w.h;
    const double t = p + 0x1.8p52;
    const double n = t - 0x1.8p52;
    const double f = (p - n) + fma(r, w.l, fma(r, w.h, -p));
    flip = (unsigned)__double2loint(t) << 31;
    const double z = f * f;
    double s = 7.697867842612836e-07;
    s = fma(s, z, -2.190350118138285e-05);
    s = fma(s, z, 0.00046629981785790416);
    s = fma(s, z, -0.007370430506269734);
    s = fma(s, z, 0.08214588657314423);
    s = fma(s, z, -0.5992645293189474);
    s = fma(s, z, 2.5501640398773007);
    s = fma(s, z, -5.167712780049969);
    s = fma(s, z, 3.141592653589793);
    sn = s * f;
    double c = 4.166426859672091e-06;
    c = fma(c, z, -0.00010458288765729972);
    c = fma(c, z, 0.0019295626607217936);
    c = fma(c, z, -0.025806890027280493);
    c = fma(c, z, 0.23533063027228068);
    c = fma(c, z, -1.3352627688518854);
    c = fma(c, z, 4.058712126416736);
    c = fma(c, z, -4.934802200544679);
    cs = fma(c, z, 1.0);
}

__device__ __forceinline__ double flip_sign(double x, unsigned flip)
{
    return __hiloint2double(__double2hiint(x) ^ (int)flip, __double2loint(x));
}

}  // namespace bem
