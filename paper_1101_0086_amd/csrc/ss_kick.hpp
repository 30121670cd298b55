// The nonlinear sub-step of Eq. 4 (device code of both split-step paths).
#pragma once

#include "cx.hpp"

namespace mpa {

// cos and sin of phi, |phi| <= 2^20: phi = q pi/2 + r + t with |r| <= pi/4 (pi/2 as its
// 32 leading bits, whose multiples by q < 2^20 are exact, plus a double; t is what r's
// rounding leaves), the Taylor polynomials of sin and cos through r^17 and r^16 (next
// terms below 1e-19 and 2e-18), and the quadrant's signs.  The leading terms r and
// 1 - r^2 / 2 are added last, the rounding of 1 - r^2 / 2 carried: rms error 3.9e-17
// over |phi| <= 2^20, 3.8e-17 for correctly rounded values.
__device__ __forceinline__ cx<double> cis_reduced(double phi) {
    const double q = rint(phi * 0x1.45f306dc9c883p-1);          // 2 / pi
    const double a = fma(-q, 0x1.921fb544p+0, phi);
    const double r = fma(-q, 0x1.0b4611a626331p-34, a);
    const double t = fma(-q, 0x1.0b4611a626331p-34, a - r);
    const double x = r * r;
    double ps = 1.0 / 355687428096000.0, pc = 1.0 / 20922789888000.0;
    ps = fma(x, ps, -1.0 / 1307674368000.0);
    pc = fma(x, pc, -1.0 / 87178291200.0);
    ps = fma(x, ps, 1.0 / 6227020800.0);
    pc = fma(x, pc, 1.0 / 479001600.0);
    ps = fma(x, ps, -1.0 / 39916800.0);
    pc = fma(x, pc, -1.0 / 3628800.0);
    ps = fma(x, ps, 1.0 / 362880.0);
    pc = fma(x, pc, 1.0 / 40320.0);
    ps = fma(x, ps, -1.0 / 5040.0);
    pc = fma(x, pc, -1.0 / 720.0);
    ps = fma(x, ps, 1.0 / 120.0);
    pc = fma(x, pc, 1.0 / 24.0);
    ps = fma(x, ps, -1.0 / 6.0);
    const double h = 0.5 * x, w = 1.0 - h;
    const double s = r + fma(r * x, ps, t * w);
    const double c = w + (((1.0 - w) - h) + fma(x * x, pc, -(r * t)));
    const int k = (int)q;
    const double cs = (k & 1) ? s : c, sn = (k & 1) ? c : s;
    return {((k + 1) & 2) ? -cs : cs, (k & 2) ? -sn : sn};
}

// v_m exp(i phi_m), phi = sigma dz |A|^2, for a thread's 8 points, in one of
// three ways that the largest of their phases decides (one test, not one per
// point, lets the points' polynomials overlap):
//   |phi| <= 1/64 (every step of a weakly nonlinear link): the Taylor polynomials
//     through phi^7 and phi^8 (next terms 1e-20 of sin, 2e-25 of cos).  Their
//     coefficients are products: written as nested divisions (seven FP64 divides
//     a point, 11 instructions each) the kick took longer than the two transforms
//     around it: 84 us per split-step at 2^22 modes, 74 us with products.
//   |phi| <= 2^20: cis_reduced, about 40 operations a point.
//   larger, and infinities: the library's sincos, one point after another (one
//     copy of its code).
// With the library's sincos for every phase above 1/64 a strongly nonlinear run
// waited for its latency, us a step, phases to 2, FP64: 512 modes 4.07, now 2.61
// (2.0 in a weakly nonlinear run); 4096 8.12, 5.96 (4.9); 2^22 105.5, 92.1 (83.8).
// WAVE: the largest phase of the wave decides, so that a wave runs one form only
// (the four-step columns; 2^16 modes, FP64, phases to 1/32: 9.6 us a step when each
// thread decides, 9.2).  In the one-workgroup runs the compiler then keeps the constants
// of every form over the steps and spills (4096 modes 4.86 -> 5.03).  LEAN (kernels held
// to 128 registers, the columns of 1024 points): phases beyond the first form are formed
// again from v, and its points follow one another.
template <bool WAVE, bool LEAN = false>
__device__ __forceinline__ void kick(cx<double> (&v)[8], double sdz) {
    double phi[8], most = 0.0;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        phi[m] = sdz * norm2(v[m]);
        most = fmax(most, fabs(phi[m]));
    }
    const auto beyond = [&](double bound) { return WAVE ? __any(most > bound) != 0 : most > bound; };
    if (!beyond(0.015625)) {
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const double p = phi[m], p2 = p * p;
            const double s = p * fma(p2, fma(p2, fma(p2, -1.0 / 5040.0, 1.0 / 120.0), -1.0 / 6.0), 1.0);
            const double c = fma(p2, fma(p2, fma(p2, fma(p2, 1.0 / 40320.0, -1.0 / 720.0), 1.0 / 24.0), -0.5), 1.0);
            v[m] = cmul(v[m], cx<double>{c, s});
        }
        return;
    }
    if constexpr (LEAN) asm volatile("" : "+v"(sdz));
    if (!beyond(1048576.0)) {
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            v[m] = cmul(v[m], cis_reduced(LEAN ? sdz * norm2(v[m]) : phi[m]));
            if constexpr (LEAN) __builtin_amdgcn_sched_barrier(0);
        }
    } else {
#pragma unroll 1
        for (int m = 0; m < 8; ++m) {
            // the point's registers are picked by selects: one copy of sincos
            double re = v[0].re, im = v[0].im;
#pragma unroll
            for (int q = 1; q < 8; ++q) {
                re = m == q ? v[q].re : re;
                im = m == q ? v[q].im : im;
            }
            double s, c;
            sincos(sdz * norm2(cx<double>{re, im}), &s, &c);
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (m == q) v[q] = cmul(v[q], cx<double>{c, s});
        }
    }
}

}  // namespace mpa
