// The nonlinear sub-step of Eq. 4 (device code of both split-step paths).
#pragma once

#include "cx.hpp"

namespace mpa {

// v_m exp(i phi_m), phi = sigma dz |A|^2, for a thread's 8 points.  For
// |phi| <= 1/64 at all of them (every step of a weakly nonlinear link) sin and
// cos are their Taylor polynomials through phi^7 and phi^8 (truncation below
// 2e-22 relative); larger phi takes the library's sincos.  The coefficients
// are products: written as nested divisions (seven FP64 divides a point, 11
// instructions each) the kick took longer than the two transforms around it:
// 84 us per split-step at 2^22 modes, 74 us with products.
// One test per thread, not per point, lets the points' polynomials overlap.
__device__ __forceinline__ void kick(cx<double> (&v)[8], double sdz) {
    double phi[8], most = 0.0;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        phi[m] = sdz * norm2(v[m]);
        most = fmax(most, fabs(phi[m]));
    }
    if (most <= 0.015625) {
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const double p = phi[m], p2 = p * p;
            const double s = p * fma(p2, fma(p2, fma(p2, -1.0 / 5040.0, 1.0 / 120.0), -1.0 / 6.0), 1.0);
            const double c = fma(p2, fma(p2, fma(p2, fma(p2, 1.0 / 40320.0, -1.0 / 720.0), 1.0 / 24.0), -0.5), 1.0);
            v[m] = cmul(v[m], cx<double>{c, s});
        }
    } else {
#pragma unroll 1
        for (int m = 0; m < 8; ++m) {
            // the point's registers are picked by selects: one copy of sincos
            double ph = phi[0];
#pragma unroll
            for (int q = 1; q < 8; ++q) ph = m == q ? phi[q] : ph;
            double s, c;
            sincos(ph, &s, &c);
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (m == q) v[q] = cmul(v[q], cx<double>{c, s});
        }
    }
}

}  // namespace mpa
