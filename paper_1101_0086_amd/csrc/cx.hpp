// Complex arithmetic on interleaved (re, im) pairs for device code.
#pragma once

#include <hip/hip_runtime.h>

namespace mpa {

template <typename T>
struct __align__(2 * sizeof(T)) cx {
    T re, im;
};

template <typename T>
__device__ __forceinline__ cx<T> mk(T re, T im) { return cx<T>{re, im}; }

template <typename T>
__device__ __forceinline__ cx<T> operator+(cx<T> a, cx<T> b) { return {a.re + b.re, a.im + b.im}; }

template <typename T>
__device__ __forceinline__ cx<T> operator-(cx<T> a, cx<T> b) { return {a.re - b.re, a.im - b.im}; }

// Products are written with explicit fused multiply-adds, so that which
// product of a sum is fused is fixed by the source rather than chosen by the
// compiler per call site: the same operation then rounds the same way in
// every kernel that uses it (the fused and node-parallel schedules rely on
// this to produce the same field).  A scaled value is rounded before it is
// added (its products may not be fused into a transform's first additions,
// which the compiler did in one kernel and not in another).
template <typename T>
__device__ __forceinline__ cx<T> scale(cx<T> a, T s) {
#pragma clang fp contract(off)
    return {a.re * s, a.im * s};
}

// a s + b
template <typename T>
__device__ __forceinline__ cx<T> mad(cx<T> a, T s, cx<T> b) { return {fma(a.re, s, b.re), fma(a.im, s, b.im)}; }

// a * b
template <typename T>
__device__ __forceinline__ cx<T> cmul(cx<T> a, cx<T> b) {
    return {fma(a.re, b.re, -(a.im * b.im)), fma(a.re, b.im, a.im * b.re)};
}

// a * conj(b)
template <typename T>
__device__ __forceinline__ cx<T> cmulc(cx<T> a, cx<T> b) {
    return {fma(a.re, b.re, a.im * b.im), fma(a.im, b.re, -(a.re * b.im))};
}

// multiply by +i (SIGN = +1) or -i (SIGN = -1)
template <int SIGN, typename T>
__device__ __forceinline__ cx<T> rot(cx<T> a) {
    if constexpr (SIGN > 0) return {-a.im, a.re};
    else return {a.im, -a.re};
}

template <typename T>
__device__ __forceinline__ T norm2(cx<T> a) { return fma(a.re, a.re, a.im * a.im); }

// The nonlinearity of a node is c |a|^2 a, a = F^-1[psi e^{i beta}] before its
// scale c_l, with c = c_l^3 d_l (cube_scale) in place of scaling A by c_l and
// the increment by d_l = sigma dz e^{-Gamma_l} (five products instead of
// eight per point).  |a|^2 is B^2 |A|^2 before the factor: in range up to
// |A|^2 = 2e31 at B = 4096 in FP32, where |A|^3 ends at 5e25.  c |a|^2 is the
// factor of the point in the transform that follows (block_fft_scaled).
template <typename T>
__device__ __forceinline__ T cube_factor(cx<T> a, T c) { return norm2(a) * c; }

template <typename T>
__device__ __forceinline__ T cube_scale(T cl, T dl) {
    const double c = cl;
    return T(c * c * c * double(dl));
}

}  // namespace mpa
