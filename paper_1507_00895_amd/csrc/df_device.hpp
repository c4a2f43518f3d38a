// Device helpers shared by the dual-fermion kernels: complex arithmetic,
// global loads and stores, the k-grid.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace df {

// ----------------------------------------------------------------- complex
template <typename T> struct alignas(2 * sizeof(T)) cplx {
    T re, im;
};
using cd = cplx<double>;
using cf = cplx<float>;

template <typename T> __device__ __forceinline__ cplx<T> mk(T r, T i) { return {r, i}; }
template <typename T> __device__ __forceinline__ cplx<T> operator+(cplx<T> a, cplx<T> b) {
    return {a.re + b.re, a.im + b.im};
}
template <typename T> __device__ __forceinline__ cplx<T> operator-(cplx<T> a, cplx<T> b) {
    return {a.re - b.re, a.im - b.im};
}
template <typename T> __device__ __forceinline__ cplx<T> operator*(cplx<T> a, cplx<T> b) {
    return {fma(a.re, b.re, -a.im * b.im), fma(a.re, b.im, a.im * b.re)};
}
template <typename T> __device__ __forceinline__ cplx<T> scale(cplx<T> a, T s) {
    return {a.re * s, a.im * s};
}
template <typename T> __device__ __forceinline__ cplx<T> conj(cplx<T> a) { return {a.re, -a.im}; }
// c - a*b
template <typename T> __device__ __forceinline__ cplx<T> fms(cplx<T> c, cplx<T> a, cplx<T> b) {
    T r = fma(-a.re, b.re, c.re);
    r = fma(a.im, b.im, r);
    T i = fma(-a.re, b.im, c.im);
    i = fma(-a.im, b.re, i);
    return {r, i};
}
// c + a*b
template <typename T> __device__ __forceinline__ cplx<T> fma_c(cplx<T> c, cplx<T> a, cplx<T> b) {
    T r = fma(a.re, b.re, c.re);
    r = fma(-a.im, b.im, r);
    T i = fma(a.re, b.im, c.im);
    i = fma(a.im, b.re, i);
    return {r, i};
}
// 1 / a (Smith's algorithm)
template <typename T> __device__ __forceinline__ cplx<T> recip(cplx<T> a) {
    if (fabs(a.re) >= fabs(a.im)) {
        T r = a.im / a.re;
        T d = a.re + a.im * r;
        T inv = T(1) / d;
        return {inv, -r * inv};
    } else {
        T r = a.re / a.im;
        T d = a.re * r + a.im;
        T inv = T(1) / d;
        return {r * inv, -inv};
    }
}
template <typename T> __device__ __forceinline__ cplx<T> cdiv(cplx<T> a, cplx<T> b) {
    return a * recip(b);
}
template <typename T> __device__ __forceinline__ T cabs1(cplx<T> a) { return fabs(a.re) + fabs(a.im); }

// Every array these kernels read or write through ld/st lives in device
// global memory: say so, so that the compiler emits global (not flat) loads
// and stores, which do not share a wait counter with LDS traffic.
typedef double dv2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ cd ld(const double *p, size_t i) {
    const dv2 v = *(__attribute__((address_space(1))) const dv2 *)(const void *)(p + 2 * i);
    return {v.x, v.y};
}
__device__ __forceinline__ void st(double *p, size_t i, cd v) {
    *(__attribute__((address_space(1))) dv2 *)(void *)(p + 2 * i) = dv2{v.re, v.im};
}
// FP32 pairs and quadruples (element i of an array of them)
typedef float fv2 __attribute__((ext_vector_type(2)));
typedef float fv4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ fv2 ld2f(const float *p, size_t i) {
    return *(__attribute__((address_space(1))) const fv2 *)(const void *)(p + 2 * i);
}
__device__ __forceinline__ fv4 ld4f(const float *p, size_t i) {
    return *(__attribute__((address_space(1))) const fv4 *)(const void *)(p + 4 * i);
}
__device__ __forceinline__ void st2f(float *p, size_t i, float a, float b) {
    *(__attribute__((address_space(1))) fv2 *)(void *)(p + 2 * i) = fv2{a, b};
}
__device__ __forceinline__ void st4f(float *p, size_t i, float a, float b, float c, float d) {
    *(__attribute__((address_space(1))) fv4 *)(void *)(p + 4 * i) = fv4{a, b, c, d};
}

// ----------------------------------------------------------------- k-grid
// Flat index in C order over D axes of nk = 2^lognk points; every axis is a
// field of lognk bits.
struct Grid {
    int D, lognk, nk, N;
};

}  // namespace df
