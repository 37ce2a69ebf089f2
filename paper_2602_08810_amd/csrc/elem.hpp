// Real and complex numbers for the scans that come in both.
#pragma once
#include "chain.hpp"
#include <type_traits>

namespace lrnnx {

template <bool CPLX, class F = float> struct Elem;
template <class F> struct Elem<false, F> {
    using T = F;
    static __device__ __forceinline__ T zero() { return 0; }
    static __device__ __forceinline__ T one() { return 1; }
    static __device__ __forceinline__ T mul(T a, T b) { return a * b; }
    static __device__ __forceinline__ T fma(T a, T x, T b) { return a * x + b; }
    static __device__ __forceinline__ T nan() { return __builtin_nanf(""); }
    static __device__ __forceinline__ T conj(T a) { return a; }
    static __device__ __forceinline__ T up(T a, int lanes) { return __shfl_up(a, lanes); }
    static __device__ __forceinline__ T pick(bool c, T a, T b) { return c ? a : b; }
    template <class S> static __device__ __forceinline__ T from(S a) { return (T)a; }
};
template <> __device__ __forceinline__ float Elem<false, float>::fma(float a, float x, float b) { return __builtin_fmaf(a, x, b); }
template <> __device__ __forceinline__ double Elem<false, double>::fma(double a, double x, double b) { return __builtin_fma(a, x, b); }

template <class F> struct Elem<true, F> {
    using T = std::conditional_t<sizeof(F) == 4, float2, double2>;
    static __device__ __forceinline__ T make(F x, F y) { T t; t.x = x; t.y = y; return t; }
    static __device__ __forceinline__ T zero() { return make(0, 0); }
    static __device__ __forceinline__ T one() { return make(1, 0); }
    static __device__ __forceinline__ T mul(T a, T b) { return make(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
    static __device__ __forceinline__ T fma(T a, T b, T c) {
        using R = Elem<false, F>;
        return make(R::fma(a.x, b.x, R::fma(-a.y, b.y, c.x)), R::fma(a.x, b.y, R::fma(a.y, b.x, c.y)));
    }
    static __device__ __forceinline__ T nan() { return make(__builtin_nanf(""), __builtin_nanf("")); }
    static __device__ __forceinline__ T conj(T a) { return make(a.x, -a.y); }
    static __device__ __forceinline__ T up(T a, int lanes) { return make(__shfl_up(a.x, lanes), __shfl_up(a.y, lanes)); }
    static __device__ __forceinline__ T pick(bool c, T a, T b) { return make(c ? a.x : b.x, c ? a.y : b.y); }
    template <class S> static __device__ __forceinline__ T from(S a) { return make((F)a.x, (F)a.y); }
};

}  // namespace lrnnx
