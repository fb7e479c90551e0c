// Scalar types of the device code: double, and forward-mode dual numbers with K
// tangent lanes (exact Jacobian-vector products and K seeded columns of the element
// blocks).  Non-smooth operations follow one convention everywhere: max/min return
// the first argument on ties, |x| has slope +1 at x = 0, and the tangent of the
// branch not taken is never propagated.
#pragma once
#include <hip/hip_runtime.h>

#define FR_HD __host__ __device__ __forceinline__

template <int K>
struct Dual {
    double v;
    double d[K];
};

FR_HD double val(double x) { return x; }
template <int K> FR_HD double val(const Dual<K>& x) { return x.v; }

// ---- reciprocal: hardware estimate refined by two Newton steps (error well below 1 ulp
// of the quantities it feeds; replaces the much longer IEEE division sequence)
__device__ __forceinline__ double frcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    r = fma(fma(-x, r, 1.0), r, r);
    return r;
}
__device__ __forceinline__ double rcp(double x) { return frcp(x); }
template <int K> __device__ __forceinline__ Dual<K> rcp(const Dual<K>& a) { Dual<K> r; r.v = frcp(a.v);
    const double s = -r.v * r.v;
#pragma unroll
    for (int k = 0; k < K; ++k) r.d[k] = a.d[k] * s; return r; }

template <int K> FR_HD Dual<K> mkconst(double a) { Dual<K> r; r.v = a;
#pragma unroll
    for (int k = 0; k < K; ++k) r.d[k] = 0.0; return r; }

// ---- arithmetic
template <int K> FR_HD Dual<K> operator+(const Dual<K>& a, const Dual<K>& b) { Dual<K> r; r.v = a.v + b.v;
#pragma unroll
    for (int k = 0; k < K; ++k) r.d[k] = a.d[k] + b.d[k]; return r; }
template <int K> FR_HD Dual<K> operator-(const Dual<K>& a, const Dual<K>& b) { Dual<K> r; r.v = a.v - b.v;
#pragma unroll
    for (int k = 0; k < K; ++k) r.d[k] = a.d[k] - b.d[k]; return r; }
template <int K> FR_HD Dual<K> operator-(const Dual<K>& a) { Dual<K> r; r.v = -a.v;
#pragma unroll
    for (int k = 0; k < K; ++k) r.d[k] = -a.d[k]; return r; }
template <int K> FR_HD Dual<K> operator*(const Dual<K>& a, const Dual<K>& b) { Dual<K> r; r.v = a.v * b.v;
#pragma unroll
    for (int k = 0; k < K; ++k) r.d[k] = a.d[k] * b.v + a.v * b.d[k]; return r; }
template <int K> __device__ __forceinline__ Dual<K> operator/(const Dual<K>& a, const Dual<K>& b) { Dual<K> r;
    const double ib = frcp(b.v);
    r.v = a.v * ib;
#pragma unroll
    for (int k = 0; k < K; ++k) r.d[k] = (a.d[k] - r.v * b.d[k]) * ib; return r; }
template <int K> FR_HD Dual<K> operator+(const Dual<K>& a, double b) { Dual<K> r = a; r.v += b; return r; }
template <int K> FR_HD Dual<K> operator+(double b, const Dual<K>& a) { Dual<K> r = a; r.v += b; return r; }
template <int K> FR_HD Dual<K> operator-(const Dual<K>& a, double b) { Dual<K> r = a; r.v -= b; return r; }
template <int K> FR_HD Dual<K> operator-(double b, const Dual<K>& a) { Dual<K> r; r.v = b - a.v;
#pragma unroll
    for (int k = 0; k < K; ++k) r.d[k] = -a.d[k]; return r; }
template <int K> FR_HD Dual<K> operator*(const Dual<K>& a, double b) { Dual<K> r; r.v = a.v * b;
#pragma unroll
    for (int k = 0; k < K; ++k) r.d[k] = a.d[k] * b; return r; }
template <int K> FR_HD Dual<K> operator*(double b, const Dual<K>& a) { return a * b; }
template <int K> FR_HD Dual<K> operator/(const Dual<K>& a, double b) { return a * (1.0 / b); }
template <int K> FR_HD Dual<K> operator/(double a, const Dual<K>& b) { Dual<K> r; r.v = a / b.v;
    const double s = -r.v / b.v;
#pragma unroll
    for (int k = 0; k < K; ++k) r.d[k] = s * b.d[k]; return r; }
template <int K> FR_HD Dual<K>& operator+=(Dual<K>& a, const Dual<K>& b) { a = a + b; return a; }
template <int K> FR_HD Dual<K>& operator-=(Dual<K>& a, const Dual<K>& b) { a = a - b; return a; }

// fused multiply-add on the value; tangent by the product rule
FR_HD double fma_(double a, double b, double c) { return fma(a, b, c); }
template <int K> FR_HD Dual<K> fma_(double a, const Dual<K>& b, const Dual<K>& c) { Dual<K> r; r.v = fma(a, b.v, c.v);
#pragma unroll
    for (int k = 0; k < K; ++k) r.d[k] = fma(a, b.d[k], c.d[k]); return r; }

// ---- elementary functions
// square root g and half its reciprocal h = 1 / (2 sqrt(x)) from an estimate y of 1/sqrt(x) good to
// 2^-23: coupled Newton steps for both (Goldschmidt's iteration), then a residual step for g, which
// equals sqrt(x) but for an ulp in rare cases (none of 50 million), and a Newton step for h on that g:
// no further off than 0.5 / sqrt(x) rounded twice, 1.5 ulp.  For normal x > 0; zeros, negatives and infinities give NaN (the callers' quantities
// are not finite there in any case).  sqrt() and a division took 17 and 12 more instructions.
FR_HD void sqrt_steps(double x, double y, double& g, double& h) {
    g = x * y;
    h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    g = fma(fma(-g, g, x), h, g);
    h = fma(h, fma(-h, g + g, 1.0), h);
}
__device__ __forceinline__ void fsqrt_both(double x, double& g, double& h) {
    sqrt_steps(x, __builtin_amdgcn_rsq(x), g, h);
}
__device__ __forceinline__ double ssqrt(double x) {
    double g, h;
    fsqrt_both(x, g, h);
    return g;
}
template <int K> __device__ __forceinline__ Dual<K> ssqrt(const Dual<K>& a) { Dual<K> r;
    double h;
    fsqrt_both(a.v, r.v, h);
#pragma unroll
    for (int k = 0; k < K; ++k) r.d[k] = a.d[k] * h; return r; }
FR_HD double sabs(double x) { return x >= 0.0 ? x : -x; }
template <int K> FR_HD Dual<K> sabs(const Dual<K>& a) { return a.v >= 0.0 ? a : -a; }
template <class T> FR_HD T smax(const T& a, const T& b) { return val(a) >= val(b) ? a : b; }
template <class T> FR_HD T smin(const T& a, const T& b) { return val(a) <= val(b) ? a : b; }

// generic constant constructor
template <class T> struct Make { FR_HD static T c(double a) { return T(a); } };
template <int K> struct Make<Dual<K>> { FR_HD static Dual<K> c(double a) { return mkconst<K>(a); } };
template <class T> FR_HD T cst(double a) { return Make<T>::c(a); }

// ---- memory helpers: a T is stored as (1 + K) consecutive doubles
template <class T> struct Store;
template <> struct Store<double> {
    static constexpr int W = 1;
    FR_HD static double ld(const double* p) { return *p; }
    FR_HD static void st(double* p, double x) { *p = x; }
};
template <int K> struct Store<Dual<K>> {
    static constexpr int W = 1 + K;
    FR_HD static Dual<K> ld(const double* p) { Dual<K> r; r.v = p[0];
#pragma unroll
        for (int k = 0; k < K; ++k) r.d[k] = p[1 + k]; return r; }
    FR_HD static void st(double* p, const Dual<K>& x) { p[0] = x.v;
#pragma unroll
        for (int k = 0; k < K; ++k) p[1 + k] = x.d[k]; }
};
