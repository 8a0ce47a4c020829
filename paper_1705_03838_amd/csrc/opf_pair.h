// Unevaluated sums of two doubles (Dekker 1971; products by multiply-add):
// about 106 bits.
//
// Every function turns contraction off: with it, which is hipcc's default, the
// sum of a product and its rounding error becomes one multiply-add, and the
// error is then counted twice (a product right to 53 bits).
#pragma once
#include <cmath>

#include <hip/hip_runtime.h>

namespace opf {

struct dd {
    double hi, lo;
};
__host__ __device__ inline dd two_sum(double a, double b) {
#pragma clang fp contract(off)
    const double s = a + b, t = s - a;
    return {s, (a - (s - t)) + (b - t)};
}
__host__ __device__ inline dd renorm(double a, double b) {  // |a| >= |b|
#pragma clang fp contract(off)
    const double s = a + b;
    return {s, b - (s - a)};
}
__host__ __device__ inline dd operator+(dd a, dd b) {
#pragma clang fp contract(off)
    const dd s = two_sum(a.hi, b.hi), t = two_sum(a.lo, b.lo);
    const dd u = renorm(s.hi, s.lo + t.hi);
    return renorm(u.hi, u.lo + t.lo);
}
__host__ __device__ inline dd operator*(dd a, double b) {
#pragma clang fp contract(off)
    const double p = a.hi * b;
    return renorm(p, fma(a.hi, b, -p) + a.lo * b);
}
__host__ __device__ inline dd madd(dd s, dd a, double b) { return s + a * b; }  // s + a b

}  // namespace opf
